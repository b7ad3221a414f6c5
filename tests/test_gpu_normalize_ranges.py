"""gcn_normalize from 2^31 keys on, where they are sorted in ranges: its workspace,
and its result on long lists of few different edges, bit for bit the CSR of those
edges alone (repeats collapse): several ranges, a hub whose row is more than a
range, one edge that is, 32-bit and 64-bit keys, dense output, a bad id."""
import pytest
import torch

from paper_2010_12635_amd import gcn as G


# 32-bit and 64-bit keys; the last two as long as the device memory allows
@pytest.mark.parametrize("n,E", [(65536, 1 << 30), (1 << 22, 1 << 30), (1 << 27, 1 << 31), (1 << 28, 1 << 32)])
def test_workspace(n, E):
    """The 4 bytes per key and 25 per vertex that counting and scattering the
    edges by row would take, not the 16 of two buffers of all keys."""
    keys = 2 * E + n
    assert G.gcn_normalize_workspace_size(n, E) <= 4.7 * keys
    below = ((1 << 31) - 1 - n) // 2
    assert G.gcn_normalize_workspace_size(n, below) >= (8 if n <= 65536 else 16) * (2 * below + n)


def build(n, src, dst, prec, with_dense=False):
    cap = 2 * src.numel() + n
    out = dict(rowptr=torch.full((n + 1,), -1, dtype=torch.int64, device="cuda"),
               colidx=torch.empty(cap, dtype=torch.int32, device="cuda"),
               deg=torch.empty(n, dtype=torch.int32, device="cuda"),
               dinv=torch.empty(n, device="cuda"),
               values=torch.empty(cap, dtype=G.torch_dtype(prec), device="cuda"))
    ld = (n + 7) // 8 * 8
    dense = torch.full((n, ld), 3.0, dtype=G.torch_dtype(prec), device="cuda") if with_dense else None
    ws = torch.empty(G.gcn_normalize_workspace_size(n, src.numel()), dtype=torch.uint8, device="cuda")
    nnz = G.gcn_normalize(n, src, dst, G.GCN_I64, out["rowptr"], out["colidx"], out["deg"], out["dinv"], prec,
                          out["values"], dense, ld, ws)
    for k in ("colidx", "values"):
        out[k] = out[k][:nnz].clone()
    return out, dense


E_LONG = (1 << 30) + 12345


def edges(kind, n, gen):
    """A few million edges, and the index of one of them at every place of the list."""
    m = 3_000_001
    u, v = (torch.randint(0, n, (m,), generator=gen, device="cuda", dtype=torch.int32) for _ in range(2))
    pick = torch.randint(0, m, (E_LONG,), generator=gen, device="cuda", dtype=torch.int32)
    if kind == "hub":                                    # 3 of 4 places: an edge of vertex n / 3
        k = 2_000_000
        u[:k] = n // 3
        pick = torch.where(torch.randint(0, 4, (E_LONG,), generator=gen, device="cuda", dtype=torch.int8) > 0,
                           pick % k, pick)
    if kind == "one":                                    # 7 of 10 places: one edge
        pick = torch.where(torch.randint(0, 10, (E_LONG,), generator=gen, device="cuda", dtype=torch.int8) > 2,
                           torch.full_like(pick, 5), pick)
    return u, v, pick


def take(x, pick):
    out = torch.empty(pick.numel(), dtype=x.dtype, device=x.device)
    for lo in range(0, pick.numel(), 1 << 27):
        out[lo:lo + (1 << 27)] = x[pick[lo:lo + (1 << 27)].long()]
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("n,kind,prec", [(65536, "hub", 1), (3_000_000, "even", 0), (3_000_000, "hub", 2),
                                         (70001, "one", 1), (1000, "one", 0)])
def test_long_list(n, kind, prec):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    u, v, pick = edges(kind, n, gen)
    here = torch.zeros(u.numel(), dtype=torch.bool, device="cuda")
    for lo in range(0, pick.numel(), 1 << 27):
        here[pick[lo:lo + (1 << 27)].long()] = True
    with_dense = n == 1000
    want, wd = build(n, u[here].contiguous(), v[here].contiguous(), prec, with_dense)
    src, dst = take(u, pick), take(v, pick)
    del pick
    print(f"[ranges] n={n} {kind}: normalize", flush=True)
    got, gd = build(n, src, dst, prec, with_dense)
    for k in want:
        assert torch.equal(got[k], want[k]), k
    if with_dense:
        assert torch.equal(gd, wd)
    if kind == "one":                                    # an id outside [0, n) is still refused
        src[E_LONG - 1] = n
        with pytest.raises(G.GcnError) as e:
            build(n, src, dst, prec)
        assert e.value.status == 8                       # GCN_ERR_GRAPH
