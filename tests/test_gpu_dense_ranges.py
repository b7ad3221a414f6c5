"""The tiled dense aggregation where its row blocks, column tiles and k
ranges end, ragged n and F, in every storage type, against float64 on the
stored values: F <= 64 with 64-row blocks alone and 128-row blocks with one and
with several k ranges (fewer row blocks than compute units, or a last round of
them nearly empty); wider F with each tile of the matrix-core kernel, whole
and cut k ranges, odd and even chunk counts; and the k ranges of whole layers,
with a workspace and in the fixed scratch."""
import ctypes

import pytest
import torch

from paper_2010_12635_amd import gcn as G

PNAME = {0: "f32", 1: "f16", 2: "bf16"}


def tile(A, prec):
    """A (n x n, storage dtype) in the tiled operand order documented in gcn.h."""
    n = A.shape[0]
    kc = 16 if prec == G.GCN_F32 else 32
    nc, nb = (n + kc - 1) // kc, (n + 63) // 64
    P = torch.zeros((nb * 64, nc * kc), dtype=A.dtype, device=A.device)
    P[:n, :n] = A
    return P.view(nb, 4, 16, nc, 4, kc // 4).permute(0, 3, 1, 4, 2, 5).contiguous().view(-1)


CASES = [
    # 16-bit: 64-row blocks (the first two), several ranges, 128-row blocks over the whole range
    (1, 300, 64), (1, 2048, 33), (1, 6001, 64), (2, 8200, 17), (1, 9000, 48), (2, 20000, 50), (1, 32768, 64),
    # fp32: 64-row blocks (n = 140 and F = 1), ranges of 69 to 1250 chunks
    (0, 140, 64), (0, 1100, 64), (0, 2049, 1), (0, 2048, 32), (0, 3001, 16), (0, 6001, 48), (0, 8191, 63),
    (0, 20000, 64),
    # wide: 64-row blocks (n up to 1100; n = 2529), 128 x 128, 256 x 128, 256 x 192 and 256 x 256 tiles
    (1, 257, 70), (1, 1100, 100), (2, 1100, 520), (1, 2500, 130), (2, 2529, 200), (1, 4096, 1000), (2, 6000, 250),
    (1, 6001, 2040), (1, 8200, 380), (2, 12000, 129), (1, 12001, 1000), (1, 16384, 100), (2, 16384, 512),
    (0, 257, 70), (0, 700, 300), (0, 2500, 192), (0, 4100, 200), (0, 5001, 1030),
]


@pytest.mark.gpu
@pytest.mark.parametrize("prec,n,F", CASES, ids=lambda v: str(v))
def test_tiled_aggregation(prec, n, F):
    dt = G.torch_dtype(prec)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + F)
    A = torch.rand((n, n), generator=gen, device="cuda").to(dt)
    ld = (F + 7) // 8 * 8
    X = torch.zeros((n, ld), dtype=dt, device="cuda")
    X[:, :F] = torch.randn((n, F), generator=gen, device="cuda").to(dt)
    bias = torch.randn(ld, generator=gen, device="cuda")
    At = tile(A, prec)
    a = G.GcnAdj()
    a.n, a.nnz, a.format, a.value_prec, a.dense = n, 0, G.GCN_DENSE_TILED, prec, At.data_ptr()
    Y = torch.full((n, ld), float("nan"), dtype=dt, device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(G.gcn_aggregate_workspace_size(a, F, prec), dtype=torch.uint8, device="cuda")
    out = []
    for _ in range(2):
        G.gcn_aggregate(a, F, prec, X, ld, bias, G.GCN_ACT_RELU, 0.0, False, 0, 0, 0, Y, ld, flag, ws)
        out.append(Y[:, :F].clone())
    assert torch.equal(out[0], out[1])               # run-to-run identical
    assert flag.item() == 0
    Ad, Xd = A.double(), X[:, :F].double()
    want = (Ad @ Xd + bias[:F].double()).clamp_(min=0)
    # n terms summed in fp32 in some order, then one rounding to storage
    mag = Ad @ Xd.abs() + bias[:F].double().abs()
    u = {0: 2.0 ** -24, 1: 2.0 ** -11, 2: 2.0 ** -8}[prec]
    bound = (n + 1) * 2.0 ** -24 * mag + u * want + 1e-30
    assert bool(((Y[:, :F].double() - want).abs() <= bound).all())
    # a non-finite input stays in its own rows and columns
    X[n - 1, F - 1] = float("inf")
    G.gcn_aggregate(a, F, prec, X, ld, None, G.GCN_ACT_NONE, 0.0, False, 0, 0, 0, Y, ld, flag, ws)
    fin = torch.isfinite(Y[:, :F].float())
    assert bool(fin[:, :F - 1].all()) and not bool(fin[A[:, n - 1] > 0, F - 1].any()) and flag.item() == 1


@pytest.mark.gpu
@pytest.mark.parametrize("n,F,chains", [(20928, 16, 8), (880, 80, 8), (8192, 128, 8), (8192, 100, 8), (24000, 160, 8),
                                        (7076, 504, 2), (1433, 778, 4)])
def test_fp32_sums_keep_to_short_chains(n, F, chains):
    """On a full A_hat an fp32 output is the sum of several chains of additions.
    A chain of m additions of zero-mean terms, four products each, has partial
    sums of rms sqrt(4 k) s after k of them and a rounding error of at most 2^-24
    of it each time: 2^-24 s sqrt(2) m in all, `chains` of them with m = n / (4
    chains) against the result's rms sqrt(n) s: 2^-24 sqrt(n / (8 chains))."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + F)
    A = torch.randn((n, n), generator=gen, device="cuda")
    X = torch.randn((n, F), generator=gen, device="cuda")
    At = tile(A, G.GCN_F32)
    a = _adj(n, G.GCN_F32, At.data_ptr())
    ld = (F + 7) // 8 * 8
    X = torch.nn.functional.pad(X, (0, ld - F)).contiguous()
    Y = torch.empty_like(X)
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(G.gcn_aggregate_workspace_size(a, F, G.GCN_F32), dtype=torch.uint8, device="cuda")
    G.gcn_aggregate(a, F, G.GCN_F32, X, ld, None, G.GCN_ACT_NONE, 0.0, False, 0, 0, 0, Y, ld, flag, ws)
    rows = torch.arange(0, n, 8, device="cuda")
    want = A[rows].double() @ X[:, :F].double()
    err = float((Y[rows, :F].double() - want).norm() / want.norm())
    assert err <= 2.0 ** -24 * (n / (8 * chains)) ** 0.5, err


def plan(prec, n, F):
    """(kernel, rows, columns, k ranges, chunks of the longest range, chunks of its
    chains) of a tiled product."""
    out = (ctypes.c_int64 * 6)()
    G.lib().gcn_internal_dense_plan(ctypes.c_int32(prec), ctypes.c_int64(n), ctypes.c_int64(F), out)
    return tuple(out)


def _adj(n, prec, dense):
    a = G.GcnAdj()
    a.n, a.nnz, a.format, a.value_prec, a.dense = n, 0, G.GCN_DENSE_TILED, prec, dense
    return a


def _layer(f_in, f_out):
    return G.GcnLayer(f_in, f_out, (f_in + 7) // 8 * 8, (f_out + 7) // 8 * 8, G.GCN_ACT_NONE, 0.0, 0, 0)


# partials of 23 to 88 MB: with the transposed columns more than
# GCN_NOALLOC_SCRATCH_BYTES in all but the first two
LAYERS = [(1, 6001, 16, 64), (2, 12000, 40, 256), (1, 12000, 24, 384), (2, 16384, 16, 512), (1, 20000, 16, 256),
          (0, 20000, 16, 128)]


@pytest.mark.parametrize("prec,n,f_in,f_out", LAYERS)
def test_layer_workspace_holds_every_range(prec, n, f_in, f_out):
    """A layer call cuts the k range as gcn_aggregate does: its workspace has
    room for the transposed columns and the partials of all ranges."""
    ranges = plan(prec, n, f_out)[3]
    assert ranges > 1
    size = G.gcn_layer_workspace_size(_adj(n, prec, 4096), _layer(f_in, f_out), prec)   # never read
    assert size >= n * f_out * (4 if prec == 0 else 2) + ranges * n * f_out * 4


def _operands(prec, n, f_in, f_out):
    dt = G.torch_dtype(prec)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + f_out)
    At = tile(torch.rand((n, n), generator=gen, device="cuda").to(dt), prec)
    H = torch.relu(torch.randn((n, f_in), generator=gen, device="cuda")).to(dt)
    W = torch.randn((f_in, f_out), generator=gen, device="cuda").to(dt)
    dZ = torch.randn((n, f_out), generator=gen, device="cuda").to(dt)
    return _adj(n, prec, At.data_ptr()), At, H, W, dZ


@pytest.mark.gpu
@pytest.mark.parametrize("prec,n,f_in,f_out", LAYERS)
def test_layer_forward_is_transform_and_aggregate(prec, n, f_in, f_out):
    a, At, H, W, X = _operands(prec, n, f_in, f_out)
    L = _layer(f_in, f_out)
    ov = torch.zeros(1, dtype=torch.int32, device="cuda")
    S, Y, S2, Y2 = (torch.empty_like(X) for _ in range(4))
    ws = torch.empty(G.gcn_layer_workspace_size(a, L, prec), dtype=torch.uint8, device="cuda")
    G.gcn_layer_fwd(a, L, prec, False, H, W, None, 0, 0, S, Y, ov, ws)
    wt = torch.empty(G.gcn_transform_workspace_size(n, f_in, f_out, prec), dtype=torch.uint8, device="cuda")
    G.gcn_transform(n, f_in, f_out, prec, H, f_in, W, f_out, S2, f_out, ov, wt)
    wa = torch.empty(G.gcn_aggregate_workspace_size(a, f_out, prec), dtype=torch.uint8, device="cuda")
    G.gcn_aggregate(a, f_out, prec, S2, f_out, None, G.GCN_ACT_NONE, 0.0, False, 0, 0, 0, Y2, f_out, ov, wa)
    assert torch.equal(S, S2) and torch.equal(Y, Y2)


def _noalloc_against_workspace(prec, n, f_in, f_out):
    a, At, H, W, dZ = _operands(prec, n, f_in, f_out)
    L = _layer(f_in, f_out)
    ws = torch.empty(G.gcn_layer_workspace_size(a, L, prec), dtype=torch.uint8, device="cuda")
    res = []
    for call in ("workspace", "noalloc"):
        dW, db = (torch.full(s, 7.0, device="cuda") for s in ((f_in, f_out), (f_out,)))
        dZb, GS = torch.empty_like(H), torch.empty_like(dZ)
        ov = torch.zeros(1, dtype=torch.int32, device="cuda")
        if call == "workspace":
            G.gcn_layer_bwd(a, L, prec, H, W, dZ, G.GCN_ACT_RELU, 0.5, dW, db, dZb, GS, ov, ws)
        else:
            G.gcn_layer_bwd_noalloc(a, L, prec, H, W, dZ, G.GCN_ACT_RELU, 0.5, dW, db, dZb, GS, ov)
        res.append((dW, db, dZb, GS, ov))
    torch.cuda.synchronize()
    for x, y in zip(*res):
        assert torch.equal(x, y)


@pytest.mark.gpu
@pytest.mark.parametrize("prec,n,f_in,f_out", LAYERS)
def test_noalloc_takes_the_rows_in_several_launches(prec, n, f_in, f_out):
    """Less scratch than the partials of all rows: the same bits."""
    _noalloc_against_workspace(prec, n, f_in, f_out)


@pytest.mark.gpu
def test_noalloc_where_the_scratch_ends():
    """The column sums of dZ_below (512 floats per feature) leave less and less
    of the fixed scratch: room for the partials of some rows, of one row of
    tiles, of none (then neither call cuts the k range), and no room at all."""
    prec, n, f_out = 0, 30000, 160
    ranges = plan(prec, n, f_out)[3]
    assert ranges > 1
    everything, least = ranges * n * f_out * 4, ranges * 256 * f_out * 4
    limit = G.NOALLOC_SCRATCH_BYTES

    def without(f_in):
        return G.gcn_layer_workspace_size(_adj(n, prec, 4096), _layer(f_in, f_out), prec) - everything

    def last(bytes_left):
        lo, hi = 8, 1 << 17                          # widest f_in that leaves so much
        while hi - lo > 8:
            mid = (lo + hi) // 16 * 8
            lo, hi = (mid, hi) if without(mid) + bytes_left <= limit else (lo, mid)
        return lo

    some, one, none = last(everything // 2), last(least), last(0)
    assert some < one < none
    for f_in in (some, one, none):
        _noalloc_against_workspace(prec, n, f_in, f_out)
    with pytest.raises(G.GcnError) as e:
        _noalloc_against_workspace(prec, n, none + 8, f_out)
    assert e.value.status == 5                       # GCN_ERR_CAPACITY
