"""gcn_normalize's sort-based construction at the sizes where it can go
wrong, bit for bit against the oracle: edges of a sort tile (4096 keys) and of
a compaction tile (2048), one and two vertices, both sides of the change from
32-bit to 64-bit keys (n = 65536), digit widths from 2 to 9 bits, a list that
is one hub, a list that is one edge over and over, more than 2^32 keys."""
import numpy as np
import pytest
import torch

from oracle import gcn_oracle as O
from paper_2010_12635_amd import gcn as G
from paper_2010_12635_amd.model import DeviceGraph
from tests.parity import hub_graph

pytestmark = pytest.mark.gpu


def check(n, src, dst, index=G.GCN_I32):
    g = O.graph(n, src, dst)
    dg = DeviceGraph(n, src, dst, prec=G.GCN_F32, index=index, schedule=False)
    rp, ci = dg.csr_host()
    assert dg.nnz == g.nnz
    assert np.array_equal(rp, g.rowptr) and np.array_equal(ci, g.colidx)
    assert np.array_equal(dg.deg.cpu().numpy(), g.deg)
    assert np.array_equal(dg.dinv.cpu().numpy(), O.dinv_f32(g))
    # one fp32 product of two fp32 factors: within one rounding of the oracle's
    # product of the same factors
    vals = dg.values[: dg.nnz].cpu().numpy()
    d = O.dinv_f32(g)
    rows = np.repeat(np.arange(n), np.diff(g.rowptr))
    assert np.array_equal(vals, d[rows] * d[g.colidx])


# 2 E + n on either side of a tile edge: 2048, 4096 and two tiles of 4096
@pytest.mark.parametrize("keys", [2047, 2048, 2049, 4095, 4096, 4097, 8191, 8193, 12289])
def test_tile_edges(keys):
    n = 301 if keys % 2 else 300
    e = (keys - n) // 2
    rng = np.random.default_rng(keys)
    check(n, rng.integers(0, n, e).astype(np.int32), rng.integers(0, n, e).astype(np.int32))


# 1: 2-bit keys; 65536: the last with 32-bit keys; 65537: 34-bit keys; 300000: 38 bits, five passes
@pytest.mark.parametrize("n", [1, 2, 3, 513, 65535, 65536, 65537, 300000])
@pytest.mark.parametrize("index", [G.GCN_I32, G.GCN_I64])
def test_key_widths(n, index):
    src, dst = hub_graph(n, 4 * n, [(n - 1, 9000)], seed=n)
    check(n, src % n, dst % n, index)


@pytest.mark.parametrize("n", [5000, 70000])
def test_skewed(n):
    # every edge at one hub; then one edge repeated (in one digit's run of every tile)
    rng = np.random.default_rng(n)
    check(n, np.full(40000, n // 2, np.int32), rng.integers(0, n, 40000).astype(np.int32))
    check(n, np.full(40000, 3, np.int32), np.full(40000, n - 1, np.int32))


# 34.2 M keys: the first size with 16 items per thread; 2^32 + 2^26 keys
@pytest.mark.parametrize("n", [1 << 19, 1 << 26])
def test_many_keys(n):
    # vertex i linked to i + 1 .. i + 32 (mod n): every row has 65 entries
    k = 32
    src = torch.empty(n * k, dtype=torch.int32, device="cuda")
    dst = torch.empty(n * k, dtype=torch.int32, device="cuda")
    base = torch.arange(n, dtype=torch.int32, device="cuda")
    for j in range(k):
        src[j * n:(j + 1) * n] = base
        dst[j * n:(j + 1) * n] = (base + (j + 1)) % n
    dg = DeviceGraph(n, src, dst, prec=G.GCN_F16, index=G.GCN_I64, schedule=False)
    del src, dst
    assert dg.nnz == 65 * n
    assert torch.equal(dg.rowptr, torch.arange(n + 1, device="cuda") * 65)
    assert bool((dg.deg == 65).all())
    cols = dg.colidx[: dg.nnz].view(n, 65)
    step = min(n, 1 << 22)
    for lo in range(0, n, step):
        rows = torch.arange(lo, lo + step, device="cuda")[:, None]
        want = (rows + torch.arange(-k, k + 1, device="cuda")[None, :]) % n
        if lo == 0 or lo + step == n:        # the rows that wrap around
            want = want.sort(1).values
        assert torch.equal(cols[lo:lo + step].long(), want)
    want = torch.tensor(1.0 / 65, device="cuda").half()
    assert bool(((dg.values[: dg.nnz] - want).abs() <= want * 2.0 ** -10).all())
