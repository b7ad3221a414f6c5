"""The row-streaming products at the edges of their column blocks and row tiles:
few rows (narrowed column blocks), blocks cut for LDS, widths just past a
16-column tile, a 128-byte staging step and a block; S = H W, and dZ_below with
its column sums on a graph without edges (A_hat = I).  Against float64 of the
stored inputs with the rounding bound of an fp32 sum of K terms."""
import pytest
import torch

from paper_2010_12635_amd import gcn as G
from paper_2010_12635_amd.model import DeviceGraph, round8

pytestmark = pytest.mark.gpu

U = {0: 2.0 ** -24, 1: 2.0 ** -11, 2: 2.0 ** -8}


def rnd(shape, prec, gen, pad=True):
    n, f = shape
    t = torch.zeros((n, round8(f)), dtype=G.torch_dtype(prec), device="cuda")
    t[:, :f] = torch.randn(shape, generator=gen, device="cuda").to(t.dtype)
    t[:, f:] = 3.0                                   # padding is ignored
    return t


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("M", [1024, 1087, 20011])
@pytest.mark.parametrize("K,N", [(5, 8), (33, 17), (128, 33), (256, 65), (300, 130), (512, 16), (600, 200), (64, 257)])
def test_transform(prec, M, K, N):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + K + N)
    H, W = rnd((M, K), prec, gen), rnd((K, N), prec, gen)
    S = torch.full((M, round8(N) + 8), 7.0, dtype=H.dtype, device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(G.gcn_transform_workspace_size(M, K, N, prec), dtype=torch.uint8, device="cuda")
    G.gcn_transform(M, K, N, prec, H, H.shape[1], W, W.shape[1], S, S.shape[1], flag, ws)
    Hd, Wd = H[:, :K].double(), W[:, :N].double()
    want, mag = Hd @ Wd, Hd.abs() @ Wd.abs()
    assert bool(((S[:, :N].double() - want).abs() <= (K + 1) * 2.0 ** -24 * mag + U[prec] * want.abs() + 1e-30).all())
    assert bool((S[:, round8(N):] == 7.0).all()) and flag.item() == 0
    H[M - 1, K - 1] = float("inf")                   # the last row, nowhere else
    G.gcn_transform(M, K, N, prec, H, H.shape[1], W, W.shape[1], S, S.shape[1], flag, ws)
    assert flag.item() == 1 and bool(torch.isfinite(S[:M - 1, :N].float()).all())


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("n,f_in,f_out", [(1024, 17, 40), (3001, 128, 64), (20011, 200, 33), (2048, 72, 256)])
@pytest.mark.parametrize("relu", [True, False])
def test_input_gradient(prec, n, f_in, f_out, relu):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + f_in)
    dg = DeviceGraph(n, [], [], prec=prec)
    H, W, dZ = rnd((n, f_in), prec, gen), rnd((f_in, f_out), prec, gen), rnd((n, f_out), prec, gen)
    L = G.GcnLayer(f_in, f_out, H.shape[1], W.shape[1], G.GCN_ACT_NONE, 0.0, 1, 0)
    GS, dZb = torch.empty_like(dZ), torch.empty_like(H)
    dW = torch.empty((f_in, W.shape[1]), device="cuda")
    db, dbb = torch.empty(W.shape[1], device="cuda"), torch.empty(H.shape[1], device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(G.gcn_layer_workspace_size(dg.adj, L, prec), dtype=torch.uint8, device="cuda")
    p = 0.5 if relu else 0.0
    G.gcn_layer_bwd(dg.adj, L, prec, H, W, dZ, G.GCN_ACT_RELU if relu else G.GCN_ACT_NONE, p, dW, db, dZb, GS, flag,
                    ws, dbias_below=dbb)
    assert torch.equal(GS[:, :f_out], dZ[:, :f_out])                 # A_hat = I
    m = ((H[:, :f_in] > 0).double() / (1 - p)) if relu else 1.0
    Zd, Wd = dZ[:, :f_out].double(), W[:, :f_out].double()
    want, mag = (Zd @ Wd.T) * m, (Zd.abs() @ Wd.abs().T) * m
    got = dZb[:, :f_in].double()
    assert bool(((got - want).abs() <= (f_out + 2) * 2.0 ** -24 * mag + U[prec] * want.abs() + 1e-30).all())
    # the sums of what was stored, n fp32 terms in some order
    assert bool(((dbb[:f_in].double() - got.sum(0)).abs() <= n * 2.0 ** -24 * got.abs().sum(0)).all())
    assert bool((dbb[f_in:] == 0).all()) and flag.item() == 0


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("n,f_in,f_out", [(1024, 17, 40), (3001, 128, 64), (20011, 200, 33), (2048, 72, 256),
                                          (70003, 130, 16)])
@pytest.mark.parametrize("relu", [True, False])
def test_column_sums_of_whole_numbers(prec, n, f_in, f_out, relu):
    """Operands of -1, 0 and 1 make dZ_below whole numbers, times 2 under the
    mask, and its column sums whole numbers below 2^24: exact in every order, so
    that a row, step or tile left out of a sum shows (the rounding bound above is
    wider than one tile's part where workgroups take several)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + f_out)
    dt = G.torch_dtype(prec)

    def whole(rows, cols):
        t = torch.full((rows, round8(cols)), 3.0, dtype=dt, device="cuda")
        t[:, :cols] = torch.randint(-1, 2, (rows, cols), generator=gen, device="cuda").to(dt)
        return t

    dg = DeviceGraph(n, [], [], prec=prec)
    H, W, dZ = whole(n, f_in), whole(f_in, f_out), whole(n, f_out)
    L = G.GcnLayer(f_in, f_out, H.shape[1], W.shape[1], G.GCN_ACT_NONE, 0.0, 1, 0)
    GS, dZb = torch.empty_like(dZ), torch.empty_like(H)
    dW = torch.empty((f_in, W.shape[1]), device="cuda")
    db, dbb = torch.empty(W.shape[1], device="cuda"), torch.empty(H.shape[1], device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(G.gcn_layer_workspace_size(dg.adj, L, prec), dtype=torch.uint8, device="cuda")
    G.gcn_layer_bwd(dg.adj, L, prec, H, W, dZ, G.GCN_ACT_RELU if relu else G.GCN_ACT_NONE, 0.5 if relu else 0.0, dW, db,
                    dZb, GS, flag, ws, dbias_below=dbb)
    want = dZ[:, :f_out].double() @ W[:, :f_out].double().T
    if relu:
        want = want * 2 * (H[:, :f_in] > 0)
    assert float(want.abs().max()) <= (512 if relu else 256) and float(want.abs().sum(0).max()) < 2 ** 24
    assert torch.equal(dZb[:, :f_in].double(), want)
    assert torch.equal(dbb[:f_in].double(), want.sum(0))
    assert torch.equal(db[:f_out].double(), dZ[:, :f_out].double().sum(0))
    assert torch.equal(dW[:, :f_out].double(), H[:, :f_in].double().T @ dZ[:, :f_out].double())
    assert flag.item() == 0
