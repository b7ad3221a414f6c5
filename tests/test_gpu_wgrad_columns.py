"""dW = H^T G_S at the edges of the column counts that have kernels of their own
(16, 32, 48, 64, wider), with few and with ragged rows, on a graph without edges
(A_hat = I, so G_S = dZ).  Against float64 of the stored inputs with the
rounding bound of an fp32 sum of n terms."""
import pytest
import torch

from paper_2010_12635_amd import gcn as G
from paper_2010_12635_amd.model import DeviceGraph, round8

pytestmark = pytest.mark.gpu


def rnd(shape, prec, gen):
    n, f = shape
    t = torch.zeros((n, round8(f)), dtype=G.torch_dtype(prec), device="cuda")
    t[:, :f] = torch.randn(shape, generator=gen, device="cuda").to(t.dtype)
    t[:, f:] = float("nan")                          # padding is masked out of the products
    return t


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("n,f_in", [(1031, 17), (5003, 130)])
@pytest.mark.parametrize("f_out", [1, 16, 17, 32, 33, 48, 49, 64, 65])
def test_weight_gradient(prec, n, f_in, f_out):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + f_out)
    dg = DeviceGraph(n, [], [], prec=prec)
    H, dZ = rnd((n, f_in), prec, gen), rnd((n, f_out), prec, gen)
    dZ[:, f_out:] = 0
    W = torch.zeros((f_in, round8(f_out)), dtype=H.dtype, device="cuda")
    L = G.GcnLayer(f_in, f_out, H.shape[1], W.shape[1], G.GCN_ACT_NONE, 0.0, 1, 0)
    GS = torch.full_like(dZ, float("nan"))
    dW = torch.full((f_in, W.shape[1]), 7.0, device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(G.gcn_layer_workspace_size(dg.adj, L, prec), dtype=torch.uint8, device="cuda")
    G.gcn_layer_bwd(dg.adj, L, prec, H, W, dZ, G.GCN_ACT_NONE, 0.0, dW, None, None, GS, flag, ws)
    Hd, Zd = H[:, :f_in].double(), dZ[:, :f_out].double()
    want, mag = Hd.T @ Zd, Hd.abs().T @ Zd.abs()
    assert bool(((dW[:, :f_out].double() - want).abs() <= (n + 1) * 2.0 ** -24 * mag).all())
    assert bool((dW[:, f_out:] == 0).all()) and flag.item() == 0
