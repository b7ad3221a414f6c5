"""The pair loss where a lane group takes several pairs per iteration, each side
of the count from which it does.

A pair's inner product of F terms and its logistic loss are summed in fp32:
|score - exact| <= F 2^-23 sum |a b|, and the mean loss is within the largest
score error (the loss has slope at most 1) plus 2^-20 of itself for exp, log
and the sums."""
import numpy as np
import pytest
import torch

from paper_2010_12635_amd import gcn as G

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x)).cuda()


# 512 workgroups of 4 waves: from 131072 pairs up to 8 lanes per pair, 65536
# with 16, 32768 with 32, 16384 with 64; a pair each side of the line, ragged ends
@pytest.mark.parametrize("prec,F,K", [(1, 64, 131071), (1, 64, 131073), (1, 9, 131072), (2, 100, 65537), (0, 64, 70001),
                                      (0, 3, 131100), (0, 100, 32769), (0, 256, 16385), (1, 500, 16384 + 300)])
def test_pair_loss_rounds(prec, F, K):
    rng = np.random.default_rng(F + K)
    n, ld = 3001, (F + 7) // 8 * 8
    dt = G.torch_dtype(prec)
    Z = torch.full((n, ld), float("nan"), dtype=dt, device="cuda")      # padding columns are never used
    Z[:, :F] = dev((rng.standard_normal((n, F)) / np.sqrt(F) * 2).astype(np.float32)).to(dt)
    u, v = (rng.integers(0, n, K).astype(np.int32) for _ in range(2))
    u[5], v[K - 1], u[K // 2] = -1, n, 2**31 - 1                       # skipped, and raise the flag
    bad = np.zeros(K, bool)
    bad[[5, K - 1, K // 2]] = True
    n_pos = K // 3
    scores = torch.empty(K, dtype=torch.float32, device="cuda")
    g = torch.empty_like(scores)
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(G.gcn_pair_loss_workspace_size(K) // 4 + 64, dtype=torch.float32, device="cuda")
    st = torch.zeros(4, dtype=torch.int32, device="cuda")
    st.view(torch.float32)[0] = 1024.0
    G.gcn_pair_loss(n, F, ld, prec, Z, dev(u), dev(v), n_pos, K - n_pos, st, loss, scores, g, flag, ws)
    z = Z[:, :F].double().cpu().numpy()
    uc, vc = np.where(bad, 0, u), np.where(bad, 0, v)
    dot = np.einsum("kf,kf->k", z[uc], z[vc])
    bound = F * 2.0**-23 * np.einsum("kf,kf->k", np.abs(z[uc]), np.abs(z[vc]))
    got = scores.double().cpu().numpy()
    assert np.isnan(got[bad]).all() and (np.abs(got - dot)[~bad] <= bound[~bad]).all()
    y = (np.arange(K) < n_pos).astype(np.float64)
    want = np.where(bad, 0.0, 1 / (1 + np.exp(-dot)) - y) * 1024.0 / K
    # the sigmoid has slope at most 1/4; 8 roundings of exp, sum, quotient, difference and scale
    assert (np.abs(g.double().cpu().numpy() - want) <= (bound / 4 + 8 * 2.0**-24) * 1024.0 / K).all()
    ref = np.where(bad, 0.0, np.logaddexp(0, dot) - y * dot).sum() / K
    assert abs(loss.item() - ref) <= bound.max() + 2.0**-20 * ref
    assert flag.item() == 1
