"""The sorts of gcn_pair_backward and gcn_pair_metrics at the sizes where a tile
doubles (2^27 endpoints, 2^25 scores) and on either side: whole-number inputs,
whose sums and counts are exact."""
import pytest
import torch

from paper_2010_12635_amd import gcn as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [(1 << 24) + 777, (1 << 26) - 1, (1 << 26) + 4099])
@pytest.mark.parametrize("n", [300, 1 << 19])
def test_pair_backward(n, K):
    F, ld = 4, 8
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K % 1009 + n)
    Z = torch.randint(0, 4, (n, ld), generator=gen, device="cuda").float()
    u, v = (torch.randint(0, n, (K,), generator=gen, device="cuda", dtype=torch.int32) for _ in range(2))
    g = torch.randint(-1, 2, (K,), generator=gen, device="cuda").float()
    dZ = torch.full((n, ld), 7.0, device="cuda")
    ov = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(G.gcn_pair_backward_workspace_size(n, K, F), dtype=torch.uint8, device="cuda")
    G.gcn_pair_backward(n, F, ld, G.GCN_F32, Z, u, v, K, g, dZ, ld, ov, ws)
    # at most 2 K / 300 entries of magnitude 3 in a row: partial sums below 2^24
    for c in range(F):
        want = torch.bincount(u, g.double() * Z[v.long(), c], n) + torch.bincount(v, g.double() * Z[u.long(), c], n)
        assert torch.equal(dZ[:, c].double(), want), c
    assert ov.item() == 0


@pytest.mark.parametrize("total", [(1 << 25) - 3, (1 << 25) + 5])
def test_pair_metrics(total):
    P, levels = total // 3, 1 << 18
    gen = torch.Generator(device="cuda")
    gen.manual_seed(total % 1009)
    lv = torch.randint(0, levels, (total,), generator=gen, device="cuda")
    lv[:P] = torch.maximum(lv[:P], torch.randint(0, levels, (P,), generator=gen, device="cuda"))
    scores = (lv - levels // 2).float()                  # both signs, many ties
    out = torch.zeros(2, dtype=torch.float64, device="cuda")
    ws = torch.empty(G.gcn_pair_metrics_workspace_size(P, total - P), dtype=torch.uint8, device="cuda")
    G.gcn_pair_metrics(scores, P, total - P, out, ws)
    pos, neg = torch.bincount(lv[:P], minlength=levels), torch.bincount(lv[P:], minlength=levels)
    auc2 = int((pos * (2 * (neg.cumsum(0) - neg) + neg)).sum())
    assert out[0].item() == auc2 / (2.0 * P * (total - P))
    ge = lambda x: x.flip(0).cumsum(0).flip(0).double()
    ap = float((pos.double() * ge(pos) / ge(pos + neg).clamp(min=1)).sum()) / P
    assert abs(out[1].item() - ap) <= 1e-11 * ap
