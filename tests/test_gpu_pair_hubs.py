"""gcn_pair_backward where a row's 64-entry blocks go to a whole workgroup: rows
of 32 to 35 blocks (the change from one lane group), several such rows next to
each other, one of hundreds of blocks, lane groups of 1 to 64 lanes, a padded
output; against the oracle, and twice with the same bits."""
import numpy as np
import pytest
import torch

from oracle import gcn_oracle as O
from paper_2010_12635_amd import gcn as G
from paper_2010_12635_amd.model import round8
from tests.parity import assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,F", [(0, 3), (0, 60), (0, 256), (1, 7), (1, 33), (1, 500), (2, 64), (2, 130)])
@pytest.mark.parametrize("rows", [(32 * 64, 33 * 64 - 1, 33 * 64 + 1, 34 * 64 + 65), (30000, 64, 5000, 2300)])
def test_hub_blocks(prec, F, rows):
    n = 700
    rng = np.random.default_rng(F + rows[0])
    # `rows` entries of the vertices 100, 101, ...; their partners and some
    # other pairs among the rest
    u = np.concatenate([np.full(k, 100 + i) for i, k in enumerate(rows)] + [rng.integers(0, 90, 999)])
    v = np.concatenate([rng.integers(200, n, u.size - 999), rng.integers(0, 90, 999)])
    swap = rng.random(u.size) < 0.5
    u, v = np.where(swap, v, u).astype(np.int32), np.where(swap, u, v).astype(np.int32)
    order = rng.permutation(u.size)
    u, v = u[order], v[order]
    z = (0.5 * rng.standard_normal((n, F))).astype(np.float32)
    gk = (rng.standard_normal(u.size) * 1e-2).astype(np.float32)
    dt, ld, ldz = G.torch_dtype(prec), round8(F), round8(F) + 8
    Z = torch.zeros((n, ld), dtype=dt, device="cuda")
    Z[:, :F] = torch.as_tensor(z).cuda().to(dt)
    dZ = torch.full((n, ldz), 7.0, dtype=dt, device="cuda")
    ov = torch.zeros(1, dtype=torch.int32, device="cuda")
    K = u.size
    ws = torch.empty(G.gcn_pair_backward_workspace_size(n, K, F), dtype=torch.uint8, device="cuda")
    du, dv, dg = (torch.as_tensor(a).cuda() for a in (u, v, gk))
    out = []
    for _ in range(2):
        G.gcn_pair_backward(n, F, ld, prec, Z, du, dv, K, dg, dZ, ldz, ov, ws)
        out.append(dZ[:, :F].clone())
    assert torch.equal(out[0], out[1]) and ov.item() == 0
    want = O.pair_backward(n, Z[:, :F].double().cpu().numpy(), u, v, gk.astype(np.float64))
    assert_close(out[0].double().cpu().numpy(), want, prec, "dZ")
