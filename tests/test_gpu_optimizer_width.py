"""The optimiser's four-wide kernels against its one-wide ones: the same
arithmetic per element, so the bits agree.  Arrays one element off a boundary
take the one-wide kernels at every length."""
import pytest
import torch

from paper_2010_12635_amd import gcn as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("count", [(1 << 18) - 1, 1 << 18, (1 << 18) + 1, (1 << 18) + 3, 3000001])
def test_widths_agree(prec, count):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(count)
    w0, g0, m0 = (torch.randn(count, generator=gen, device="cuda") for _ in range(3))
    v0 = torch.rand(count, generator=gen, device="cuda")
    cfg = G.GcnAdamConfig(0.01, 0.9, 0.999, 1e-8, 0.5, 2.0, 2000, 1.0, 2.0**24)
    outs = []
    for off in (0, 1):
        def buf(x, dt=torch.float32):
            b = torch.full((count + 8,), 7.0, dtype=dt, device="cuda")
            b[off:off + count] = x
            return b
        w, g, m, v = buf(w0), buf(g0 * 1024), buf(m0), buf(v0)
        wk = buf(0.0, G.torch_dtype(prec))
        st = torch.zeros(4, dtype=torch.int32, device="cuda")
        st.view(torch.float32)[0] = 1024.0
        flag = torch.zeros(1, dtype=torch.int32, device="cuda")
        args = [t[off:] for t in (w, g, m, v, wk)]
        G.gcn_optimizer_step(count, *args, prec, cfg, st, flag)
        G.gcn_optimizer_step(count, *args, prec, cfg, st, flag)
        before = [t.clone() for t in (w, m, v, wk)]
        g[off + count - 1] = float("nan")            # the last element: the step is skipped
        G.gcn_optimizer_step(count, *args, prec, cfg, st, flag)
        assert all(torch.equal(a, b) for a, b in zip(before, (w, m, v, wk)))
        assert st[2:].tolist() == [2, 1] and flag.item() == 0
        assert all(bool((t[off + count:] == 7.0).all()) and bool((t[:off] == 7.0).all()) for t in (w, m, v, wk))
        outs.append([t[off:off + count] for t in (w, m, v, wk)])
    assert not torch.equal(outs[0][0], w0)
    assert all(torch.equal(a, b) for a, b in zip(*outs))
