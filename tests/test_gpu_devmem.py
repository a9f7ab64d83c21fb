"""Device buffers are kept after release and handed out again: a plan built on
the buffers of destroyed plans (of other media, sizes and precisions) gives
bit for bit what a plan on its own memory gave, and two live plans never share
a buffer."""
import numpy as np
import pytest

from paper_1804_02297_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _solve(n, seed, prec, nrhs=2):
    from paper_1804_02297_amd.binding import Plan
    k = I.wavenumber_for(n)
    plan = Plan(n, k, torch.from_numpy(I.medium_bumps(n, seed)).to("cuda:0"), max_rhs=nrhs)
    plan.stencil_fit(0)
    plan.factor_gpu(prec)
    v = torch.from_numpy(I.random_field(nrhs, n, 5)).to("cuda:0")
    return plan, plan.precond(v), plan.apply(v)


@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_reused_buffers_leave_no_trace(lib, prec):
    plan, z0, y0 = _solve(16, 1, prec)
    keep = [t.cpu().numpy() for t in (z0, y0)]
    plan.close()
    for n, seed, pr in ((15, 2, "c128"), (16, 3, "c64"), (14, 4, "c128"), (16, 5, "c128")):
        print(f"n={n} {pr}", flush=True)
        _solve(n, seed, pr)[0].close()
    a, za, ya = _solve(16, 1, prec)
    b, zb, yb = _solve(16, 6, prec)           # while a lives
    for t, ref in zip((za, ya, a.precond(torch.from_numpy(I.random_field(2, 16, 5)).to("cuda:0"))),
                      (keep[0], keep[1], keep[0])):
        assert np.array_equal(t.cpu().numpy(), ref)
    assert not np.array_equal(zb.cpu().numpy(), keep[0])
    a.close()
    b.close()
