"""Device buffers are kept after release and handed out again: a plan built on
the buffers of destroyed plans (of other media, sizes and precisions) gives
bit for bit what a plan on its own memory gave, and two live plans never share
a buffer."""
import time

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


def _free():
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def _comes_back(level, seconds=30):
    end = time.monotonic() + seconds
    while _free() < level and time.monotonic() < end:
        time.sleep(0.5)
    return _free() >= level


def test_memory_of_a_destroyed_plan_comes_back(lib):
    """After a plan is destroyed its device memory is free again for the rest
    of the process: without any further call, and at once on request."""
    from paper_1804_02297_amd.binding import release_memory
    n, prec = 24, "c128"
    _solve(n, 1, prec)[0].close()               # code objects, scratch memory
    release_memory()
    before = _free()
    for ask in (False, True):
        plan, z, y = _solve(n, 2, prec)
        del z, y
        used = before - _free()
        print(f"plan holds {used / 2**20:.0f} MiB", flush=True)
        assert used >= 400 << 20
        plan.close()
        if ask:
            release_memory()
        assert _comes_back(before - used // 16, 1 if ask else 30)


@pytest.mark.parametrize("ask", [False, True])
def test_memory_comes_back_during_capture(lib, ask):
    """Blocks that go back while this thread captures a graph, by themselves or
    on request: they do, and the graph replays as the eager call."""
    from paper_1804_02297_amd.binding import release_memory
    n = 16
    plan, _, _ = _solve(n, 1, "c128")
    x = torch.from_numpy(I.random_field(2, n, 7)).to("cuda:0")
    y, want = torch.empty_like(x), plan.apply(x)
    _solve(24, 2, "c128")[0].close()
    release_memory()
    before = _free()
    _solve(24, 2, "c128")[0].close()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.apply(x, y)
        release_memory() if ask else time.sleep(8)
    assert _comes_back(before - (64 << 20))
    for seed in (7, 8, 9):
        x.copy_(torch.from_numpy(I.random_field(2, n, seed)))
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, plan.apply(x)), seed
    x.copy_(torch.from_numpy(I.random_field(2, n, 7)))
    g.replay()
    torch.cuda.synchronize()
    assert torch.equal(y, want)
    plan.close()
