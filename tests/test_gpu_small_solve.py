"""FP64 multigrid solves of grids whose hierarchy fits one workgroup's LDS run
as one launch: bitwise the launched solve (subtree off), norms and counts
included, over the edges of its range."""
import numpy as np
import pytest

from gpu_helpers import need_gpu, say, to_dev, rand_problem

pytestmark = pytest.mark.gpu

CASES = [
    # m, n, nu1, nu2, omega, source, stop, tol, max_iter
    (9, 9, 2, 2, 1.0, True, "rel_l2", 1e-10, 40),       # the smallest with two levels
    (25, 17, 2, 2, 1.0, False, "res_inf", 1e-6, 40),    # the chamber's size
    (9, 65, 1, 1, 1.15, True, "rel_l2", 1e-10, 60),
    (65, 9, 3, 1, 1.0, False, "rel_l2", 1e-10, 60),     # a single sweep opens: norms not flipped
    (65, 65, 2, 2, 1.0, True, "rel_l2", 1e-10, 40),     # 1024 patches: one a thread
    (65, 49, 0, 2, 1.0, True, "rel_l2", 1e-10, 60),     # norms from the residual kernel
    (81, 57, 2, 2, 1.0, False, "rel_l2", 1e-10, 40),    # two patches a thread, ragged
    (129, 65, 2, 2, 1.0, True, "rel_l2", 1e-10, 40),    # 2048 patches, two norm windows
    (65, 33, 2, 2, 1.0, True, "rel_l2", 0.0, 3),        # max_iter ends it
    (17, 17, 2, 2, 1.0, True, "rel_l2", 0.0, 1200),     # more cycles than one launch runs
    (33, 33, 2, 2, 1.0, True, "rel_l2", 2.0, 5),        # the first test ends it
]


@pytest.mark.parametrize("m,n,nu1,nu2,omega,source,stop,tol,max_iter", CASES)
def test_one_launch_solve_bitwise(m, n, nu1, nu2, omega, source, stop, tol, max_iter):
    torch, lap = need_gpu()
    psi, f, dx, dy = rand_problem(m, n, seed=m + 3 * n, dx=1.0 / (m - 1), dy=1.1 / (m - 1), source=source)
    say("small solve", m, n, nu1, nu2, omega, source, stop, tol, max_iter)
    got = []
    for sub in (0, -1):
        ctx = lap.Context(arena_bytes=64 << 20)
        ctx.set_subtree(sub)
        ctx.set_timing(1)
        g = ctx.grid(to_dev(torch, psi), to_dev(torch, f) if source else None, dx, dy)
        info = g.solve("mg", tol=tol, max_iter=max_iter, stop=stop, nu1=nu1, nu2=nu2, omega=omega)
        again = g.solve("mg", tol=tol, max_iter=2, stop=stop, nu1=nu1, nu2=nu2, omega=omega)   # continues
        swept = g.solve("sor", omega=1.2, tol=0.0, max_iter=3, check_every=3)                  # two-buffer method after it
        stats = ctx.kernel_stats(9)["launches"], ctx.kernel_stats(5)["launches"]
        got.append((info, again, swept, g.read().cpu().numpy(), stats))
        g.destroy()
        ctx.close()
    off, on = got
    assert on[4][0] >= 2 and on[4][1] < off[4][1]          # the one-launch path ran: no finalise launches of its own
    for a, b in zip(off[:3], on[:3]):
        for key in ("iterations", "status", "rel_res_l2", "res_l2", "res_linf", "res0_l2"):
            assert a[key] == b[key], key
    assert np.array_equal(off[3], on[3])
