"""Mixed solves whose residual overflows FP32: the solve diverges, and the
Dirichlet data come back as they went in."""
import numpy as np
import pytest

from gpu_helpers import need_gpu, rand_problem, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(129, 129), (33, 33), (1025, 257)])
@pytest.mark.parametrize("kw", [dict(), dict(inner=4), dict(nu1=1, nu2=1), dict(smoother="zebra", nu1=1, nu2=1)])
def test_perimeter_survives_an_overflow(m, n, kw):
    torch, lap = need_gpu()
    psi, f, dx, dy = rand_problem(m, n, seed=m + n)
    f[1:-1, 1] = f[1:-1, -2] = 1e42   # finite in FP64 (and its square), infinite in FP32, beside the walls
    f[1, 1:-1] = f[-2, 1:-1] = -1e42
    say("overflow", m, n, kw)
    ctx = lap.Context(arena_bytes=256 << 20)
    gs = [ctx.grid(to_dev(torch, psi), to_dev(torch, f), dx, dy) for _ in range(2)]
    info = gs[0].solve("mg", precision="mixed", max_iter=5, **kw)
    infos = [info] + ctx.solve_batch(gs[1:], method="mg", precision="mixed", max_iter=5, **kw)
    for g, info in zip(gs, infos):
        assert info["status"] == -4 and info["iterations"] >= 1   # diverged, after a step
        u = g.read().cpu().numpy()
        for edge in (np.s_[0, :], np.s_[-1, :], np.s_[:, 0], np.s_[:, -1]):
            assert np.array_equal(u[edge], psi[edge])
        g.write(to_dev(torch, psi))                               # and the grid is as good as new
        assert not np.isnan(g.solve("mg", precision="fp64", tol=0.0, max_iter=2)["res_l2"])
    ctx.close()
