"""The residual-type stopping rules of the paper's sequential methods: the
monitored ||r||_2 / ||r_0||_2 is the sum of 1024 lanes (lane t adds nodes t,
t + 1024, ... in order, a butterfly per 64 lanes, their results in order),
bit for bit, whatever workgroup forms it; max|r| has no order."""
import numpy as np
import pytest

from gpu_helpers import need_gpu, rand_problem, say, to_dev

pytestmark = pytest.mark.gpu

DX, DY = 0.25, 0.5   # exact coefficients


def _residual(u, f):
    cx, cy = 1.0 / DX ** 2, 1.0 / DY ** 2
    lu = (cx * (u[1:-1, :-2] + u[1:-1, 2:]) + cy * (u[:-2, 1:-1] + u[2:, 1:-1])) - 2.0 * (cx + cy) * u[1:-1, 1:-1]
    return ((f[1:-1, 1:-1] if f is not None else 0.0) - lu).ravel()


def _sum_1024(r):
    sq = np.zeros(-(-r.size // 1024) * 1024)
    sq[:r.size] = r * r
    lanes = np.zeros(1024)
    for row in sq.reshape(-1, 1024):
        lanes = lanes + row
    waves = lanes.reshape(16, 64)
    for o in (32, 16, 8, 4, 2, 1):
        waves = waves + waves[:, np.arange(64) ^ o]
    total = waves[0, 0]
    for k in range(1, 16):
        total = total + waves[k, 0]
    return total


@pytest.mark.parametrize("m,n", [(3, 3), (10, 10), (11, 9), (25, 17), (34, 34), (35, 33), (97, 97), (9, 900)])
@pytest.mark.parametrize("method", ["jacobi", "sor_lex", "slor_lex", "adi_lex"])
def test_monitored_residual_bitwise(m, n, method):
    torch, lap = need_gpu()
    psi, f, _, _ = rand_problem(m, n, seed=m + n, dx=DX, dy=DY, source=m % 2 == 1)
    say("paper monitor", m, n, method)
    ctx = lap.Context(arena_bytes=64 << 20)
    for stop in ("rel_l2", "res_inf"):
        g = ctx.grid(to_dev(torch, psi), to_dev(torch, f) if f is not None else None, DX, DY, alloc=lap.LAP_ALLOC_ADI)
        info = g.solve(method, omega=1.0 if method == "jacobi" else 1.1, tol=0.0, stop=stop, max_iter=3)
        r = _residual(g.read().cpu().numpy(), f)
        want = (np.sqrt(_sum_1024(r)) / np.sqrt(_sum_1024(_residual(psi, f))) if stop == "rel_l2"
                else np.max(np.abs(r)))
        assert info["iterations"] == 3
        assert info["monitor"] == want, stop
        g.destroy()
    ctx.close()
