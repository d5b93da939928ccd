"""Red-black SOR with four-sweep passes: counts, norms and field against one
launch per sweep, and alone against in a batch."""
import numpy as np
import pytest

from gpu_helpers import need_gpu, rand_problem, say, to_dev

pytestmark = pytest.mark.gpu

KC_FOUR = 14


@pytest.mark.parametrize("m,n,ce,source", [(33, 33, 6, True), (129, 40, 10, True), (300, 211, 7, False),
                                           (1026, 259, 50, True), (1600, 1400, 9, False)])
def test_four_sweep_norms(m, n, ce, source):
    """The test's norms are formed by the check block's first pass, fused or
    not: the same residuals, summed over walks in either direction (1e-12
    relative holds for any order of 2.2e6 squares), the same maximum."""
    torch, lap = need_gpu()
    psi, f, dx, dy = rand_problem(m, n, seed=m + n, dx=1.0 / (m - 1), dy=1.2 / (m - 1), source=source)
    kw = dict(omega=1.7, tol=0.0, max_iter=3 * ce, check_every=ce)
    say("sor norms", m, n, ce, source)
    out = []
    for fuse in (False, True):
        ctx = lap.Context(arena_bytes=512 << 20)
        ctx.set_fusion(fuse)
        gs = [ctx.grid(to_dev(torch, psi), to_dev(torch, f) if source else None, dx, dy, alloc=lap.LAP_ALLOC_ADI)
              for _ in range(3)]
        ctx.set_timing(1)
        alone = gs[0].solve("sor", **kw)
        assert (ctx.kernel_stats(KC_FOUR)["launches"] > 0) == fuse
        ctx.set_timing(0)
        u = gs[0].read().cpu().numpy()
        for g, info in zip(gs[1:], ctx.solve_batch(gs[1:], method="sor", **kw)):
            for key in ("iterations", "rel_res_l2", "res_l2", "res_linf", "res0_l2"):
                assert info[key] == alone[key], key
            assert np.array_equal(g.read().cpu().numpy(), u)
        out.append((alone, u))
        ctx.close()
    (a, ua), (b, ub) = out
    assert a["iterations"] == b["iterations"] == 3 * ce
    for key in ("rel_res_l2", "res_l2", "res0_l2"):
        assert abs(a[key] - b[key]) <= 1e-12 * abs(a[key]), key
    assert a["res_linf"] == b["res_linf"]
    assert np.array_equal(ua, ub)
