"""FP64 grids on both sides of 2^21 interior nodes, from where on a grid solved
alone takes one pass per cycle over its finest level: in a batch or in ticks
it runs the merged plans, and ends where it ends alone, bit for bit."""
import numpy as np
import pytest

from gpu_helpers import need_gpu, rand_problem, say, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(1537, 1537), (129, 97), (2049, 1025), (1025, 1537)]   # 2.36e6, small, 2.10e6 (just above), 1.57e6


def _problems(torch):
    out = []
    for k, (m, n) in enumerate(SHAPES):
        psi, f, dx, dy = rand_problem(m, n, seed=90 + k, dx=1.0 / (m - 1), dy=1.1 / (m - 1), source=k % 2 == 0)
        out.append((to_dev(torch, psi), to_dev(torch, f) if f is not None else None, dx, dy))
    return out


def _alone(torch, lap, probs, **kw):
    ctx = lap.Context(arena_bytes=2 << 30)
    out = []
    for p, (m, n) in zip(probs, SHAPES):
        say("large alone", m, n)
        g = ctx.grid(*p, alloc=lap.LAP_ALLOC_FP64)
        info = g.solve("mg", **kw)
        out.append((info, g.read().cpu().numpy()))
        g.destroy()
    ctx.close()
    return out


def _same(info, u, ref):
    for key in ("iterations", "status", "rel_res_l2", "res_l2", "res_linf", "res0_l2"):
        assert info[key] == ref[0][key], key
    assert np.array_equal(u, ref[1])


@pytest.mark.parametrize("steps", [1, 3])
def test_fp64_ticks_match_alone(steps):
    torch, lap = need_gpu()
    probs = _problems(torch)
    alone = _alone(torch, lap, probs, tol=1e-9, max_iter=1000)
    ctx = lap.Context(arena_bytes=2 << 30)
    gs = [ctx.grid(*p, alloc=lap.LAP_ALLOC_FP64) for p in probs]
    for g in gs:
        g.set_tol(1e-9)
    say("large ticks", SHAPES, steps)
    left, infos = set(range(len(gs))), {}
    for _ in range(60):
        todo = sorted(left)
        done, ins = ctx.batch_step([gs[k] for k in todo], precision="fp64", steps=steps)
        for k, d, i in zip(todo, done, ins):
            if d:
                infos[k] = i
                left.discard(k)
        if not left:
            break
    assert not left
    for k, g in enumerate(gs):
        _same(infos[k], g.read().cpu().numpy(), alone[k])
    ctx.close()


@pytest.mark.parametrize("kw", [dict(tol=1e-9, max_iter=30), dict(tol=0.0, max_iter=3)])
def test_fp64_batch_matches_alone(kw):
    torch, lap = need_gpu()
    probs = _problems(torch)
    alone = _alone(torch, lap, probs, **kw)
    ctx = lap.Context(arena_bytes=2 << 30)
    gs = [ctx.grid(*p, alloc=lap.LAP_ALLOC_FP64) for p in probs]
    say("large batch", SHAPES, kw)
    infos = ctx.solve_batch(gs, method="mg", **kw)
    for g, info, ref in zip(gs, infos, alone):
        _same(info, g.read().cpu().numpy(), ref)
    ctx.close()


@pytest.mark.parametrize("tol", [0.5, 2e-3, 1e-9])
def test_solve_between_ticks_ends_them(tol):
    """A solve alone leaves its control block as it ended it, however its
    result came about (formed again behind the test, or before it): a tick
    that follows finds the grid done, with the solve's counts and field."""
    torch, lap = need_gpu()
    ctx = lap.Context(arena_bytes=1 << 30)
    g = ctx.grid(*_problems(torch)[0], alloc=lap.LAP_ALLOC_FP64)
    g.set_tol(1e-12)
    say("solve between ticks", SHAPES[0], tol)
    done, _ = ctx.batch_step([g], precision="fp64")
    assert done == [False]
    ref = g.solve("mg", tol=tol, max_iter=30)
    u = g.read().cpu().numpy()
    done, infos = ctx.batch_step([g], precision="fp64")
    assert done == [True]
    _same(infos[0], g.read().cpu().numpy(), (ref, u))
    ctx.close()


@pytest.mark.parametrize("kw", [dict(nu1=2, nu2=2), dict(nu1=1, nu2=1), dict(nu1=3, nu2=1), dict(nu1=0, nu2=2),
                                dict(fmg=True), dict(precision="mixed"), dict(precision="mixed", nu1=1, nu2=1),
                                dict(method="sor", omega=1.6, check_every=4, max_iter=8),
                                dict(method="adi", check_every=2, max_iter=4)])
def test_norms_of_large_grids(kw):
    """Every pass that forms the norms of a large grid, reduced by the count
    of its own tiling: the norms of the last test are those of the field it
    left, computed by the residual kernel (sums of other walks over the same
    2.4e6 squares: 1e-12 relative holds for any order); alone and in a batch."""
    torch, lap = need_gpu()
    kw = dict(dict(method="mg", tol=0.0, max_iter=2), **kw)
    probs = _problems(torch)[:2]
    ctx = lap.Context(arena_bytes=2 << 30)
    say("large norms", kw)
    for batch in (False, True):
        if batch and "fmg" in kw:
            continue
        gs = [ctx.grid(*p) for p in probs]
        infos = ctx.solve_batch(gs, **kw) if batch else [g.solve(**kw) for g in gs]
        for g, info in zip(gs, infos):
            l2, linf = g.residual()
            assert info["iterations"] == kw["max_iter"]
            assert abs(info["res_l2"] - l2) <= 1e-12 * l2
            assert info["res_linf"] == linf
            g.destroy()
    ctx.close()


def test_defect_correction_rings_bitwise():
    """The FP64 defect correction's row ring follows the launch's wavefronts:
    1120 alone (12 rows), 3360 in a batch of three (6 rows)."""
    torch, lap = need_gpu()
    m = n = 2049
    kw = dict(method="mg", precision="mixed", nu1=1, nu2=1, tol=0.0, max_iter=3)
    ctx = lap.Context(arena_bytes=2 << 30)
    gs, alone = [], []
    for k in range(3):
        psi, f, dx, dy = rand_problem(m, n, seed=60 + k, source=k != 1)
        p = to_dev(torch, psi)
        g = ctx.grid(p, to_dev(torch, f) if f is not None else None, dx, dy, alloc=lap.LAP_ALLOC_MIXED)
        say("defect ring alone", m, n, k)
        alone.append((g.solve(**kw), g.read().cpu().numpy()))
        g.write(p)
        gs.append(g)
    say("defect ring batch")
    infos = ctx.solve_batch(gs, **kw)
    for g, info, ref in zip(gs, infos, alone):
        _same(info, g.read().cpu().numpy(), ref)
    ctx.close()
