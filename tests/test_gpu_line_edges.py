"""Line solves and last tests at the edges of their kernels: workgroup sizes
of the segmented solver (blocks of a line: 64 | 128 | 256 along rows, 8 | 32 |
128 along columns), coupling that reaches over many blocks, merged launches
of grids on both sides of those lines, the paper's line methods on grids that
leave no room for their tables, and solves that end at max_iter."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import maxabs, need_gpu, rand_problem, say, to_dev
from oracle import lines as olines, solve as osolve

pytestmark = pytest.mark.gpu


# K unknowns a line, S = (K + 16) // 16 blocks: the last K of one workgroup size and the first of the next;
# rows K = 1023 | 1024, 2047 | 2048; columns K = 127 | 128, 511 | 512, 2047 | 2048
@pytest.mark.parametrize("m,n,direction", [(1025, 7, 0), (1026, 6, 0), (2049, 5, 0), (2050, 140, 0), (19, 129, 1),
                                           (70, 130, 1), (9, 513, 1), (130, 514, 1), (6, 2049, 1), (11, 2050, 1)])
@pytest.mark.parametrize("ratio", [1.0, 30.0, 1.0 / 30.0])
def test_line_half_at_workgroup_edges(m, n, direction, ratio):
    """One parity of one direction against the oracle.  The line matrix has
    condition (d + 2E) / (d - 2E), E the coupling along the line; both
    solvers are backward stable, so they differ by a few eps of that."""
    torch, lap = need_gpu()
    dx, dy = 0.1, 0.1 * ratio
    say("line edges", m, n, direction, ratio)
    psi, f, _, _ = rand_problem(m, n, m + 3 * n, dx=dx, dy=dy)
    u = lap.pitched(to_dev(torch, psi))
    lap.op_adi_half(m, n, dx, dy, 1.1, direction, 0, u, lap.pitched(to_dev(torch, f)))
    ref = psi.copy()
    fn = olines.adi_zebra_rows_half if direction == 0 else olines.adi_zebra_cols_half
    fn(ref, f, dx, dy, 1.1, "A")
    cx, cy = 1.0 / dx ** 2, 1.0 / dy ** 2
    e, d = (cx if direction == 0 else cy), 2.0 * (cx + cy)
    cond = (d + 2 * e) / (d - 2 * e)
    tol = max(1e-13, 8 * np.finfo(float).eps * cond)
    assert maxabs(u[:, :m].cpu().numpy(), ref) <= tol * max(1.0, np.max(np.abs(ref)))


def test_merged_line_launches_bitwise():
    """Merged launches give long and short lines other workgroups than a grid
    alone gets; norms of grids on both sides of the two-launch limits."""
    torch, lap = need_gpu()
    shapes = [(1026, 40), (2050, 33), (40, 514), (33, 2050), (130, 129), (17, 19)]
    ctx = lap.Context(arena_bytes=256 << 20)
    gs, alone = [], []
    for k, (m, n) in enumerate(shapes):
        psi, f, dx, dy = rand_problem(m, n, 50 + k, dx=0.1, dy=0.07, source=k % 2 == 0)
        g = ctx.grid(to_dev(torch, psi), to_dev(torch, f) if k % 2 == 0 else None, dx, dy, alloc=lap.LAP_ALLOC_ADI)
        say("merged lines alone", m, n)
        info = g.solve("adi", omega=1.0, tol=0.0, max_iter=4, check_every=2)
        alone.append((info["rel_res_l2"], g.read().cpu().numpy()))
        g.write(to_dev(torch, psi))
        gs.append(g)
    say("merged lines batch")
    infos = ctx.solve_batch(gs, method="adi", omega=1.0, tol=0.0, max_iter=4, check_every=2)
    for g, info, (rel, u) in zip(gs, infos, alone):
        assert np.array_equal(g.read().cpu().numpy(), u)
        assert info["rel_res_l2"] == rel
        g.destroy()
    ctx.close()


@pytest.mark.parametrize("method,form", [("slor_lex", "inside"), ("adi_lex", "after"), ("adi_lex", "inside")])
@pytest.mark.parametrize("m,n", [(97, 97), (100, 98), (57, 170)])
def test_paper_lines_near_the_lds_limit_bitwise(m, n, method, form):
    """Grids that fill LDS, with and without room for the line tables."""
    torch, lap = need_gpu()
    psi, f, dx, dy = rand_problem(m, n, m, dx=0.05, dy=0.06)
    say("paper lines", m, n, method, form)
    ctx = lap.Context(arena_bytes=64 << 20)
    g = ctx.grid(to_dev(torch, psi), to_dev(torch, f), dx, dy, alloc=lap.LAP_ALLOC_ADI)
    info = g.solve(method, omega=1.2, adi_form=form, stop="delta", tol=0.0, max_iter=2)
    names = {("slor_lex", "inside"): "slorb", ("adi_lex", "after"): "adi_lex_a", ("adi_lex", "inside"): "adi_lex_b"}
    ref, _, _ = osolve.iterate(names[(method, form)], psi, f, dx, dy, 1.2, "delta", 0.0, max_iter=2)
    assert info["iterations"] == 2
    assert np.array_equal(g.read().cpu().numpy(), ref)
    g.destroy()
    ctx.close()


@pytest.mark.parametrize("kw", [dict(method="sor", omega=1.6, check_every=5), dict(method="adi", check_every=2),
                                dict(method="mg", precision="mixed"), dict(method="mg"),
                                dict(method="mg", smoother="zebra", nu1=1, nu2=1)])
def test_solves_that_end_at_max_iter(kw):
    """The last test of a solve runs alone: a solve cut at max_iter and one
    with room for more blocks stand where the same blocks lead."""
    torch, lap = need_gpu()
    kw = dict(kw)
    method = kw.pop("method")
    ce = kw.get("check_every", 1)
    psi, f, dx, dy = rand_problem(257, 129, 9, dx=1 / 256, dy=1 / 256)
    ctx = lap.Context(arena_bytes=64 << 20)
    g = ctx.grid(to_dev(torch, psi), to_dev(torch, f), dx, dy)
    got = []
    for k in (2, 3):
        g.write(to_dev(torch, psi))
        say("max_iter", method, kw, k)
        info = g.solve(method, tol=0.0, max_iter=k * ce, **kw)
        assert info["iterations"] == k * ce
        got.append((info, g.read().cpu().numpy()))
    # a tolerance between the residuals after 2 and 3 blocks stops at 3, tested by a full step
    tol = np.sqrt(got[0][0]["rel_res_l2"] * got[1][0]["rel_res_l2"])
    assert got[1][0]["rel_res_l2"] < got[0][0]["rel_res_l2"]
    g.write(to_dev(torch, psi))
    info = g.solve(method, tol=tol, max_iter=20 * ce, **kw)
    assert info["iterations"] == 3 * ce
    assert info["rel_res_l2"] == got[1][0]["rel_res_l2"]
    assert np.array_equal(g.read().cpu().numpy(), got[1][1])
    g.destroy()
    ctx.close()
