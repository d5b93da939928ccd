"""Field upload and read-back: every value, for grids of few and of many rows
(the read splits rows over the launch when there are few)."""
import numpy as np
import pytest

from gpu_helpers import need_gpu, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(3, 3), (1023, 3), (1025, 5), (5000, 3), (100001, 3), (4099, 700), (1026, 1025),
                                 (2049, 2050), (7, 20000)])
def test_read_returns_what_was_written(m, n):
    torch, lap = need_gpu()
    say("field", m, n)
    a = np.random.default_rng(m + n).standard_normal((2, n, m))
    ctx = lap.Context(arena_bytes=lap.footprint(m, n, lap.LAP_ALLOC_ADI) + (8 << 20))
    g = ctx.grid(to_dev(torch, a[0]), None, 0.1, 0.1, alloc=lap.LAP_ALLOC_ADI)
    assert np.array_equal(g.read().cpu().numpy(), a[0])
    g.write(to_dev(torch, a[1]))
    assert np.array_equal(g.read().cpu().numpy(), a[1])
    g.destroy()
    ctx.close()
