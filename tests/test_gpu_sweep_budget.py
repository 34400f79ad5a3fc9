"""The memory that a sweep takes for several queries' prefix arrays at once goes back: under a budget, a
graph that loads, builds and counts beside another one does so as well after sweeps of that one."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import say

pytestmark = pytest.mark.gpu

import paper_2106_02762_amd as dt  # noqa: E402

DELTAS = [(500, 400, 300 + 20 * j) for j in range(8)]
SCRATCH = (40000 + 25000 + 4) * 8 * 8   # of one query: eight 64-bit arrays over the source edges, at least


def _second(m, n=50_000):
    """m random edges on n vertices: a build of about 120 bytes an edge."""
    rng = np.random.default_rng(4)
    src, dst = rng.integers(0, n, m), rng.integers(0, n, m)
    dst[src == dst] = (src[src == dst] + 1) % n
    return synth.TemporalGraph(n, src.astype(np.uint32), dst.astype(np.uint32),
                               np.sort(rng.integers(0, 10**6, m)).astype(np.int64), name="second")


def _run(budget, first, second, sweeps):
    """Whether the second graph fits beside the first, after its count and `sweeps` sweeps."""
    say("budget", budget, "sweeps", sweeps)
    ctx = dt.dt_ctx_create(0, budget)
    graphs = []
    try:
        for g in (first, second):
            h = dt.dt_graph_load(ctx, g.n, g.src, g.dst, g.t)
            graphs.append(h)
            if g is first:
                dt.dt_graph_set_tuning(h, force_path=2, autotune=1)
            dt.dt_graph_build(h)
            if g is first:
                want = [oracle.cpu_dottt(g.n, g.src, g.dst, g.t, *d) for d in DELTAS]
                assert np.array_equal(dt.dt_count(h, *DELTAS[0]), want[0])
                for _ in range(sweeps):
                    assert np.array_equal(dt.dt_count_sweep(h, DELTAS), np.stack(want))
        return True
    except dt.DtError as e:
        assert e.code == dt.DT_ENOMEM
        return False
    finally:
        for h in graphs:
            dt.dt_graph_free(h)
        dt.dt_ctx_destroy(ctx)


def test_a_sweep_gives_its_memory_back():
    first = synth.long_lists_graph(1, sizes=(40000, 25000, 700))
    second = _second(1_100_000)
    lo, hi = 16 << 20, 1 << 30   # budgets: too small, enough
    assert _run(hi, first, second, 0) and not _run(lo, first, second, 0)
    while hi - lo > (2 << 20):
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if _run(mid, first, second, 0) else (mid, hi)
    # The second graph needs twice what a sweep of eight takes, so that the sweep finds room for all of them,
    # and the eighth that a cached block may waste is less than they take: kept, they would be missing.
    budget = hi + hi // 8 + (4 << 20)
    assert hi > 2 * 8 * SCRATCH and budget - hi < 7 * SCRATCH
    assert _run(budget, first, second, 0)
    assert _run(budget, first, second, 2)
