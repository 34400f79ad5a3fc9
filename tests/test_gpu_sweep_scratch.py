"""A sweep whose triangles all take the prefix procedures: the queries share one set of launches when
their scratch may be had together, and run one after the other under a budget that holds only one
query's.  Both equal the sequential procedures on the CPU, with windows, for 1, 2, 8 and 11 triples."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import INF, say

pytestmark = pytest.mark.gpu

import paper_2106_02762_amd as dt  # noqa: E402

DELTAS = [(10, 10, 10), (500, 100, 450), (4000, 4000, 4000), (9000, 100, 9000), (0, 0, 0), (INF, INF, INF),
          (20000, 15000, 8000), (39999, 39999, 1), (7, 3, 5), (100, 60, 80), (2500, 2000, 1500)]


def _build(budget, g):
    ctx = dt.dt_ctx_create(0, budget)
    h = dt.dt_graph_load(ctx, g.n, g.src, g.dst, g.t)
    dt.dt_graph_build(h)
    dt.dt_graph_set_tuning(h, force_path=2, autotune=1)
    return ctx, h


@pytest.mark.parametrize("tight", [False, True])
def test_sweep_of_prefix_triangles(tight):
    g = synth.long_lists_graph(1, sizes=(40000, 25000, 700))
    budget = 0
    if tight:   # what the graph and one query's scratch take
        ctx, h = _build(0, g)
        dt.dt_count(h, 10, 10, 10)
        budget = dt.dt_ctx_memory(ctx)[0] + (2 << 20)
        dt.dt_graph_free(h)
        dt.dt_ctx_destroy(ctx)
    ctx, h = _build(budget, g)
    dt.dt_count(h, 10, 10, 10)
    for w in [(dt.INT64_MIN, INF), (3000, 31000)]:
        want = np.stack([oracle.cpu_dottt(g.n, g.src, g.dst, g.t, *d, *w) for d in DELTAS])
        for k in (1, 2, 8, 11):
            say("sweep", tight, k, w)
            assert np.array_equal(dt.dt_count_sweep(h, DELTAS[:k], *w), want[:k]), (k, w)
    dt.dt_graph_free(h)
    dt.dt_ctx_destroy(ctx)
