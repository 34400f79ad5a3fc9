"""Loading: inputs in time order (whose order is kept), out of order (sorted first), with self-loops
at the ends and in between, around the sizes where the grouping changes -- 1024 edges of a wavefront's
tile, 65,536 vertices (32- and 64-bit pair keys).  Counts, pair statistics and core numbers (which
read the neighbour lists) equal the oracle's."""
import numpy as np
import pytest

import oracle
from gpu_common import say

pytestmark = pytest.mark.gpu

import paper_2106_02762_amd as dt  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    c = dt.dt_ctx_create(0)
    yield c
    dt.dt_ctx_destroy(c)


def _edges(n, m, loops, order, seed):
    """m edges on a few hundred of the n ids (the first and last among them), `loops` self-loops."""
    rng = np.random.default_rng([seed, n, m, loops])
    ids = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, min(n, 3 + m // 8))]))
    src = rng.choice(ids, m)
    dst = rng.choice(ids, m)
    same = src == dst
    dst[same] = ids[(np.searchsorted(ids, src[same]) + 1) % ids.shape[0]]
    at = rng.choice(m, loops, replace=False)
    if loops >= 2:
        at[:2] = (0, m - 1)
    dst[at] = src[at]
    t = rng.integers(-50, 50 + m // 2, m)
    if order == "sorted":
        t.sort()
    elif order == "reversed":
        t = np.sort(t)[::-1].copy()
    elif order == "last":        # one edge out of place, at the very end
        t.sort()
        t[-1] = t[0] - 1
    return src.astype(np.uint32), dst.astype(np.uint32), t.astype(np.int64)


@pytest.mark.parametrize("order", ["sorted", "reversed", "mixed", "last"])
@pytest.mark.parametrize("n,m,loops", [
    (2, 1, 0), (3, 63, 5), (40, 1023, 0), (40, 1024, 2), (300, 1025, 30), (65536, 4096, 3), (65537, 4097, 0),
    (3_000_001, 20_000, 700)])
def test_load(ctx, n, m, loops, order):
    src, dst, t = _edges(n, m, loops, order, 7)
    say("load", n, m, loops, order)
    h = dt.dt_graph_load(ctx, n, src, dst, t)
    dt.dt_graph_build(h)
    ost, core = oracle.stats(n, src, dst, t, core=True)
    st = dt.dt_graph_stats(h)
    for ours, theirs in (("m_loaded", "m"), ("self_loops_dropped", "self_loops"), ("m_static", "m_static"),
                         ("max_multiplicity", "max_multiplicity"), ("n_static_triangles", "n_triangles"),
                         ("degeneracy", "degeneracy"), ("t_min", "t_min"), ("t_max", "t_max")):
        if ours == "m_loaded":
            assert st[ours] == m - int((src == dst).sum())
        elif ost["m_static"] or not ours.startswith("t_"):
            assert st[ours] == ost[theirs], ours
    assert np.array_equal(dt.dt_graph_order(h, n)[0], core)
    for d in ((7, 3, 5), (m, m // 3, m // 2), (dt.DT_INF,) * 3):
        assert np.array_equal(dt.dt_count(h, *d), oracle.count(n, src, dst, t, *d)), d
    dt.dt_graph_free(h)


def test_all_self_loops(ctx):
    ids = np.arange(100, dtype=np.uint32)
    h = dt.dt_graph_load(ctx, 100, ids, ids, np.arange(100, dtype=np.int64))
    dt.dt_graph_build(h)
    st = dt.dt_graph_stats(h)
    assert (st["m_loaded"], st["m_static"], st["self_loops_dropped"]) == (0, 0, 100)
    assert not dt.dt_count(h, 5, 5, 5).any()
    dt.dt_graph_free(h)
