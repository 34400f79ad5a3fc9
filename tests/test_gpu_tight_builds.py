"""Builds under the smallest budget that holds them: less than the first attempts of the enumeration (with
the unit keys beside it) and of the schedule (with room for every triangle in both classes) need, so that
the attempts that follow them are what succeeds; classes and counts are right there."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import say
from test_gpu_unit_split import QUERIES, _graph

pytestmark = pytest.mark.gpu

import paper_2106_02762_amd as dt  # noqa: E402


def _build(g, budget, check=None):
    """The statistics of a build, or None where the budget is too small; check(handle) while it is there."""
    say("build", g.name, "budget", budget)
    ctx = dt.dt_ctx_create(0, budget)
    h = None
    try:
        h = dt.dt_graph_load(ctx, g.n, g.src, g.dst, g.t)
        dt.dt_graph_set_tuning(h, autotune=1)
        dt.dt_graph_build(h)
        if check:
            check(h)
        return dt.dt_graph_stats(h)
    except dt.DtError as e:
        assert e.code == dt.DT_ENOMEM
        return None
    finally:
        if h is not None:
            dt.dt_graph_free(h)
        dt.dt_ctx_destroy(ctx)


def _smallest(g, lo, hi):
    assert _build(g, hi) and not _build(g, lo)
    while hi - lo > (2 << 20):
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if _build(g, mid) else (mid, hi)
    return hi


def _held(st):
    """Bytes of what stays of the load, the ordering and the orientation, and of the triangle list."""
    return 32 * st["m_static"] + 25 * st["m_loaded"] + 20 * st["n"], 12 * 4 * st["m_static"]


def test_schedule_of_counted_sizes():
    g, n_unit = _graph(1_000_000, 0.3)
    st = _build(g, 4 << 30)
    k = st["n_static_triangles"]
    assert (k, st["n_unit_triangles"]) == (1_000_000, n_unit)
    graph, tri_list = _held(st)
    # both classes' rooms beside the list and the keys, then the light list and its copy
    first = graph + tri_list + 8 * st["m_static"] + 18 * k + 12 * k + 24 * st["n_light_triangles"]
    budget = _smallest(g, 64 << 20, 4 << 30)
    say("smallest", budget, "first attempt", first)
    assert budget < first

    def check(h):
        assert dt.dt_graph_stats(h)["n_unit_triangles"] == n_unit
        for q in QUERIES:
            assert np.array_equal(dt.dt_count(h, *q), oracle.cpu_dottt(g.n, g.src, g.dst, g.t, *q)), q

    assert _build(g, budget + (8 << 20), check)   # (and room for the counts' scratch)


def test_enumeration_without_the_keys():
    """4M random pairs of 2M vertices and a clique of 70, whose runs are long enough for bitmaps."""
    rng = np.random.default_rng(8)
    n, m = 2_000_000, 4_000_000
    u, v = rng.integers(70, n, m), rng.integers(70, n, m)
    a, b = np.triu_indices(70, 1)
    src, dst = np.concatenate([u[u != v], a]), np.concatenate([v[u != v], b])
    t = np.sort(rng.integers(0, 10**6, src.shape[0]))
    g = synth.TemporalGraph(n, src.astype(np.uint32), dst.astype(np.uint32), t.astype(np.int64), name="keys")
    st = _build(g, 4 << 30)
    graph, tri_list = _held(st)
    first = graph + tri_list + 8 * st["m_static"] + 32 * n   # the keys, and the bitmaps' tables by vertex
    budget = _smallest(g, 64 << 20, 4 << 30)
    say("smallest", budget, "first attempt", first)
    assert budget < first
    want = oracle.cpu_dottt(g.n, g.src, g.dst, g.t, *QUERIES[0])

    def check(h):
        assert dt.dt_graph_stats(h)["n_unit_triangles"] == st["n_unit_triangles"]
        assert np.array_equal(dt.dt_count(h, *QUERIES[0]), want)

    assert _build(g, budget + (8 << 20), check)
