"""The split of the triangle list into unit records and the rest: lists around the tile of 2,048
entries, with no, some and only unit triangles (the rest beyond its first room of 65,536 as well), a
schedule made again for the built graph, and builds under budgets that leave less and less memory;
counts against the oracle, classes against the graph's construction."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import INF, Built, say

pytestmark = pytest.mark.gpu

import paper_2106_02762_amd as dt  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    c = dt.dt_ctx_create(0)
    yield c
    dt.dt_ctx_destroy(c)


def _graph(k, share, seed=5):
    """k disjoint triangles; a share of them has one edge on each pair, the others two on one pair."""
    rng = np.random.default_rng([seed, k])
    unit = np.arange(k) < round(share * k)
    rng.shuffle(unit)
    v = 3 * np.arange(k)
    x = np.concatenate([v, v, v + 1, (v + 1)[~unit]])
    y = np.concatenate([v + 1, v + 2, v + 2, (v + 2)[~unit]])
    flip = rng.random(x.shape[0]) < 0.5
    src, dst = np.where(flip, y, x), np.where(flip, x, y)
    p = rng.permutation(x.shape[0])
    t = rng.integers(0, 1000, x.shape[0])
    return synth.TemporalGraph(3 * k, src[p].astype(np.uint32), dst[p].astype(np.uint32), t.astype(np.int64),
                               name=f"units{k}x{share}"), int(unit.sum())


QUERIES = [(INF, INF, INF), (300, 200, 150), (500, 500, 500, 250, 700)]


@pytest.mark.parametrize("share", [0.0, 0.6, 1.0])
@pytest.mark.parametrize("k", [1, 63, 65, 256, 2047, 2048, 2049, 70_000])
def test_split_sizes(ctx, k, share):
    g, n_unit = _graph(k, share)
    b = Built(ctx, g, g.name)
    for again in (False, True):
        if again:
            dt.dt_graph_set_tuning(b.h, light_pair_cap=4)
        st = dt.dt_graph_stats(b.h)
        assert (st["n_static_triangles"], st["n_unit_triangles"]) == (k, n_unit)
        for q in QUERIES:
            assert np.array_equal(b.count(*q), oracle.cpu_dottt(g.n, g.src, g.dst, g.t, *q)), q
    b.free()


def test_split_under_budgets():
    g, n_unit = _graph(120_000, 0.4)
    want = [oracle.cpu_dottt(g.n, g.src, g.dst, g.t, *q) for q in QUERIES]
    ok = 0
    for mib in (512, 128, 104, 88, 76, 68, 60, 54, 48, 42, 36):
        say("budget", mib, "MiB")
        c = dt.dt_ctx_create(0, hbm_budget_bytes=mib << 20)
        h = None
        try:
            h = dt.dt_graph_load(c, g.n, g.src, g.dst, g.t)
            dt.dt_graph_build(h)
            assert dt.dt_graph_stats(h)["n_unit_triangles"] == n_unit
            for q, w in zip(QUERIES, want):
                assert np.array_equal(dt.dt_count(h, *q), w), (mib, q)
            ok += 1
        except dt.DtError as e:
            assert e.code == dt.DT_ENOMEM
        finally:
            if h is not None:
                dt.dt_graph_free(h)
            dt.dt_ctx_destroy(c)
    assert ok
