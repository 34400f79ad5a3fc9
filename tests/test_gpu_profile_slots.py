"""The profile of a count names each path that ran, for small counts as well, and profiling changes no
count."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import INF, Built, say

pytestmark = pytest.mark.gpu

import paper_2106_02762_amd as dt  # noqa: E402


def test_small_count_has_every_path():
    ctx = dt.dt_ctx_create(0)
    rng = np.random.default_rng(5)
    v = 3 * np.arange(3000)
    x, y = np.concatenate([v, v, v + 1]), np.concatenate([v + 1, v + 2, v + 2])
    k = np.where(np.arange(3000) % 3 == 0, 1, np.where(np.arange(3000) % 3 == 1, 2, 12))   # unit, light, medium
    k = np.concatenate([k, k, k])
    x, y = np.repeat(x, k), np.repeat(y, k)
    t = np.sort(rng.integers(0, 1000, x.shape[0]))
    g = synth.TemporalGraph(9000, x.astype(np.uint32), y.astype(np.uint32), t.astype(np.int64), name="slots")
    b = Built(ctx, g, g.name)
    st = dt.dt_graph_stats(b.h)
    assert st["n_unit_triangles"] and st["n_light_triangles"] and st["n_medium_triangles"]
    for d in ((300, 200, 150), (INF, INF, INF)):
        want = oracle.cpu_dottt(g.n, g.src, g.dst, g.t, *d)
        assert np.array_equal(b.count(*d), want)
        dt.dt_ctx_set_profiling(ctx, True)
        say("profiled")
        assert np.array_equal(b.count(*d), want)
        p = dt.dt_ctx_last_profile(ctx)
        # (the triangles that are neither take the medium path or the prefix procedures, by their deltas)
        assert p["light"] > 0 and p["unit"] > 0 and p["medium"] + p["heavy_count"] > 0 and p["reduce"] > 0, p
        dt.dt_ctx_set_profiling(ctx, False)
        assert np.array_equal(b.count(*d), want)
    b.free()
    dt.dt_ctx_destroy(ctx)
