"""A new split of a built graph under budgets that hold the graph but not every split of it: where it fails
for want of memory, the graph's counts are refused or right, never counts of a schedule that is gone, and a
new build under the former tuning counts again."""
import numpy as np
import pytest

import oracle
from gpu_common import say
from test_gpu_unit_split import QUERIES, _graph

pytestmark = pytest.mark.gpu

import paper_2106_02762_amd as dt  # noqa: E402


def test_failed_split():
    g, n_unit = _graph(120_000, 1.0)   # unit triangles only: as prefix triangles they take far more memory
    want = [oracle.cpu_dottt(g.n, g.src, g.dst, g.t, *q) for q in QUERIES]
    failed = 0
    for mib in range(30, 110, 2):
        ctx = dt.dt_ctx_create(0, hbm_budget_bytes=mib << 20)
        h = None
        try:
            h = dt.dt_graph_load(ctx, g.n, g.src, g.dst, g.t)
            dt.dt_graph_set_tuning(h, autotune=1)
            dt.dt_graph_build(h)
            say("new split", mib, "MiB")
            try:
                dt.dt_graph_set_tuning(h, force_path=2, autotune=1)
            except dt.DtError as e:
                assert e.code == dt.DT_ENOMEM
                failed += 1
            for q, w in zip(QUERIES, want):
                try:
                    assert np.array_equal(dt.dt_count(h, *q), w), (mib, q)
                except dt.DtError as e:
                    assert e.code in (dt.DT_ENOTBUILT, dt.DT_ENOMEM), (mib, q, e)
            dt.dt_graph_set_tuning(h, autotune=1)
            dt.dt_graph_build(h)
            assert dt.dt_graph_stats(h)["n_unit_triangles"] == n_unit
            assert np.array_equal(dt.dt_count(h, *QUERIES[0]), want[0]), mib
        except dt.DtError as e:
            assert e.code == dt.DT_ENOMEM, (mib, e)
        finally:
            if h is not None:
                dt.dt_graph_free(h)
            dt.dt_ctx_destroy(ctx)
    assert failed
