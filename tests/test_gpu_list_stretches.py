"""The triangle list's positions, reserved in stretches of the room at hand: lists that fit with few and
with many triangles a wavefront, that just pass the first room of 65,536 entries, and that pass it by far
(the pass runs again).  The static triangles are the oracle's, each once, and so are the counts."""
import numpy as np
import pytest

import oracle
from gpu_common import Built
from test_gpu_enumerate import _cliques

pytestmark = pytest.mark.gpu

import paper_2106_02762_amd as dt  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    c = dt.dt_ctx_create(0)
    yield c
    dt.dt_ctx_destroy(c)


@pytest.mark.parametrize("size,copies,noise_n", [
    (58, 2, 0),         # 61,712 triangles on 3,306 pairs: nearly the whole room
    (59, 2, 100),       # 65,018: with what the stretches leave empty, about all of it
    (74, 1, 0), (75, 1, 0),   # 64,824 and 67,525: either side of it
    (90, 3, 5000),      # three and a half times the triangles that fit
    (200, 1, 0),        # 1.3M triangles on 19,900 pairs
    (40, 300, 100000),  # 3M triangles on 384,000 pairs: twice what fits, in packs of short runs
])
def test_lists(ctx, size, copies, noise_n):
    g = _cliques(size, copies, noise_n, 4)
    b = Built(ctx, g, g.name)
    want = oracle.triangles(g.n, g.src, g.dst, g.t)
    assert dt.dt_graph_stats(b.h)["n_static_triangles"] == want.shape[0]
    got = dt.dt_graph_triangles(b.h)
    got = got[np.lexsort((got[:, 2], got[:, 1], got[:, 0]))]
    assert np.array_equal(got, want)
    d = (20000, 9000, 15000)
    ref = oracle.count(g.n, g.src, g.dst, g.t, *d)
    assert np.array_equal(b.count(*d), ref)
    dt.dt_graph_set_tuning(b.h, light_pair_cap=4)   # (enumerated and scheduled again)
    assert np.array_equal(b.count(*d), ref)
    b.free()
