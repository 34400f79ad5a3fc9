"""The level peel's finish where its (core, phase, degree class) cells come near the room for them: 8,160
to 8,192 vertices of a complete bipartite part (one high core number, no triangles), a path of many phases and
isolated vertices.  Core numbers equal the construction's, the ordering is a permutation, and no vertex
has more than core(v) neighbours after it."""
import numpy as np
import pytest

from test_gpu_peel import _G, _check, _static_pairs

pytestmark = pytest.mark.gpu

import paper_2106_02762_amd as dt  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    c = dt.dt_ctx_create(0)
    yield c
    dt.dt_ctx_destroy(c)


@pytest.mark.parametrize("n,side,path", [
    (8160, 1314, 400), (8161, 1314, 400), (8175, 1314, 400), (8191, 1314, 400), (8192, 1314, 400),
    (8161, 2621, 200), (8191, 2629, 200),
    (8160, 654, 200), (8161, 655, 200), (8191, 655, 200), (8191, 656, 200), (8191, 657, 200), (8192, 655, 200),
])
def test_cells_near_their_room(ctx, n, side, path):
    rng = np.random.default_rng([n, side])
    a, b = np.divmod(np.arange(side * side), side)
    p = 2 * side + np.arange(path - 1)
    u, v = np.concatenate([a, p]), np.concatenate([side + b, p + 1])
    core = np.zeros(n, np.uint32)
    core[:2 * side], core[2 * side:2 * side + path] = side, 1
    name = rng.permutation(n)
    of = np.empty(n, np.uint32)
    of[name] = core
    t = np.sort(rng.integers(0, 1000, u.shape[0])).astype(np.int64)
    g = _G(f"room(n={n}, {side}, {path})", n, name[u].astype(np.uint32), name[v].astype(np.uint32), t)
    got = _check(ctx, g, 0, 0, of, _static_pairs(g), (200, 100, 150, dt.INT64_MIN, dt.DT_INF))
    assert (got == 0).all()
