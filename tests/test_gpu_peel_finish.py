"""The level peel's finish (falling bounds, then every shell at once) at the sizes where it changes: one
block or many, vertex counts around a block's share and around what it takes over at most, rows of
exactly 64 packed entries, of whole and broken pieces, and longer than the registers hold.  Core numbers
equal the oracle's, and no vertex has more than core(v) neighbours after it."""
import numpy as np
import pytest

import oracle
from test_gpu_peel import _G, _check, _static_pairs

pytestmark = pytest.mark.gpu

import paper_2106_02762_amd as dt  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    c = dt.dt_ctx_create(0)
    yield c
    dt.dt_ctx_destroy(c)


def _graph(n, hubs, cliques, extra, seed):
    """n vertices: the first ones hubs of the given degrees, disjoint cliques of the given sizes among the
    others, and `extra` random pairs; one temporal edge per pair, vertex ids shuffled."""
    rng = np.random.default_rng([seed, n, extra])
    u, v = [], []
    for i, d in enumerate(hubs):
        u.append(np.full(d, i))
        v.append(len(hubs) + rng.choice(n - len(hubs), d, replace=False))
    at = len(hubs)
    for k in cliques:
        iu, ju = np.triu_indices(k, 1)
        u.append(iu + at)
        v.append(ju + at)
        at += k
    u.append(rng.integers(0, n, extra))
    v.append(rng.integers(0, n, extra))
    u, v = np.concatenate(u), np.concatenate(v)
    ok = u != v
    name = rng.permutation(n)
    t = np.sort(rng.integers(0, 1000, int(ok.sum())))
    return _G(f"finish(n={n})", n, name[u[ok]].astype(np.uint32), name[v[ok]].astype(np.uint32), t.astype(np.int64))


@pytest.mark.parametrize("n,hubs,cliques,extra,tails", [
    (1, [], [], 0, [0]),
    (2, [1], [], 0, [0, 1]),
    (1023, [64, 65, 700], [9, 33], 900, [0, 500]),
    (1024, [127, 128, 129], [64, 65, 66], 3000, [0]),
    (1025, [1000, 1023], [20], 2000, [0, 1024]),
    (4097, [255, 256, 257, 1023, 1024, 1025, 2047, 2048, 2049], [130, 140], 30000, [0, 3000]),
    (16321, [12000, 5000], [40] * 30, 60000, [0, 16320]),
    (65536, [60000, 1025], [70] * 20, 200000, [0]),
    (65537, [30000, 3000], [129, 257], 150000, [0]),
    (90000, [70000, 66000], [100, 101], 400000, [0, 16320]),
])
def test_finish(ctx, n, hubs, cliques, extra, tails):
    g = _graph(n, hubs, cliques, extra, 5)
    _, core = oracle.stats(g.n, g.src, g.dst, g.t, core=True)
    pairs = _static_pairs(g)
    query = (200, 100, 150, dt.INT64_MIN, dt.DT_INF)
    want = oracle.count(g.n, g.src, g.dst, g.t, *query)
    for tail in tails:
        assert (_check(ctx, g, 0, tail, core, pairs, query) == want).all(), tail
