"""The ordering that the level peel's finish takes from the phases its bounds fall in: long paths (a phase
for every pair of vertices) beside cliques, so that (core, phase) pairs are far more than vertices, stars
and trees of paths, and one to many blocks.  Core numbers equal the oracle's, and no vertex has more than
core(v) neighbours after it."""
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


def _graph(paths, cliques, extra, seed=3):
    """Disjoint paths and cliques of the given sizes, each next one joined to the last by one pair, and
    `extra` random pairs; one temporal edge per pair, vertex ids shuffled."""
    rng = np.random.default_rng([seed, extra, len(paths)])
    u, v, at = [], [], 0
    for k in paths:
        u.append(np.arange(at, at + k - 1))
        v.append(np.arange(at + 1, at + k))
        at += k
    for k in cliques:
        iu, ju = np.triu_indices(k, 1)
        u.append(iu + at)
        v.append(ju + at)
        if at:
            u.append([at - 1])
            v.append([at])
        at += k
    u.append(rng.integers(0, at, extra))
    v.append(rng.integers(0, at, extra))
    u, v = np.concatenate(u).astype(np.int64), np.concatenate(v).astype(np.int64)
    ok = u != v
    name = rng.permutation(at)
    t = np.sort(rng.integers(0, 1000, int(ok.sum())))
    return _G(f"phases(n={at})", at, name[u[ok]].astype(np.uint32), name[v[ok]].astype(np.uint32), t.astype(np.int64))


@pytest.mark.parametrize("paths,cliques,extra,tails", [
    ([5], [], 0, [0]),
    ([600], [200], 0, [0]),                      # one block, more pairs than room
    ([1700], [300], 0, [0, 1500]),               # two blocks, more pairs than room
    ([900, 350, 351], [300, 20, 21, 22], 3, [0]),
    ([6000], [60] * 40, 0, [0]),
    ([40] * 900, [3, 4, 5, 6, 7, 8, 9, 100], 200, [0, 16000]),
    ([2] * 3000, [12] * 500, 9000, [0]),
])
def test_phases(ctx, paths, cliques, extra, tails):
    g = _graph(paths, cliques, extra)
    _, core = oracle.stats(g.n, g.src, g.dst, g.t, core=True)
    pairs = _static_pairs(g)
    query = (200, 100, 150, dt.INT64_MIN, dt.DT_INF)
    want = oracle.cpu_dottt(g.n, g.src, g.dst, g.t, *query)
    for tail in tails:
        assert (_check(ctx, g, 0, tail, core, pairs, query) == want).all(), tail
