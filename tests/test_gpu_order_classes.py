"""The ordering within one shell and phase of the level peel's finish: by degree over the core number, so
that a hub comes after the other vertices of its shell.  Gadgets of a clique whose vertices have one leaf
each and a hub joined to them and to many leaves: all settle in one phase with one core number."""
import numpy as np
import pytest

import oracle
from test_gpu_peel import _G, _check, _static_pairs

pytestmark = pytest.mark.gpu

import paper_2106_02762_amd as dt  # noqa: E402


@pytest.mark.parametrize("copies", [3, 60])   # one block, many
def test_hubs_come_last(copies):
    k, leaves = 10, 500
    size = k + 1 + k + leaves   # clique, hub, a leaf of each clique vertex, the hub's leaves
    a, b = np.triu_indices(k + 1, 1)
    u = np.concatenate([a, np.arange(k), np.full(leaves, k)])
    v = np.concatenate([b, k + 1 + np.arange(k), 2 * k + 1 + np.arange(leaves)])
    at = size * np.repeat(np.arange(copies), u.shape[0])
    u, v = np.tile(u, copies) + at, np.tile(v, copies) + at
    n = size * copies
    rng = np.random.default_rng(copies)
    name = rng.permutation(n).astype(np.uint32)
    t = np.sort(rng.integers(0, 1000, u.shape[0])).astype(np.int64)
    g = _G(f"hubs({copies})", n, name[u], name[v], t)
    ctx = dt.dt_ctx_create(0)
    _, core = oracle.stats(g.n, g.src, g.dst, g.t, core=True)
    query = (200, 100, 150, dt.INT64_MIN, dt.DT_INF)
    want = oracle.cpu_dottt(g.n, g.src, g.dst, g.t, *query)
    assert (_check(ctx, g, 0, 0, core, _static_pairs(g), query) == want).all()
    h = dt.dt_graph_load(ctx, g.n, g.src, g.dst, g.t)
    dt.dt_graph_build(h)
    _, rank = dt.dt_graph_order(h, g.n)
    dt.dt_graph_free(h)
    dt.dt_ctx_destroy(ctx)
    for c in range(copies):
        clique, hub = name[size * c + np.arange(k)], name[size * c + k]
        assert core[hub] == k and (core[clique] == k).all()
        assert (rank[clique] < rank[hub]).all(), c
