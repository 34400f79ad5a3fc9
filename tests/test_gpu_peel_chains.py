"""Graphs whose core bounds fall one vertex a phase -- paths, thick chains, lattices, alone, beside a
power-law part and behind leaves that the levels take first -- which the level peel's finish leaves to the
levels, on the grid and in one workgroup; and rows that a block's wavefronts walk together.  Core numbers
equal the oracle's, no vertex has more than core(v) neighbours after it, and a chain's phases end."""
import numpy as np
import pytest

import oracle
from gpu_common import say
from test_gpu_peel import _G, _check, _static_pairs

pytestmark = pytest.mark.gpu

import paper_2106_02762_amd as dt  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    c = dt.dt_ctx_create(0)
    yield c
    dt.dt_ctx_destroy(c)


def _chain(k, p=1, at=0):
    """k vertices in a row, each joined to the next p."""
    i = at + np.arange(k)
    return np.concatenate([i[:k - s] for s in range(1, p + 1)]), np.concatenate([i[s:] for s in range(1, p + 1)])


def _lattice(w):
    """w x w vertices, joined to the right, below and diagonally."""
    i = np.arange(w * w).reshape(w, w)
    e = [(i[:, :-1], i[:, 1:]), (i[:-1], i[1:]), (i[:-1, :-1], i[1:, 1:])]
    return np.concatenate([a.ravel() for a, _ in e]), np.concatenate([b.ravel() for _, b in e])


def _power(n, m, seed=1):
    rng = np.random.default_rng(seed)
    c = np.cumsum(np.arange(1, n + 1) ** -0.9)
    return tuple(np.searchsorted(c, rng.random(m) * c[-1]) for _ in range(2))


def _hubs(n, sizes, extra, seed=2):
    rng = np.random.default_rng(seed)
    u = np.concatenate([np.full(d, i) for i, d in enumerate(sizes)] + [rng.integers(0, n, extra)])
    v = np.concatenate([rng.choice(n - len(sizes), d, replace=False) + len(sizes) for d in sizes] +
                       [rng.integers(0, n, extra)])
    return u, v


def _graph(n, *parts):
    u, v = np.concatenate([p[0] for p in parts]), np.concatenate([p[1] for p in parts])
    ok = u != v
    rng = np.random.default_rng(n)
    name = rng.permutation(n).astype(np.uint32)
    t = np.sort(rng.integers(0, 1000, int(ok.sum()))).astype(np.int64)
    return _G(f"chains(n={n})", n, name[u[ok]], name[v[ok]], t)


GRAPHS = {
    "path of one block": lambda: _graph(1000, _chain(1000)),
    "path in one workgroup": lambda: _graph(16000, _chain(16000)),
    "path on the grid": lambda: _graph(60000, _chain(60000)),
    "thick chain": lambda: _graph(3000, _chain(3000, 5)),
    "thick chain on the grid": lambda: _graph(30000, _chain(30000, 5)),
    "lattice": lambda: _graph(40000, _lattice(200)),
    "beside a power law": lambda: _graph(31000, _power(30000, 300000), _chain(1001, 4, 29999)),
    "behind leaves": lambda: _graph(90000, _chain(60000, 4), (60000 + np.arange(30000), np.arange(30000) * 2)),
    "behind leaves, both": lambda: _graph(91000, _power(30000, 300000), _chain(31000, 3, 29999),
                                          (60999 + np.arange(30001), np.arange(30001))),
    "shared rows": lambda: _graph(40000, _hubs(40000, [2047, 2048, 2049, 3000, 17000, 30000], 50000)),
    "many shared rows": lambda: _graph(65536, _hubs(65536, [2100] * 30 + [9000] * 12 + [60000] * 2, 100000)),
}


@pytest.mark.parametrize("name", GRAPHS)
def test_orders(ctx, name):
    g = GRAPHS[name]()
    _, core = oracle.stats(g.n, g.src, g.dst, g.t, core=True)
    pairs = _static_pairs(g)
    query = (200, 100, 150, dt.INT64_MIN, dt.DT_INF)
    want = oracle.cpu_dottt(g.n, g.src, g.dst, g.t, *query)
    for tail in (0, 16000):
        assert (_check(ctx, g, 0, tail, core, pairs, query) == want).all(), tail


@pytest.mark.parametrize("name", ["path on the grid", "thick chain on the grid", "lattice", "beside a power law"])
def test_phases_of_a_chain_end(ctx, name):
    """Far fewer rounds than a phase for every hop (15,000 and more on the first two, 997 on the last)."""
    g = GRAPHS[name]()
    say("rounds", name)
    h = dt.dt_graph_load(ctx, g.n, g.src, g.dst, g.t)
    dt.dt_graph_build(h)
    rounds = dt.dt_graph_stats(h)["peel_rounds"]
    dt.dt_graph_free(h)
    assert rounds < 900 and (name != "lattice" or rounds < 150), rounds


def _phases(g, pairs):
    """Phases of bounds that fall at once to the largest t such that t neighbours have bounds of at least t."""
    u = np.concatenate(pairs)
    v = np.concatenate(pairs[::-1])
    start = np.concatenate([[0], np.cumsum(np.bincount(u, minlength=g.n))])
    h, n = np.diff(start), 0
    while True:
        order = np.lexsort((-h[v], u))           # every vertex's neighbours by falling bound
        w = u[order]
        new = np.bincount(w, h[v][order] >= np.arange(w.shape[0]) - start[w] + 1, minlength=g.n).astype(np.int64)
        new, n = np.minimum(new, h), n + 1
        if (new == h).all():
            return n
        h = new


def test_shared_rows_are_exact(ctx):
    """Every row of more than 1,024 entries is walked by a whole block, whose new bounds are exact: as many
    phases as bounds that fall all the way at once need."""
    g = GRAPHS["shared rows"]()
    say("rounds", g.name)
    h = dt.dt_graph_load(ctx, g.n, g.src, g.dst, g.t)
    dt.dt_graph_build(h)
    rounds = dt.dt_graph_stats(h)["peel_rounds"]
    dt.dt_graph_free(h)
    assert rounds == _phases(g, _static_pairs(g))
