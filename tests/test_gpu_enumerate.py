"""The enumeration's work split: runs of consecutive vertices packed into one LDS slice, and the
tickets' classes (split, single, four and many vertices).  The static triangles equal the oracle's,
and so does the one-shot count (the same pass, counting as it finds), around the places where the
split changes: longest runs of 64 and 65 heads, runs whose lengths sum to just past the slice, vertex
counts that are not a multiple of a ticket's, and vertices without any run."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import Built

pytestmark = pytest.mark.gpu

import paper_2106_02762_amd as dt  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    c = dt.dt_ctx_create(0)
    yield c
    dt.dt_ctx_destroy(c)


def _cliques(size, copies, noise_n, seed):
    """`copies` disjoint cliques and `noise_n` further vertices joined to one or two random ones,
    every pair one temporal edge; some vertex ids are used by no edge."""
    rng = np.random.default_rng([seed, size, copies, noise_n])
    iu, ju = np.triu_indices(size, 1)
    base = np.repeat(np.arange(copies) * size, iu.shape[0])
    u, v = np.tile(iu, copies) + base, np.tile(ju, copies) + base
    n = size * copies + noise_n
    k = noise_n + noise_n // 2
    a = size * copies + (np.arange(k) % max(noise_n, 1))
    b = rng.integers(0, n, k)
    ok = (a != b) & (a % 7 != 0)
    u, v = np.concatenate([u, a[ok]]), np.concatenate([v, b[ok]])
    name = rng.permutation(n)
    flip = rng.random(u.shape[0]) < 0.5
    src, dst = np.where(flip, name[v], name[u]), np.where(flip, name[u], name[v])
    t = np.sort(rng.integers(0, 10**5, u.shape[0]))
    return synth.TemporalGraph(n, src.astype(np.uint32), dst.astype(np.uint32), t.astype(np.int64),
                               name=f"cliques({size}x{copies}+{noise_n})")


@pytest.mark.parametrize("size,copies,noise_n", [
    (3, 1, 0), (3, 5000, 0), (33, 40, 1), (33, 40, 4097), (65, 1, 0), (65, 2, 7001), (66, 1, 0),
    (66, 3, 30011), (24, 200, 300007), (130, 2, 25000)])
def test_packs_and_tickets(ctx, size, copies, noise_n):
    g = _cliques(size, copies, noise_n, 3)
    b = Built(ctx, g, g.name)
    st = dt.dt_graph_stats(b.h)
    assert st["max_out_degree"] >= size - 1   # (64 | 65: the two ticket plans)
    want = oracle.triangles(g.n, g.src, g.dst, g.t)
    got = dt.dt_graph_triangles(b.h)
    got = got[np.lexsort((got[:, 2], got[:, 1], got[:, 0]))]
    assert np.array_equal(got, want)
    d = (20000, 9000, 15000)
    ref = oracle.count(g.n, g.src, g.dst, g.t, *d)
    assert np.array_equal(b.count(*d), ref)
    assert np.array_equal(dt.dt_count_oneshot(b.h, *d), ref)
    b.free()
