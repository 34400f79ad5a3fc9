"""The pairwise paths around the length at which the third edges are searched instead of read one by
one: {v,w} lists of 1 to 200 edges split unevenly over the two directions, with equal times, counted as
light and as medium triangles against the oracle over deltas, windows that cut the lists, sweeps and
batches."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import INF, Built

pytestmark = pytest.mark.gpu

import paper_2106_02762_amd as dt  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    c = dt.dt_ctx_create(0)
    yield c
    dt.dt_ctx_destroy(c)


def _graph(lengths, seed, t_range=400):
    """One triangle per entry of lengths: its three pairs hold that many edges (shuffled over the
    pairs) and one and two others; a share of each pair's edges, from none to all, points back."""
    rng = np.random.default_rng([seed, len(lengths)])
    src, dst = [], []
    for i, k in enumerate(lengths):
        a, b, c = 3 * i, 3 * i + 1, 3 * i + 2
        pairs = [(a, b), (a, c), (b, c)]
        rng.shuffle(pairs)
        for (x, y), m in zip(pairs, (k, int(rng.integers(1, 3)), int(rng.integers(1, 3)))):
            flip = rng.random(m) < rng.choice([0.0, 0.1, 0.5, 1.0])
            src.append(np.where(flip, y, x))
            dst.append(np.where(flip, x, y))
    src, dst = np.concatenate(src), np.concatenate(dst)
    t = np.sort(rng.integers(0, t_range, src.shape[0]))
    p = rng.permutation(src.shape[0])
    return synth.TemporalGraph(3 * len(lengths), src[p].astype(np.uint32), dst[p].astype(np.uint32), t.astype(np.int64),
                               name=f"thirds{len(lengths)}")


@pytest.mark.parametrize("path", [0, 1, 3])
@pytest.mark.parametrize("lengths", [
    [1, 2, 3, 4, 5, 6, 7, 8, 9, 10], [7] * 70 + [8] * 70 + [9] * 70, [63, 64, 65, 200] * 9])
def test_third_edges(ctx, path, lengths):
    g = _graph(lengths, 3)
    b = Built(ctx, g, g.name, path=path)
    deltas = [(0, 0, 0), (30, 10, 25), (90, 90, 5), (200, 120, 150), (INF, INF, INF)]
    windows = [(dt.INT64_MIN, INF), (100, 300), (199, 201), (390, 1000)]
    for w in windows:
        want = [oracle.count(g.n, g.src, g.dst, g.t, *d, *w) for d in deltas]
        for d, x in zip(deltas, want):
            assert np.array_equal(b.count(*d, *w), x), (d, w)
        assert np.array_equal(dt.dt_count_sweep(b.h, deltas, *w), np.stack(want)), w
        qs = [dt.make_query(*d, *w) for d in deltas]
        assert np.array_equal(dt.dt_count_batch(ctx, [b.h] * len(qs), qs), np.stack(want)), w
    cells = dt.dt_count_cells(b.h, 90, 60, 70)
    assert cells.sum() == oracle.count(g.n, g.src, g.dst, g.t, 90, 60, 70).sum()
    b.free()
