"""The lists of a count's schedule around the tiles they are made in (1,024 and 2,048 entries): disjoint
triangles whose pairs hold one to a few dozen edges, split over all paths or forced onto one, some with
pairs of many hundred edges whose work items fill a tile by themselves; whole-span and windowed counts
against the oracle."""
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


def _graph(k, most, span, seed=11):
    """k disjoint triangles with 1..most edges on each pair, every 97th with 40 * most on its pairs; times
    in bursts at the triangle's own place in the span, so that windows cut the list everywhere."""
    rng = np.random.default_rng([seed, k, most])
    src, dst, t = [], [], []
    for i in range(k):
        at = int(rng.integers(0, span))
        for a, b in ((0, 1), (0, 2), (1, 2)):
            m = 40 * most if i % 97 == 5 else int(rng.integers(1, most + 1))
            flip = rng.random(m) < 0.5
            src.append(3 * i + np.where(flip, b, a))
            dst.append(3 * i + np.where(flip, a, b))
            t.append(at + rng.integers(0, 500, m))
    src, dst, t = np.concatenate(src), np.concatenate(dst), np.concatenate(t)
    p = rng.permutation(src.shape[0])
    return synth.TemporalGraph(3 * k, src[p].astype(np.uint32), dst[p].astype(np.uint32), t[p].astype(np.int64),
                               name=f"tiles{k}x{most}")


QUERIES = [(INF, INF, INF), (120, 60, 90), (7, 7, 7), (400, 300, 200, 20_000, 70_000), (90, 90, 90, 50_000, 50_400)]


@pytest.mark.parametrize("path", [0, 2, 3])
@pytest.mark.parametrize("k,most", [(1, 30), (6, 30), (1022, 4), (1023, 20), (1024, 6), (1025, 20), (2047, 9), (2049, 9)])
def test_tiles(ctx, k, most, path):
    g = _graph(k, most, 100_000)
    b = Built(ctx, g, g.name, path=path)
    for q in QUERIES:
        assert np.array_equal(b.count(*q), oracle.cpu_dottt(g.n, g.src, g.dst, g.t, *q)), q
    b.free()
