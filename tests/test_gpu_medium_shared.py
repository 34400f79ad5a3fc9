"""The medium path where a workgroup shares its wavefronts' largest groups of entries: triangles with long
pairs beside short ones, entry lists from a few hundred to beyond a million (one launch for all paths, then
one a path, with one and two groups a wavefront), deltas on both sides of the one from which groups are
shared, windows; against the oracle."""
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


def _graph(lengths, span, seed=7):
    """A disjoint triangle per entry of lengths: two pairs of about that many edges, a third one shorter."""
    rng = np.random.default_rng([seed, len(lengths)])
    src, dst = [], []
    for i, k in enumerate(lengths):
        pairs = [(0, 1), (0, 2), (1, 2)]
        rng.shuffle(pairs)
        for (a, b), m in zip(pairs, (k, max(1, k - int(rng.integers(0, k))), 1 + int(rng.integers(0, 40)))):
            flip = rng.random(m) < rng.choice([0.0, 0.3, 1.0])
            src.append(3 * i + np.where(flip, b, a))
            dst.append(3 * i + np.where(flip, a, b))
    src, dst = np.concatenate(src), np.concatenate(dst)
    p = rng.permutation(src.shape[0])
    t = rng.integers(0, span, src.shape[0])
    return synth.TemporalGraph(3 * len(lengths), src[p].astype(np.uint32), dst[p].astype(np.uint32),
                               np.sort(t).astype(np.int64), name=f"shared{len(lengths)}")


SPAN = 128_000
QUERIES = [(INF, INF, INF), (SPAN, 50_000, 70_000), (1000, 700, 600), (999, 999, 999), (998, 400, 998), (5, 5, 5),
           (INF, INF, INF, 30_000, 90_000)]


@pytest.mark.parametrize("lengths", [
    [300], [3, 900, 5, 40], [511, 512, 513, 514] + [2] * 300, [60] * 500 + [1500] * 3,
    [150] * 2500 + [1100] * 40, [4] * 20_000 + [700] * 1200], ids=lambda x: str(len(x)))
def test_shared_groups(ctx, lengths):
    g = _graph(lengths, SPAN)
    b = Built(ctx, g, g.name, path=3)
    for q in QUERIES:
        assert np.array_equal(b.count(*q), oracle.cpu_dottt(g.n, g.src, g.dst, g.t, *q)), q
    b.free()
