"""Rows of the walk graph at the sizes where their kernels change path or can go wrong: rows that
fit one workgroup (up to 256 entries) and longer ones, tiles that rows straddle, chunks, groups
of 16 chunks, rows of more chunks than a wavefront has lanes, rows of zero weight, workgroups without a row of their own.  Whole numbers,
so bit for bit against the oracle.
"""
import numpy as np
import pytest

import oracle
from synth.graphs import Graph

from gpu_util import trainer_for

pytestmark = pytest.mark.gpu

CASES = {
    "single_entries": [1] * 2500,
    "around_eight": [7, 8, 9, 15, 16, 17] * 60,
    "limit_of_short": [255, 256, 257, 1, 256, 256, 257] * 12,
    "straddling": [250, 30, 256, 2, 255, 700, 210, 210] * 10,
    "one_chunk": [1023, 1024, 1025, 1, 300, 1024],
    "chunks": [2047, 2048, 2049, 3, 3000, 5000],
    "group_of_chunks": [16 * 1024, 16 * 1024 + 1, 5, 17 * 1024 - 1, 33 * 1024],
    "lanes": [64 * 1024 - 1, 64 * 1024, 64 * 1024 + 1, 63 * 1024 + 1],
    "levels": [1025 * 1024 + 3, 4, 2000],
}


def _graph(lens, seed, zero):
    """Vertex x with lens[x] arcs to or from random other vertices (a large pool: their own rows stay
    short), half of them pointing each way; `zero`: every third vertex's weights are all 0."""
    rng = np.random.default_rng(seed)
    hub = np.repeat(np.arange(len(lens), dtype=np.int32), lens)
    pool = max(64, 2 * hub.size)
    other = rng.integers(len(lens), len(lens) + pool, size=hub.size).astype(np.int32)
    flip = rng.random(hub.size) < 0.5
    w = rng.lognormal(0, 1.5, size=hub.size).astype(np.float32)
    if zero:
        w[hub % 3 == 1] = 0.0
    return Graph(n=len(lens) + pool, src=np.where(flip, other, hub).astype(np.int32),
                 dst=np.where(flip, hub, other).astype(np.int32), w=w)


@pytest.mark.parametrize("zero", [False, True])
@pytest.mark.parametrize("case", list(CASES))
def test_walk_rows_at_edges(case, zero):
    lens = CASES[case]
    g = _graph(lens, len(lens), zero)
    print(f"walk rows {case} zero={zero}: n={g.n} m={g.m}", flush=True)
    tr = trainer_for(g, d=8, K=2, orders=2, seed=5, total_samples=10, init=False)
    tr.build_walks(walk_length=10, window=2, walks_per_batch=64)
    wg = oracle.WalkGraph(oracle.Tables(g.n, g.src, g.dst, g.w), L=10, W=2, Bw=64)
    assert np.array_equal(np.diff(wg.off)[:len(lens)], lens)
    off, thr, keep, al = tr.walk_export()
    rows = np.repeat(np.arange(wg.off.size - 1), np.diff(wg.off))
    assert np.array_equal(off, wg.off)
    assert np.array_equal(thr, wg.thr)
    assert np.array_equal(keep, wg.nbr)
    assert np.array_equal(al, wg.nbr[wg.off[rows] + wg.alias])
    tr.close()
