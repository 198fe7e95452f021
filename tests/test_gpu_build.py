"""The alias build's kernels at the sizes where they change path or can go wrong: the degree
counts' three ways, tiles and chunks with remainders, and weights whose light and heavy halves
are of very different lengths (so that a workgroup's stretch of the other half does not fit in
LDS).  Every table must equal the oracle's bit for bit."""
import numpy as np
import pytest

import oracle
from synth.graphs import Graph

from gpu_util import trainer_for

pytestmark = pytest.mark.gpu


def _weights(kind, m, rng):
    if kind == "unit":
        return np.ones(m, np.float32)
    if kind == "lognormal":
        return rng.lognormal(0.0, 1.0, m).astype(np.float32)
    if kind == "few_lights":  # a few empty arcs among many just above the mean
        w = rng.uniform(1.0, 1.001, m).astype(np.float32)
        w[rng.choice(m, max(1, m // 5000), replace=False)] = 0.0
        return w
    if kind == "few_heavies":  # nearly all the weight on a few arcs
        w = rng.uniform(0.9, 1.0, m).astype(np.float32)
        w[rng.choice(m, max(1, m // 20000), replace=False)] = 1e6
        return w
    raise ValueError(kind)


def _ends(order, n, m, rng):
    x = rng.integers(0, n, m)
    x[: m // 3] = n - 1  # one node with a third of the arcs
    if order == "sorted":
        x.sort()
    else:
        rng.shuffle(x)
    return x.astype(np.int32)


@pytest.mark.parametrize("n,m,weights,order", [
    (1, 1, "unit", "shuffled"),
    (3, 70, "few_lights", "sorted"),
    (32768, 32769, "lognormal", "shuffled"),       # a counter per node in LDS, all of it
    (32769, 32769, "unit", "sorted"),              # two ranges, the second of one node
    (70_001, 262_145, "few_heavies", "shuffled"),  # tiles and ranges with remainders
    (32769, 32000, "lognormal", "shuffled"),       # fewer arcs than nodes: plain atomics
    (150_000, 700_001, "few_lights", "shuffled"),
    ((1 << 21) + 1, (1 << 21) + 5, "lognormal", "sorted"),  # more ranges than the tiles sort
])
def test_alias_tables_at_the_edges_of_the_build(n, m, weights, order):
    import paper_2604_09419_amd as lh
    rng = np.random.default_rng(n + m)
    g = Graph(n=n, src=_ends(order, n, m, rng), dst=_ends("shuffled", n, m, rng), w=_weights(weights, m, rng))
    t = oracle.Tables(g.n, g.src, g.dst, g.w)
    tr = trainer_for(g, d=8, total_samples=10, init=False)
    tr.check()
    for which, thr, alias in ((lh.LH_ALIAS_EDGE, t.ethr, t.ealias), (lh.LH_ALIAS_NEG, t.nthr, t.nalias)):
        gthr, galias = tr.export_alias(which)
        assert np.array_equal(galias, alias), (which, int((galias != alias).sum()))
        assert np.array_equal(gthr, thr), (which, int((gthr != thr).sum()))
    tr.close()
