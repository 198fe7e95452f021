"""Hogwild launches of every length: tiles shorter than 64 samples, launches with and without a
tile counter, ragged ends, K on both sides of the compiled maxima and rows that no shape covers
exactly.  With eta0 = 0 a launch leaves the tables bitwise as they were, and a short launch of
samples that share no row gives what SNAPSHOT batches of one sample give."""
import numpy as np
import pytest

from synth import rmat_graph

from gpu_util import max_row_rel_err, trainer_for

pytestmark = pytest.mark.gpu


def _tables(tr, orders):
    return [tr.read(t).cpu().numpy() for t in ((0, 1) if orders & 2 else ()) + ((2,) if orders & 1 else ())]


@pytest.mark.parametrize("dtype,d,K,orders,n", [
    ("fp32", 16, 5, 2, 3000), ("fp32", 16, 3, 3, 3000), ("fp32", 72, 8, 2, 9000), ("fp32", 64, 5, 3, 40_000),
    ("fp32", 128, 5, 2, 40_000), ("fp32", 200, 3, 1, 3000), ("bf16", 24, 8, 2, 3000), ("bf16", 128, 1, 3, 40_000),
])
def test_zero_step_launches_of_every_length_leave_tables_bitwise(dtype, d, K, orders, n):
    g = rmat_graph(int(n - 1).bit_length(), n, 8 * n, seed=5)
    tr = trainer_for(g, d=d, K=K, orders=orders, dtype=dtype, eta0=0.0, seed=6, total_samples=1 << 20)
    before = _tables(tr, orders)
    for first, count in ((0, 1), (3, 2), (7, 15), (0, 63), (1, 64), (2, 65), (5, 257), (0, 4097), (11, 100_003)):
        tr.train_steps(first, count)
    tr.check()
    for x, y in zip(before, _tables(tr, orders)):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("d,K,orders", [(16, 5, 2), (72, 8, 3), (200, 3, 1), (64, 5, 3)])
@pytest.mark.parametrize("count", [1, 5])
def test_short_launches_apply_each_sample_once(d, K, orders, count):
    """Samples that share no row do not race, so a launch of a few of them gives what SNAPSHOT
    batches of one give (binary32: each row gets one rounded update either way; 2^-20 covers the
    different order of a dot product's sum).  The graph is a perfect matching on many nodes."""
    n = 200_000
    src = np.arange(0, n, 2, dtype=np.int32)
    g = type("G", (), dict(n=n, src=src, dst=src + 1, w=np.ones(n // 2, np.float32)))
    kw = dict(d=d, K=K, orders=orders, eta0=0.05, seed=9, total_samples=1000, lam=0.01)
    a = trainer_for(g, **kw)
    first = 0
    while True:  # the first stretch of samples without a shared row
        u, v, neg = (x.cpu().numpy() for x in a.sample(first, count))
        rows = np.concatenate([u, v, neg.reshape(-1)])
        if np.unique(rows).size == rows.size:
            break
        first += 1
    b = trainer_for(g, mode="snapshot", batch=1, **kw)
    a.train_steps(first, count)
    b.train_steps(first, count)
    for x, y in zip(_tables(a, orders), _tables(b, orders)):
        assert not np.array_equal(x, np.zeros_like(x))
        assert max_row_rel_err(x, y) <= 2.0 ** -20
