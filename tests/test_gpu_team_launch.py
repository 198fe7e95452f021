"""Hogwild launches in which several wavefronts share a stream of sample tiles (binary32 tables that
fit in one L2): every sample is applied once, whatever the width, the number of negatives and the
length of the launch.

A step size of 1e-4 keeps the tables near where they began, so a launch adds the sum of its samples'
increments at the start, which is what one SNAPSHOT batch adds.  From zero context rows an element
of a context row gets +-eta/2 times an element of a vertex row per touch.  Over the at most 200
touches of a row here the vertex rows move by less than 200 eta^2 / 4 x 200 = 1e-4 of themselves, the
dot products' effect on the step sizes is smaller, and binary32 sums add 200 x 2^-24, so all touches
together are off by less than 200 x 3e-4 = 0.06 of one touch.  A sample too many or too few shows as
a whole touch: the bound is a quarter of the greatest.
"""
import numpy as np
import pytest

from synth.graphs import Graph

from gpu_util import trainer_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,K", [(8, 5), (16, 5), (16, 8), (24, 3), (32, 5), (64, 5), (104, 5), (128, 2)])
def test_every_sample_is_applied_once(d, K):
    n, eta = 3000, 1e-4
    rng = np.random.default_rng(d)
    src = rng.permutation(np.repeat(np.arange(n, dtype=np.int32), 4))
    dst = rng.permutation(np.repeat(np.arange(n, dtype=np.int32), 4))
    g = Graph(n=n, src=src, dst=dst, w=np.ones(4 * n, np.float32))
    for batch, count in ((0, 1), (3, 63), (0, 64), (5, 65), (1, 256), (7, 1000), (0, 4097), (9, 21_001)):
        first = batch * count  # (a SNAPSHOT range starts at a batch)
        kw = dict(d=d, K=K, orders=2, eta0=eta, seed=count, total_samples=1 << 40)
        a = trainer_for(g, **kw)
        b = trainer_for(g, mode="snapshot", batch=count, **kw)
        u = a.read(0).cpu().numpy()
        a.train_steps(first, count)
        b.train_steps(first, count)
        a.check()
        x, y = a.read(1).cpu().numpy(), b.read(1).cpu().numpy()
        assert np.abs(y).max() > 0
        # (a touch is as large as the vertex row's largest element: at least half of the table's here)
        assert np.abs(x - y).max() <= 0.25 * 0.5 * eta / 2 * np.abs(u).max(), (first, count)
        a.close()
        b.close()
