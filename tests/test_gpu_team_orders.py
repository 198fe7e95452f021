"""Launches of wavefront teams for every order, with weight decay, from saved tables: every table ends
where a SNAPSHOT batch of the same samples ends, up to a quarter of one touch of its rows.

Rows have norm 0.25 and a row is touched at most 110 times here (67 on average, K = 8).  A touch adds
about eta / 2 times another row, 1.2e-5, in a direction of its own, and lets the row decay by 1e-5 of itself:
over all of them a row moves by sqrt(110) x 1.2e-5 = 1.3e-4 and 0.11 % of itself, 0.16 % together, and so
do the touches that it gives to others later than SNAPSHOT, which sees it as it was.  110 of these errors
of at most 0.16 % of a touch add up to less than 0.18 of a touch if all had one direction, and to 0.02 as
they have not; binary32 adds 110 x 2^-24 x 0.25, 0.13 of a touch if all had one sign, else 0.01.  A sample too
many or too few is a whole touch.
"""
import numpy as np
import pytest

from synth.graphs import Graph

from gpu_util import trainer_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,K,orders", [(8, 5, 3), (16, 5, 1), (16, 8, 3), (40, 3, 1), (64, 5, 3), (104, 2, 1), (128, 5, 3)])
def test_every_order_applies_each_sample_once(d, K, orders):
    n, eta, lam = 1500, 1e-4, 0.1
    rng = np.random.default_rng(d + orders)
    src = rng.permutation(np.repeat(np.arange(n, dtype=np.int32), 4))
    dst = rng.permutation(np.repeat(np.arange(n, dtype=np.int32), 4))
    g = Graph(n=n, src=src, dst=dst, w=np.ones(4 * n, np.float32))
    tables = ((0, 1) if orders & 2 else ()) + ((2,) if orders & 1 else ())
    saved = {t: (rng.standard_normal((n, d)) * 0.25 / np.sqrt(d)).astype(np.float32) for t in tables}
    for batch, count in ((0, 1), (3, 65), (5, 1000), (1, 10_007)):
        first = batch * count
        kw = dict(d=d, K=K, orders=orders, eta0=eta, lam=lam, seed=count, total_samples=1 << 40)
        a = trainer_for(g, **kw)
        b = trainer_for(g, mode="snapshot", batch=count, **kw)
        for t, x in saved.items():
            a.write(t, x)
            b.write(t, x)
        a.train_steps(first, count)
        b.train_steps(first, count)
        a.check()
        for t, x in saved.items():
            p, q = a.read(t).cpu().numpy().astype(np.float64), b.read(t).cpu().numpy().astype(np.float64)
            assert not np.array_equal(q, x.astype(np.float64))
            touch = eta / 2 * np.linalg.norm(x, axis=1).mean()
            worst = np.linalg.norm(p - q, axis=1).max()
            assert worst <= 0.25 * touch, (t, first, count, worst / touch)
        a.close()
        b.close()
