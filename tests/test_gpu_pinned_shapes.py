"""A pinned kernel configuration runs as it was pinned: its wavefronts take their own tiles, as many
of them as max_conflicts allows.

The number in flight is read off what racing stores lose: with hot_rate = 1e31 no row takes atomics,
and of the updates of a row that a sample touches with probability p about 1 / (1 + W p) are kept
when W samples are in flight.  SNAPSHOT's one batch adds every touch, each eta / 2 times a vertex row,
so the projection of a Hogwild launch's change onto SNAPSHOT's is the share of touches that were kept.
"""
import numpy as np
import pytest

from synth.graphs import Graph

from gpu_util import trainer_for

pytestmark = pytest.mark.gpu


def test_a_pinned_shape_on_a_small_table_keeps_the_staleness_cap():
    """(64, 1) at d = 16: a workgroup holds 4 samples, and max_conflicts allows 4."""
    n, mids, T, K = 3000, 10, 100_000, 1
    rng = np.random.default_rng(2)
    m = 8 * n
    src = rng.integers(mids, n, m).astype(np.int32)
    dst = np.where(rng.random(m) < 0.5, rng.integers(0, mids, m), rng.integers(mids, n, m)).astype(np.int32)
    g = Graph(n=n, src=src, dst=dst, w=np.ones(m, np.float32))

    def change(**kw):
        tr = trainer_for(g, d=16, K=K, orders=2, eta0=1e-4, seed=4, total_samples=1 << 40, **kw)
        if "mode" not in kw:
            tr.set_kernel_config(64, 1, 1)
        before = tr.read(1)[:mids].double()
        tr.train_steps(0, T)
        tr.check()
        x = (tr.read(1)[:mids].double() - before).cpu().numpy()
        tr.close()
        return x

    whole = change(mode="snapshot", batch=T)
    x = change(hot_rate=1e31, max_conflicts=4.0 * (2 + K) / n + 1e-9)
    kept = float((x * whole).sum() / (whole * whole).sum())
    print(f"kept {kept:.3f}", flush=True)
    # p = 0.05: at most 4 in flight keep 1 / 1.2, 64 would keep 1 / 4
    assert kept > 0.6
