"""The binary32 shape of large tables follows the hub rows' share of the touches: two samples a
wavefront, eight workgroups per compute unit, where no row is hot; one sample where hubs are."""
import numpy as np
import pytest

from synth import rmat_graph
from synth.graphs import Graph

from gpu_util import trainer_for

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hubs():
    return rmat_graph(20, 1 << 20, 1 << 23, seed=3)


def _cfg(g, **kw):
    tr = trainer_for(g, d=128, orders=2, total_samples=1 << 30, init=False, **kw)
    c = tr.kernel_config()
    tr.close()
    return tuple(c.values())


def test_large_binary32_tables_without_hubs_take_two_samples_a_wavefront(hubs):
    n = 600_000  # 614 MB of tables
    a = np.arange(n, dtype=np.int32)
    ring = Graph(n=n, src=a, dst=((a + 1) % n).astype(np.int32), w=np.ones(n, np.float32))
    assert _cfg(ring) == (32, 4, 8)
    assert _cfg(hubs) == (64, 2, 4)
    assert _cfg(hubs, hot_rate=1e31) == (32, 4, 8)  # no row takes atomics


def test_short_launches_of_large_tables_are_no_slower_than_two_samples_a_wavefront(hubs):
    """40,000 samples: (64, 2) took 1.5 times the time of (32, 4)."""
    tr = trainer_for(hubs, d=128, orders=2, seed=3, total_samples=1 << 30)

    def best():
        times = []
        for _ in range(40):
            tr.train_steps(1 << 29, 40_000)
            times.append(tr.last_train_ms())
        return min(times)

    default = best()
    tr.set_kernel_config(32, 4, 8)
    pinned = best()
    tr.close()
    print(f"default {default:.4f} ms, pinned {pinned:.4f} ms", flush=True)
    assert default < 1.25 * pinned
