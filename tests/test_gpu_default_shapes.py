"""The binary32 shapes that the library chooses take no row's atomics away: rows of more than 64
elements run four of them a lane, and where narrower rows are spread over more lanes, which leaves fewer
samples in flight, the hot rows are still those of four elements a lane.

The second test reads the kept share of updates as test_gpu_hottest_row.py does: 1,000 nodes of 400,000
are touched with probability 4.5e-5 each.  Four elements a lane keep 33,000 samples in flight there
(max_conflicts), 1.5 of them on such a row, so it is hot; the 8,000 of (32, 1) alone would make it cold
(0.37), and racing stores would lose a tenth or more of its updates.  Each row gets 90 touches; over 1,000
rows of 32 elements the directions of different touches average out to 1 %.
"""
import numpy as np
import pytest

from synth import rmat_graph
from synth.graphs import Graph

from gpu_util import trainer_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n,shape", [(72, 40_000, (32, 4, 8)), (128, 600_000, (32, 4, 8)), (200, 9_000, (64, 4, 8)),
                                       (264, 9_000, (64, 8, 8)), (64, 40_000, (32, 2, 8)), (16, 300_000, (16, 1, 4))])
def test_shapes(d, n, shape):
    hubs = rmat_graph(int(n - 1).bit_length(), n, 4 * n, seed=3)
    tr = trainer_for(hubs, d=d, orders=2, total_samples=1 << 30, init=False)
    assert tuple(tr.kernel_config().values()) == shape
    tr.close()


def test_rows_that_four_elements_a_lane_protect_lose_no_update():
    n, mids, T = 400_000, 1000, 2_000_000
    rng = np.random.default_rng(1)
    m = 8 * n
    src = rng.integers(mids, n, m).astype(np.int32)
    dst = np.where(rng.random(m) < 0.045, rng.integers(0, mids, m), rng.integers(mids, n, m)).astype(np.int32)
    g = Graph(n=n, src=src, dst=dst, w=np.ones(m, np.float32))

    def change(**kw):
        tr = trainer_for(g, d=32, K=1, orders=2, eta0=1e-4, seed=4, total_samples=1 << 40, **kw)
        before = tr.read(1)[:mids].double()
        tr.train_steps(0, T)
        tr.check()
        x = (tr.read(1)[:mids].double() - before).cpu().numpy()
        tr.close()
        return x

    whole, x = change(mode="snapshot", batch=T), change()
    kept = float((x * whole).sum() / (whole * whole).sum())
    print(f"kept {kept:.4f}", flush=True)
    assert kept >= 0.985
