"""SNAPSHOT batches whose entries end at, before and after the edges of the sort's tiles and of
the 64 entries a wavefront looks at, rows with a few and with thousands of entries, and every
lane layout: binary32 GPU against the binary64 oracle, per row within 1e-5 (the bar of the other
SNAPSHOT tests)."""
import numpy as np
import pytest

import oracle
from synth.graphs import Graph

from gpu_util import max_row_rel_err, trainer_for

pytestmark = pytest.mark.gpu


def _graph(n, m, seed):
    rng = np.random.default_rng(seed)
    return Graph(n=n, src=rng.integers(0, n, m).astype(np.int32), dst=rng.integers(0, n, m).astype(np.int32),
                 w=rng.lognormal(0.0, 1.0, m).astype(np.float32))


@pytest.mark.parametrize("n,d,K,orders,B", [
    (3, 8, 2, 2, 15), (3, 16, 2, 2, 16), (5, 24, 2, 1, 17),  # 60, 64 and 68 entries over few rows
    (3, 40, 2, 2, 1024), (70_000, 64, 2, 2, 1025),           # 4,096 and 4,100: one tile, two
    (11, 136, 0, 3, 1000), (1_500_000, 264, 5, 1, 585),      # 23 bits of keys: three passes
    (300, 512, 8, 3, 409), (2, 8, 5, 3, 5000),               # thousands of entries a row
])
def test_snapshot_at_the_edges(n, d, K, orders, B):
    import paper_2604_09419_amd as lh
    g = _graph(n, max(4, min(5 * n, 200_000)), seed=n + d)
    T, count = 50_000, 2 * B + B // 2  # the last batch is a short one
    tr = trainer_for(g, d=d, K=K, orders=orders, eta0=0.01, lam=0.01, seed=3, total_samples=T, mode="snapshot", batch=B)
    tr.train_steps(0, count)
    tr.check()
    m = oracle.Model(oracle.Tables(g.n, g.src, g.dst, g.w), d=d, K=K, orders=orders, T=T, seed=3, eta0=0.01, lam=0.01)
    m.train(0, count, "snapshot", B)
    for name, tab, ref in (("U", lh.LH_TABLE_U, m.U), ("C", lh.LH_TABLE_C, m.C), ("U1", lh.LH_TABLE_U1, m.U1)):
        if ref is None:
            continue
        err = max_row_rel_err(tr.read(tab).cpu().numpy(), ref)
        assert err <= 1e-5, (name, err)
