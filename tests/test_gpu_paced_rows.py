"""bfloat16 launches with six to eight negatives, whose context rows are loaded one at a time when 128 or
more samples in flight want the graph's hottest row.

Arcs of probability 0.06 to one node make any launch with 3,000 samples in flight or more such a launch.  With
hot_rate 0 every row is hot, so that every update is an atomic, which nothing can overwrite.  A step of
1e-4 x (0.05)^2 changes no sigmoid, so the projection of such a launch's change of a table onto the binary32
SNAPSHOT sum of the same samples, from the same rows, is 1.  The roundings of bfloat16 are unbiased:
each unit's is at most 2^-8 x 0.25 a touch, against steps of 2.5e-6 or more, so over the 4.8 million elements or
more of a table the projection's own deviation is below 1 %.  A row that took another row's words
would lose its sample's share.  (The one node's own row is left out: it has thousands of touches.)

A launch with six negatives waits less for the hubs of an R-MAT graph than one with five, whose rows are loaded
together (0.94-0.98 of its time; with its rows together 1.09).
"""
import numpy as np
import pytest
import torch

from synth.graphs import Graph

from gpu_util import trainer_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,K,orders,lanes", [(24, 7, 1, 16), (32, 6, 2, 16), (32, 8, 3, 16), (64, 7, 2, 32),
                                              (72, 6, 1, 64), (72, 8, 2, 64)])
def test_rows_one_at_a_time(d, K, orders, lanes):
    n, T = 200_000, 400_000
    rng = np.random.default_rng(2)
    src, dst = rng.integers(1, n, (2, 8 * n)).astype(np.int32)
    dst[rng.random(8 * n) < 0.06] = 0
    g = Graph(n=n, src=src, dst=dst, w=np.ones(8 * n, np.float32))
    tables = {1: (2,), 2: (0, 1), 3: (0, 1, 2)}[orders]
    gen = torch.Generator().manual_seed(5)
    rows = {t: (torch.rand(n, d, generator=gen) * 0.1 - 0.05 + 0.05 * (t == 1)).bfloat16().float() for t in tables}

    def change(**kw):
        tr = trainer_for(g, d=d, K=K, orders=orders, eta0=1e-4, seed=4, total_samples=1 << 40, **kw)
        if kw["dtype"] == "bf16":
            assert tr.kernel_config()["lanes_per_sample"] == lanes and tr.kernel_config()["units_per_lane"] == 1
        for t in tables:
            tr.write(t, rows[t])
        tr.train_steps(0, T)
        tr.check()
        out = {t: (tr.read(t).double().cpu() - rows[t].double())[1:] for t in tables}
        tr.close()
        return out

    whole = change(dtype="fp32", mode="snapshot", batch=T)
    x = change(dtype="bf16", hot_rate=0.0)
    for t in tables:
        kept = float((x[t] * whole[t]).sum() / (whole[t] * whole[t]).sum())
        print(f"table {t} kept {kept:.4f}", flush=True)
        assert abs(kept - 1) <= 0.03


def test_six_negatives_take_no_longer_than_five():
    n, m = 400_000, 6_400_000
    gen = torch.Generator(device="cuda").manual_seed(3)
    src, dst = torch.zeros((2, m), dtype=torch.int64, device="cuda")
    for _ in range(19):  # R-MAT draws, repeated arcs kept; the nodes past n wrap around
        r = torch.rand(m, generator=gen, device="cuda")
        src = 2 * src + (r >= 0.76)
        dst = 2 * dst + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    g = Graph(n=n, src=(src % n).int(), dst=(dst % n).int(), w=torch.ones(m, device="cuda"))

    def launch_ms(K):
        """Median over nine places of the tables, which change a launch's time by 5-10 %."""
        places = []
        for i in range(9):
            pad = torch.empty((1 + 37 * i) << 19, dtype=torch.uint8, device="cuda")
            tr = trainer_for(g, d=32, K=K, orders=3, dtype="bf16", seed=3, total_samples=1 << 40)
            ms = []
            for _ in range(8):
                tr.train_steps(0, 1_000_000)
                ms.append(tr.last_train_ms())
            tr.close()
            del pad
            torch.cuda.empty_cache()
            places.append(sorted(ms)[2])
        return sorted(places)[4]

    five, six = launch_ms(5), launch_ms(6)
    print(f"five {five:.3f} ms six {six:.3f} ms ratio {six / five:.3f}", flush=True)
    assert six <= 1.04 * five
