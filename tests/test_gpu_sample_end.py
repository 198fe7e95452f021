"""Launches that end at the last sample indices that 64 bits can number: the tiles of a launch reach past
its end, and what lies past 2^64 - 1 must not come back as sample 0 (a first sample has the whole step
size, where the last ones have almost none)."""
import numpy as np
import pytest

from synth import rmat_graph

from gpu_util import trainer_for

pytestmark = pytest.mark.gpu

LAST = 2**64 - 1


@pytest.mark.parametrize("dtype,d,n,count", [
    ("fp32", 16, 3000, 1), ("fp32", 16, 3000, 1000), ("fp32", 128, 3000, 70),  # teams
    ("fp32", 32, 60_000, 7), ("bf16", 32, 3000, 7), ("bf16", 128, 3000, 130),
])
def test_no_sample_past_the_last_index_is_trained(dtype, d, n, count):
    g = rmat_graph(int(n - 1).bit_length(), n, 8 * n, seed=5)
    # eta = eta0 (1 - s / T) is exactly 0 in binary64 for every s of this launch (s / T rounds to 1)
    tr = trainer_for(g, d=d, K=5, orders=3, dtype=dtype, eta0=0.5, seed=6, total_samples=LAST)
    before = [tr.read(t).cpu().numpy() for t in (0, 1, 2)]
    tr.train_steps(LAST - count, count)
    tr.check()
    for t, x in enumerate(before):
        assert np.array_equal(tr.read(t).cpu().numpy(), x)
    tr.close()
