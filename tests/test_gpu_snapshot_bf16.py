"""One SNAPSHOT batch over bfloat16 tables at every lane layout, element by element: each touched row is the
stochastic rounding of its binary64 sum with the Philox bits that belong to (batch, table, row, unit).

The GPU's sums differ from binary64's by their binary32 parts and the fast exponential and reciprocal:
increments of 1e-2 of an element to 2e-6 of themselves, and the sum is rounded to binary32 (6e-8).  A
rounding decision compares 16 bits, steps of 2^-16 of a bfloat16 spacing of at least 2^-8, 6e-8 of the
element: at most about three steps' difference, so 3 of 65,536 decisions may differ.  The bound is 1 in
1,000; a wrong word of the bits gives half of them.
"""
import numpy as np
import pytest

from synth.graphs import Graph

from gpu_util import trainer_for

pytestmark = pytest.mark.gpu


def _bits(seed, batch, table, row, d):
    """16 bits per element of a row: block unit / 8 holds 32 bits for each of 8 units of two elements."""
    words = [np.random.Philox(key=np.array([seed, 2 << 32], np.uint64),
                              counter=np.array([batch - 1, table, row, k], np.uint64)).random_raw(4)
             for k in range((d // 2 + 7) // 8)]
    return np.concatenate(words).view(np.uint16)[:d].astype(np.uint32)


@pytest.mark.parametrize("d,K,orders", [(8, 8, 3), (24, 5, 2), (64, 8, 3), (136, 3, 3), (200, 8, 1), (264, 5, 3), (512, 8, 3)])
def test_bfloat16_batch_element_by_element(d, K, orders):
    n, B, T, eta0, lam, seed = 200, 48, 1000, 0.4, 0.01, 11
    rng = np.random.default_rng(d)
    g = Graph(n=n, src=rng.integers(0, n, 2000).astype(np.int32), dst=rng.integers(0, n, 2000).astype(np.int32),
              w=np.ones(2000, np.float32))
    tr = trainer_for(g, d=d, K=K, orders=orders, dtype="bf16", eta0=eta0, lam=lam, seed=seed, total_samples=T,
                     mode="snapshot", batch=B)
    tables = ((0, 1) if orders & 2 else ()) + ((2,) if orders & 1 else ())
    X = {}
    for t in tables:
        tr.write(t, (rng.standard_normal((n, d)) / np.sqrt(d)).astype(np.float32))
        X[t] = tr.read(t).cpu().numpy().astype(np.float64)  # (rounded to bfloat16)
    u, v, neg = (x.cpu().numpy() for x in tr.sample(B, B))
    ids = np.concatenate([v[:, None], neg], axis=1)
    eta = eta0 * (1.0 - np.arange(B, 2 * B) / T)[:, None]
    inc = {t: np.zeros((n, d)) for t in tables}
    touched = {t: np.zeros(n, bool) for t in tables}
    for A, C in ([(0, 1)] if orders & 2 else []) + ([(2, 2)] if orders & 1 else []):
        a, b = X[A][u], X[C][ids]
        sg = 1.0 / (1.0 + np.exp(-np.einsum("id,ijd->ij", a, b)))
        gr = np.concatenate([eta * (1.0 - sg[:, :1]), -eta * sg[:, 1:]], axis=1)
        np.add.at(inc[A], u, np.einsum("ij,ijd->id", gr, b) - (1 + K) * eta * lam * a)
        np.add.at(inc[C], ids.ravel(), (gr[:, :, None] * a[:, None] - eta[:, :, None] * lam * b).reshape(-1, d))
        touched[A][u] = True
        touched[C][ids.ravel()] = True
    tr.train_steps(B, B)
    tr.check()
    for t in tables:
        got = tr.read(t).cpu().numpy()
        assert np.array_equal(got[~touched[t]], X[t][~touched[t]].astype(np.float32))
        rows = np.flatnonzero(touched[t])
        want = (X[t] + inc[t]).astype(np.float32)[rows]
        bits = np.stack([_bits(seed, 1, t, int(r), d) for r in rows])
        pick = (((want.view(np.uint32).astype(np.uint64) + bits) >> 16) << 16).astype(np.uint32).view(np.float32)
        assert np.mean(got[rows] != pick) <= 1e-3, (t, np.mean(got[rows] != pick))
    tr.close()
