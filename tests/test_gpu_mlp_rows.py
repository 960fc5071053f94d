"""The surrogate's gradient over every number of rows its reduction adds (a row
per 64 samples, at most 64): each sum is that of its 64-sample pieces, added as
the reduction adds them, bit for bit.  The weights are scaled by powers of two
only between the two (the loss is a mean), so nothing else rounds."""
import numpy as np
import pytest

import workloads
from oracle import mlp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("rows", [1, 2, 3, 4, 5, 7, 8, 16, 33, 62, 63, 64])
def test_gradient_is_the_sum_of_its_rows(rows):
    import paper_1606_02862_amd as P
    n = 64 * rows
    g = workloads.rng(21)
    T, ne, Z = workloads.loguniform_rate_inputs(22, n)
    X = np.asarray(mlp.features(T, ne, Z), dtype=np.float32)
    t = g.normal(size=n).astype(np.float32)
    p = np.concatenate([np.asarray(v, dtype=np.float32).ravel() for v in
                        (lambda q: [q[k] for k in ("W1", "b1", "W2", "b2", "W3", "b3")])(mlp.init_params(4))])
    with P.Pic(workloads.reduced(3, 8, 8, 4)) as pic:
        pic.mlp_set_params(1, p, [0.0, 1.0])
        loss, grad = pic.mlp_loss_grad(1, X, t)
        again = pic.mlp_loss_grad(1, X, t)
        pieces = [pic.mlp_loss_grad(1, X[64 * r:64 * r + 64], t[64 * r:64 * r + 64]) for r in range(rows)]
    assert loss == again[0] and np.array_equal(grad, again[1])
    assert np.isclose(loss, np.mean([q[0] for q in pieces]), rtol=1e-12)
    # the mean's factor 2 / n is folded in before FP32 and BF16 roundings, so the
    # pieces' sums agree to those, and exactly where n / 64 is a power of two
    G = np.array([q[1] for q in pieces], dtype=np.float32)
    if rows & (rows - 1) == 0:
        G = G / np.float32(rows)
        part = np.zeros((4, G.shape[1]), dtype=np.float32)
        for r in range(rows):
            part[r % 4] += G[r]
        want = (part[0] + part[1]) + (part[2] + part[3])
        assert np.array_equal(grad, want)
    else:
        want = G.astype(np.float64).mean(axis=0)
        scale = np.abs(G).astype(np.float64).max() + 1e-30
        assert np.abs(grad - want).max() <= 2.0**-8 * scale
