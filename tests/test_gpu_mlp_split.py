"""Training rows split over columns (512 hidden units, batches up to 1,024
rows): gradients and loss against float64 backprop with the bf16 weights, at
one row, ragged batches, the largest split batch and the first that is not,
one and two output tiles, one and two input K steps.

The tolerances are those of the unsplit rows' tests: activations and deltas
are rounded to bf16 (2^-8 relative each), so a gradient entry may be off by
2e-2 of its layer's largest."""
import numpy as np
import pytest

import synth
from oracle import mlp as M
from oracle import space as SP
from tests.helpers import cgs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("radix,C,n", [([4, 3, 5, 2, 4, 3], 12, 1), ([4, 3, 5, 2, 4, 3], 33, 17),
                                       ([2, 3] * 10, 40, 45), ([4, 3, 5, 2, 4, 3], 32, 1001),
                                       ([4, 3, 5, 2, 4, 3], 24, 1024),
                                       ([4, 3, 5, 2, 4, 3], 24, 1025)])
def test_gradients_and_an_adam_step(radix, C, n):
    m = cgs()
    F, H = len(radix), 512
    cons = [("LE", 2 * j, 2 * j + 1, 0, 0) for j in range(8)] if F == 20 else []
    sp = m.Space(radix, [list(range(1, r + 1)) for r in radix], cons)
    g = synth.rng(95, F, C, n)
    init = synth.mlp_init((95, C, n), F, H, C)
    b = [synth.normal_noise(g, (k,), 0.1) for k in (H, H, C)]
    params = [init.w[0], b[0], init.w[1], b[1], init.w[2], b[2]]
    model = m.MLPModel(sp, params)
    cfg = sp.copy_valid()[g.integers(0, sp.n_valid, n)]
    X = M.features(SP.digits_of(cfg.astype(np.int64), radix))
    T = synth.normal_noise(g, (n, C), 1.0).astype(np.float32)
    pr = [np.asarray(p, np.float64) for p in params]
    pr = [M.bf16(p).astype(np.float64) if i % 2 == 0 else p for i, p in enumerate(pr)]
    loss_ref, g_ref = M.loss_and_grads(pr, X, T.astype(np.float64))
    flat, loss = model.gradients(cfg, T)
    assert abs(loss - loss_ref) <= 1e-2 * loss_ref
    for got, ref in zip(model.unflatten(flat), g_ref):
        got = got.astype(np.float64)
        cos = (got * ref).sum() / np.sqrt((got * got).sum() * (ref * ref).sum())
        assert cos > 0.999, cos
        assert np.abs(got - ref).max() <= 2e-2 * np.abs(ref).max()
    # the first Adam step from the same gradients, in closed form: the moments'
    # corrections cancel, theta - lr g / (|g| + eps)
    losses = model.train(cfg, T, np.arange(n, dtype=np.int32)[None], lr=1e-3)
    assert losses[0] == np.float32(loss)
    want = m.mlp_flatten(params) - 1e-3 * flat / (np.abs(flat) + 1e-8)
    assert np.abs(model.copy_params() - want).max() <= 1e-6
