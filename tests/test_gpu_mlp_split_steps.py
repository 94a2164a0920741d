"""Adam steps whose rows are split over columns (512 hidden units, up to 1,024
rows) against the gradients of single calls, which are not split: the same
losses, and two steps in closed form from the gradients before each."""
import numpy as np
import pytest

import synth
from tests.helpers import cgs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("radix,C,n", [([4, 3, 5, 2, 4, 3], 12, 1), ([4, 3, 5, 2, 4, 3], 33, 17), ([2, 3] * 10, 40, 45),
                                       ([4, 3, 5, 2, 4, 3], 32, 1001), ([4, 3, 5, 2, 4, 3], 24, 1024)])
def test_two_steps_follow_the_gradients(radix, C, n):
    m = cgs()
    F, H = len(radix), 512
    cons = [("LE", 2 * j, 2 * j + 1, 0, 0) for j in range(8)] if F == 20 else []
    sp = m.Space(radix, [list(range(1, r + 1)) for r in radix], cons)
    g = synth.rng(125, F, C, n)
    init = synth.mlp_init((125, C, n), F, H, C)
    b = [synth.normal_noise(g, (k,), 0.1) for k in (H, H, C)]
    model = m.MLPModel(sp, [init.w[0], b[0], init.w[1], b[1], init.w[2], b[2]])
    rows = [sp.copy_valid()[g.integers(0, sp.n_valid, n)] for _ in range(2)]
    T = [synth.normal_noise(g, (n, C), s).astype(np.float32) for s in (1.0, 3.0)]
    idx = np.arange(n, dtype=np.int32)[None]
    lr, b1, b2, eps = 1e-3, 0.9, 0.999, 1e-8
    mom, var = 0.0, 0.0
    theta = model.copy_params().astype(np.float64)
    for t in (1, 2):
        flat, loss = model.gradients(rows[t - 1], T[t - 1])
        losses = model.train(rows[t - 1], T[t - 1], idx, lr=lr, beta1=b1, beta2=b2, eps=eps)
        assert losses[0] == np.float32(loss)
        grad = flat.astype(np.float64)
        mom, var = b1 * mom + (1 - b1) * grad, b2 * var + (1 - b2) * grad * grad
        theta = theta - lr * (mom / (1 - b1 ** t)) / (np.sqrt(var / (1 - b2 ** t)) + eps)
        got = model.copy_params().astype(np.float64)
        # float32 moments and quotient: a few ulps of a step of at most lr sqrt(2), and of theta
        assert (np.abs(got - theta) <= 1e-5 * lr + 2.0 ** -22 * np.abs(theta)).all(), np.abs(got - theta).max()
        theta = got
