"""How many random numbers a run of Alg. 1 in a batch needs where it uses up
its space: one for each draw it makes, the one that finds nothing included."""
import numpy as np
import pytest

import synth
from tests.helpers import cgs
from tests.test_gpu_batch_tune import _ep, _setup

pytestmark = pytest.mark.gpu


def _needed(n, draws):
    """The start, then iterations of up to `draws` draws until one finds nothing."""
    left, u = n - 1, 1
    while True:
        if left == 0:
            return u + 1                      # the last iteration's only draw
        made = min(left, draws)
        left -= made
        u += made + (1 if made < draws else 0)


# runs: 64 are made on the device, 2 with a launch per iteration
@pytest.mark.parametrize("runs", [2, 64])
@pytest.mark.parametrize("radix,draws", [((3, 2), 4), ((3, 4, 2), 5), ((5, 7, 3), 33), ((2,), 3)])
def test_numbers_are_used_one_per_draw(radix, draws, runs):
    m = cgs()
    sp, table, model = _setup(m, radix, 3)
    need = _needed(sp.n_valid, draws)
    U = np.stack([synth.uniforms_u64(synth.rng(99, i), need + 40) for i in range(runs)])

    def run(k):
        batch = m.Batch([m.Session(sp) for _ in range(runs)], [model] * runs)
        return batch.tuning_run(table.runtime, table.counters, U[:, :k], draws=draws, max_tests=1000,
                                stop_at_well=False, expert=_ep(m))

    want = run(need + 40)
    for a, b in zip(want, run(need)):
        assert a[0].tolist() == b[0].tolist() and a[2] == b[2]
    with pytest.raises(m.CgsError) as ei:
        run(need - 1)
    assert ei.value.status == m.ERANGE and f"needs more than {need - 1}" in str(ei.value)
