"""Values a caller gives are checked on the device: the lowest bad position is
named, at the ends and around the check's strides; bad values leave no model,
good ones at the limits of their range do."""
import numpy as np
import pytest

import synth
from tests.helpers import cgs

pytestmark = pytest.mark.gpu


def _expect(m, build, at, what):
    with pytest.raises(m.CgsError) as ei:
        build()
    assert ei.value.status == m.EINVAL
    assert f"{what} {at} " in str(ei.value)


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf, -1e-30, -np.float32(3)])
@pytest.mark.parametrize("at", [0, 255, 1024, 4999, 9599])
def test_bad_leaf_or_prediction_is_named(value, at):
    m = cgs()
    spec = synth.Space([8, 5, 10], [list(range(1, r + 1)) for r in (8, 5, 10)])
    sp = m.Space.from_spec(spec)
    forest = synth.random_forest(synth.rng(71), spec.radix, 3, 7, 25)     # 9,600 leaf values
    leaves = forest.leaves.copy()
    leaves.reshape(-1)[at] = value
    leaves.reshape(-1)[9599] = value
    _expect(m, lambda: m.ForestModel(sp, forest.feat, forest.thr, leaves), at, "leaf value")
    pred = np.full((sp.n_valid, 24), 0.5, np.float32)                     # 9,600 predictions
    pred.reshape(-1)[at] = value
    pred.reshape(-1)[9599] = value
    _expect(m, lambda: m.TableModel(sp, pred), at, "prediction")


@pytest.mark.parametrize("at", [0, 4096, -1])
def test_bad_parameter_is_named(at):
    m = cgs()
    spec = synth.Space([4, 5], [[1, 2, 3, 4], [1, 2, 3, 4, 5]])
    sp = m.Space.from_spec(spec)
    init = synth.mlp_init((72, 1), 2, 64, 3)
    params = [init.w[0], init.b[0], init.w[1], init.b[1], init.w[2], init.b[2]]
    flat = m.mlp_flatten(params)
    at %= len(flat)
    flat[at] = np.nan
    shapes = [p.shape for p in params]
    cut = np.cumsum([0] + [p.size for p in params])
    bad = [flat[cut[i]:cut[i + 1]].reshape(shapes[i]) for i in range(6)]
    _expect(m, lambda: m.MLPModel(sp, bad), at, "parameter")


def test_limits_of_the_range_pass_and_padding_is_zero():
    m = cgs()
    spec = synth.Space([3, 7], [[1, 2, 3], list(range(1, 8))])            # 21 valid, padded to 64
    sp = m.Space.from_spec(spec)
    pred = np.zeros((21, 5), np.float32)
    pred[0, 0], pred[20, 4], pred[3, 2] = 3.4e38, 1e-45, -0.0
    model = m.TableModel(sp, pred)
    assert (model.copy_predictions() == pred).all()
    sess = m.Session(sp)                                                  # scores past the end: none
    sess.search_step(model, 3, delta=[0.5] * 5)
    raw, valid = sess.sample_next(1 << 63)
    assert 0 <= valid < 21 and sess.step_info().n_unexplored == 20
