"""Forests on both sides of every number of trees that the byte-node walk is
built for, and of the counters that decide beyond 32 trees, against the oracle."""
import types

import numpy as np
import pytest

import synth
from tests.helpers import cgs
from tests.test_gpu_forest import _check_full

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 2, 3, 16, 17, 23, 24, 25, 32, 33, 40, 41, 48, 49, 56, 57, 63, 64])
@pytest.mark.parametrize("D,C", [(3, 8), (8, 5), (6, 24), (4, 2)])
def test_equal_to_the_oracle(T, D, C):
    cgs()
    radix = [6, 7, 4, 5]                  # 840 configurations: less than a tile of 512 threads in the second
    g = synth.rng(123, T, D, C)
    spec = synth.Space(radix, [list(range(1, r + 1)) for r in radix], [])
    feat = g.integers(0, 4, (T, (1 << D) - 1)).astype(np.uint8)
    thr = (g.integers(0, 16, feat.shape) % (np.asarray(radix)[feat] - 1)).astype(np.uint8)
    leaves = g.random((T, 1 << D, C)).astype(np.float32)
    _check_full(spec, types.SimpleNamespace(feat=feat, thr=thr, leaves=leaves, depth=D, n_trees=T, n_counters=C))
