"""Forests at the edges of the byte-per-node evaluation: as many tests
(parameter, threshold) as a 64-bit word holds and one more, more trees than
the wider nodes keep in LDS, the deepest forests that fit and do not fit,
thresholds no digit exceeds, and parameters past the first 16.  Leaf ids are
whole numbers and the predictions are sums in tree order: equal to the
oracle's."""
import types

import numpy as np
import pytest

import synth
from tests.helpers import cgs
from tests.test_gpu_forest import _check_full

pytestmark = pytest.mark.gpu

CASES = [
    # radix, trees, depth, counters
    ([16, 16, 16, 16, 4], 3, 7, 8),     # 63 tests
    ([16, 16, 16, 16, 5], 3, 7, 8),     # 64 tests: nodes stay (feature, threshold)
    ([16, 16, 16, 16, 5], 17, 5, 4),    # the same with more trees than those keep in LDS
    ([2] * 18, 2, 9, 5),                # parameters past the first 16
    ([1, 7, 1, 3, 5, 1, 8], 17, 6, 12),
    ([6, 7, 4, 9], 33, 8, 24),
    ([6, 7, 4, 9], 64, 11, 4),          # 128 KB of nodes
    ([6, 7, 4, 9], 9, 14, 4),           # 144 KB
    ([6, 7, 4, 9], 10, 14, 4),          # 160 KB: does not fit
    ([6, 7, 4, 9], 16, 1, 7),
    ([6, 7, 4, 9], 5, 0, 4),            # a leaf each
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_equal_to_the_oracle(case):
    cgs()
    radix, T, D, C = CASES[case]
    g = synth.rng(94, case)
    vals = [list(range(1, r + 1)) for r in radix]
    spec = synth.Space(list(radix), vals, [])
    n_int = (1 << D) - 1
    feat = g.integers(0, len(radix), (T, n_int)).astype(np.uint8)
    thr = g.integers(0, 17, (T, n_int)).astype(np.uint8)
    exact = g.random((T, n_int)) < 0.8   # most thresholds split, the others do not
    thr = np.where(exact, thr % np.maximum(np.asarray(radix)[feat] - 1, 1), thr).astype(np.uint8)
    if n_int:
        thr[0, 0] = 255
    leaves = g.random((T, 1 << D, C)).astype(np.float32)
    _check_full(spec, types.SimpleNamespace(feat=feat, thr=thr, leaves=leaves, depth=D,
                                            n_trees=T, n_counters=C))
