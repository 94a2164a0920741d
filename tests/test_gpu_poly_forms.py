"""Polynomials whose evaluation is nested by its rule: short tiles and runs,
several subspaces a tile, constrained spaces, 128 inner combinations and one to
64 counters; and the other form beside them.  The check is that of the nested
evaluation's own tests."""
import pytest

from tests import test_gpu_poly_nested as base

pytestmark = pytest.mark.gpu

CASES = [
    # radix, constraints, order, counters
    ([5, 3, 4, 3, 5, 4, 2, 8], 0, 4, 16),          # r_in 8, 106 terms
    ([5, 3, 4, 3, 5, 2, 4, 8], 0, 3, 7),
    ([5, 3, 4, 3, 5, 2, 4, 8], 2, 3, 24),          # every configuration by itself
    ([2, 3, 2, 4, 2, 5, 2, 3, 4, 4, 3], 0, 4, 12), # 16 subspaces, up to 16 groups a tile
    ([4, 3, 5, 4, 3, 5, 4, 16, 8], 3, 2, 24),      # r_in 128, tiles partly valid
    ([4, 3, 5, 4, 3, 5, 4, 16, 8], 0, 3, 64),      # 139 terms, one column of the products a wave
    ([4] * 9, 0, 3, 33),
    ([3] * 7 + [4, 5, 9], 0, 2, 1),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_predictions_equal_the_polynomial(case, monkeypatch):
    monkeypatch.setattr(base, "CASES", CASES)
    base.test_predictions_equal_the_polynomial(case)
