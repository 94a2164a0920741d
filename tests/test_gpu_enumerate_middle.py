"""Enumeration where the low-digit table is short, so that the middle digits
come from their own: rows of 64 that run over the end of either table or of
both.  The check is that of the other edges."""
import pytest

from tests import test_gpu_enumerate_edges as base

pytestmark = pytest.mark.gpu

CASES = [
    # radix, constraints
    ([3, 16, 16, 13, 5], 2),          # 65 x 256, three values above them
    ([5, 7, 15, 15, 5], 1),           # 75 x 225
    ([2, 9, 16, 13, 5], 3),           # 65 x 144: the next radix does not fit
    ([4, 2, 16, 11, 6], 2),           # 66 x 128: nothing above them
    ([16, 16, 16, 8], 2),             # 128 x 256, two values above them
    ([7, 3, 1, 16, 1, 13, 1, 5, 1], 4),
    ([3, 2, 2, 2, 2, 2, 2, 2, 2, 16, 13, 5], 2),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_mask_list_and_lookups(case, monkeypatch):
    monkeypatch.setattr(base, "CASES", CASES)
    base.test_mask_list_and_lookups(case)
