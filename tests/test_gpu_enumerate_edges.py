"""Enumeration at the edges of its rows of 64, tiles of 2,048 and low-digit
tables (the last parameters up to 1,024 combinations, so that a row of 64 runs
over one or two values of the others), every constraint kind and the most
constraints, and the host's lookups raw -> valid: whole numbers, equal to the
oracle's."""
import numpy as np
import pytest

import synth
from oracle import space as SP
from tests.helpers import cgs

pytestmark = pytest.mark.gpu

KINDS = ("DIV", "DIV2", "PROD_LE", "PROD3_LE", "PROD_GE", "LE")
CASES = [
    # radix, constraints
    ([1], 0), ([7, 9], 1), ([16, 4], 1), ([5, 13], 1), ([16, 16, 8], 2), ([15, 15, 9], 2),
    ([2, 16, 16, 4], 3), ([3, 11, 16, 4], 3),  # a tile of 2,048; a tile and one row
    ([3, 15, 15, 5], 3),                 # low table 75: most rows run over two values
    ([11, 16, 4, 16], 2),                # low table 1,024 = 16 x 4 x 16
    ([13, 11, 13, 7], 4),                # low table 1,001
    ([2] * 17, 6),                       # parameters past the first 16
    ([1, 2] * 8 + [3, 1, 2, 5, 1, 3, 2, 2, 1, 1, 1, 1, 1, 1, 1, 2], 32),  # the most of both
    ([4, 5, 3, 6, 7, 2, 9], 8),
]


def _constraints(g, radix, vals, n):
    """n constraints over any parameters (repeats among them), each keeping
    a share of the configurations."""
    cons = []
    while len(cons) < n:
        kind = KINDS[int(g.integers(len(KINDS)))]
        a, b, c = (int(x) for x in g.integers(0, len(radix), 3))
        va, vb, vc = (np.asarray(vals[j], np.int64) for j in (a, b, c))
        bound = 0
        if kind in ("PROD_LE", "PROD_GE"):
            prod = np.sort(np.multiply.outer(va, vb).ravel())
            bound = int(prod[int((0.9 if kind == "PROD_LE" else 0.1) * (len(prod) - 1))])
        elif kind == "PROD3_LE":
            prod = np.sort(np.multiply.outer(np.multiply.outer(va, vb), vc).ravel())
            bound = int(prod[int(0.9 * (len(prod) - 1))])
        k = (kind, a, b, c, bound)
        kept = SP.valid_mask([radix[a], radix[b], radix[c]], [vals[a], vals[b], vals[c]],
                             [(kind, 0, 1, 2, bound)])
        if kind not in ("DIV", "DIV2", "LE") or kept.mean() >= 0.1 + 0.75 * (n > 8):
            cons.append(k)
    return cons


@pytest.mark.parametrize("case", range(len(CASES)))
def test_mask_list_and_lookups(case):
    m = cgs()
    radix, n_cons = CASES[case]
    g = synth.rng(93, case)
    vals = [np.sort(g.choice(np.arange(-2, 24), r, replace=False)).tolist() for r in radix]
    cons = _constraints(g, radix, vals, n_cons)
    sp = m.Space(list(radix), vals, cons)
    ref = SP.valid_mask(radix, vals, cons)
    valid = np.flatnonzero(ref)
    print(f"case {case}: {len(valid)} of {len(ref)} valid", flush=True)
    assert sp.n_raw == len(ref) and sp.n_valid == len(valid)
    assert (sp.copy_mask() == SP.mask_words(ref)).all()
    assert (sp.copy_valid() == valid).all()
    want = np.where(ref, np.cumsum(ref) - 1, -1)
    ks = np.arange(len(ref))
    if len(ks) > 6000:
        ks = np.unique(np.concatenate([g.integers(0, len(ref), 5000), [0, 31, 32, 2047, 2048, 4095,
                                                                       4096, len(ref) - 1]]))
    for k in ks:
        assert sp.valid_index(int(k)) == want[k], k
