"""Predictions of the nested evaluation of polynomial models: the inner
parameters at the end of a space, tiles of 32 outer combinations ordered by
subspace, inner monomials filled up to eights, and the blocked factorisation
of the normal equations (panels of 16 terms).

The predictions are compared with the float64 polynomial of the device's own
coefficients, so only the float32 evaluation is left: each of the T terms is a
product of at most 4 rounded features times a rounded coefficient, summed in
at most T + 8 steps, hence 2 (T + 8) 2^-24 sum_t |F_t beta_t|."""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import lsq as LS
from oracle import space as SP
from tests.helpers import cgs

pytestmark = pytest.mark.gpu

CASES = [
    # radix, constraints, order, counters
    ([3, 5, 2, 7, 2, 3, 5], 0, 2, 7),           # 420 outer combinations (13 tiles and 4), r_in 15
    ([3, 2, 5, 2, 2, 2, 2, 2, 2, 4, 4], 0, 2, 24),  # binary parameters last: up to 32 groups a tile
    ([5, 3, 2, 4, 3, 2, 5, 4, 3], 4, 3, 24),    # r_in 60, sparse and empty tiles
    ([2, 3, 2, 16, 8], 0, 4, 64),               # r_in 128, 12 outer combinations, 64 counters
    ([2, 3, 2, 16, 9], 0, 1, 1),                # only the last parameter fits: r_in 9
    ([4, 4, 4], 0, 0, 33),                      # constant term; one monomial
    ([4, 4, 4], 0, 4, 48),                      # 35 terms
    ([3, 5, 2, 4, 2], 0, 2, 5),                 # ends in a binary parameter: not nested
    ([4, 3, 5, 2, 7], 0, 2, 9),                 # r_in 7: not nested
    ([5, 3, 4, 3, 3, 4, 2, 8], 2, 3, 16),       # 120 terms, panels 7 and a half
    ([3] * 7 + [4, 2, 12], 3, 2, 12),           # 55 terms over 9 parameters, r_in 12
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_predictions_equal_the_polynomial(case):
    m = cgs()
    radix, n_cons, order, C = CASES[case]
    vals = synth.value_tables(radix, binary_radix2=True)
    cons = synth.random_constraints(synth.rng(91, case), vals, n_cons,
                                    ("DIV", "PROD_LE", "PROD_GE", "LE"), loose=0.4) if n_cons else []
    spec = synth.Space(list(radix), vals, cons)
    valid = SP.enumerate_valid(spec.radix, spec.values, spec.constraints)
    digits = SP.digits_of(valid, spec.radix)
    g = synth.rng(92, case)
    pts = g.integers(0, len(valid), min(6000, 4 * len(valid))).astype(np.uint32)
    Y = synth.measured_counters(g, digits[pts], spec.radix, C)
    print(f"case {case}: {len(valid)} valid", flush=True)
    sp = m.Space.from_spec(spec)
    model = m.PolyModel(sp, pts, Y, order)
    assert sp.n_valid == len(valid) and model.report["pivot_clamped"] == 0
    ref = LS.fit(spec.values, spec.radix, digits[pts], Y, order)
    beta = model.coefficients()
    # the normal equations, to the bound of a backward stable solve
    F = LS.basis(LS.features(spec.values, spec.radix, digits[pts]), order)
    s_pts = LS.subspace(spec.radix, digits[pts])
    for k in np.unique(s_pts):
        Fk = F[s_pts == k]
        A = Fk.T @ Fk + ref.lam[k] * np.eye(Fk.shape[1])
        R = Fk.T @ np.asarray(Y, np.float64)[s_pts == k]
        res = np.abs(A @ beta[k] - R)
        assert (res <= 1e-10 * (np.abs(A) @ np.abs(beta[k]) + np.abs(R)) + 1e-300).all(), k
    own = dataclasses.replace(ref, beta=beta)
    rows = np.arange(len(valid))
    if len(rows) > 60000:
        rows = np.sort(g.choice(len(valid), 60000, replace=False))
    got = model.copy_predictions()[rows].astype(np.float64)
    want = LS.predict(own, spec.values, spec.radix, digits[rows])
    mag = LS.abs_terms(own, spec.values, spec.radix, digits[rows])
    assert (np.abs(got - want) <= 2 * (len(ref.terms) + 8) * 2.0 ** -24 * mag).all()
