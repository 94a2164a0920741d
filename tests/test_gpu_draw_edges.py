"""Draws at the edges of their runs (16 weights, 4096-weight blocks, eight
block sums per load round of a 256-thread workgroup), bit-exact against the
oracle's draw rule with removal (Sect. 3.7, Alg. 1)."""
import numpy as np
import pytest

import synth
from oracle import sampling as S
from tests.helpers import cgs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [15, 16, 17, 4095, 4096, 4097, 256 * 4096 + 1, 8 * 256 * 4096 + 17])
def test_draws_with_removal_at_run_edges(n):
    m = cgs()
    sp = m.Space([2], [[0, 1]], [])
    g = np.random.default_rng(n)
    q = np.zeros(n, dtype=np.uint64)
    # few non-zero weights, in the first and last runs and blocks: the draws
    # exhaust them and every one is at an edge
    at = np.unique(np.clip(np.r_[0, 15, 16, n - 1, n - 16, n - 17, n // 2, n - 4096], 0, n - 1))
    q[at] = g.integers(1, 1 << 31, len(at), dtype=np.uint64)
    U = synth.uniforms_u64(synth.rng(84, n), len(at) + 2)
    U[:2] = [0, np.iinfo(np.uint64).max]
    got = sp.sample_weights(q.astype(np.uint32), U)
    left, ref = q.copy(), []
    for u in U:
        p = S.pick(left, int(u)) if left.sum() else None
        ref.append(-1 if p is None else int(p))
        if p is not None:
            left[p] = 0
    assert got.tolist() == ref
    assert sorted(got[:len(at)].tolist()) == at.tolist()
