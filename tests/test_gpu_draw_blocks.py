"""Draws over more than 2,048 blocks, whose sums are loaded in pairs by runs
that start at even blocks: odd and even numbers of blocks, picks in the first,
the last and the later blocks of a run, against exact integers."""
import numpy as np
import pytest

import synth
from tests.helpers import cgs

pytestmark = pytest.mark.gpu


def _picks(q, U):
    q = q.astype(np.int64)
    out = []
    for u in U:
        c = np.cumsum(q)
        if c[-1] == 0:
            out.append(-1)
            continue
        out.append(int(np.searchsorted(c, (int(u) * int(c[-1])) >> 64, side="right")))
        q[out[-1]] = 0
    return out


@pytest.mark.parametrize("blocks,short", [(2048, 0), (2049, 0), (2049, 4095), (2303, 77), (4097, 1), (4608, 4000)])
def test_picks_equal_exact_integers(blocks, short):
    m = cgs()
    sp = m.Space([2], [[1, 2]])
    n = 4096 * blocks - short
    g = synth.rng(124, blocks, short)
    q = np.zeros(n, np.uint32)
    per = (blocks + 255) // 256
    at = [b for b in {0, 7, 8, 9, 23, 24, per - 1, per, per + 1, blocks // 2, blocks - 2, blocks - 1} if b < blocks]
    at = np.minimum(4096 * np.asarray(sorted(at)) + g.integers(0, 4096, len(at)), n - 1)
    q[at] = g.integers(1, 1 << 32, len(at))
    U = synth.uniforms_u64(g, len(at) + 2)
    assert sp.sample_weights(q, U).tolist() == _picks(q, U)     # until nothing is left
    q = g.integers(0, 1 << 24, n).astype(np.uint32)
    U = np.concatenate([synth.uniforms_u64(g, 3), np.array([0, (1 << 64) - 1], np.uint64)])
    assert sp.sample_weights(q, U).tolist() == _picks(q, U)
