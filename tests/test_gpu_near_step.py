"""Restricted steps in one launch (up to 8,192 neighbours) at the sizes where
its split changes, against the oracle: candidates, scores, weights and picks
bit-exact, with the first draw in the step's launch and after it."""
import pytest

import synth
from tests.test_gpu_neighbourhood import NbPair

pytestmark = pytest.mark.gpu


# neighbours (valid or not): 1; 30 (two radii's first edge); 1,023 and 1,330
# (16 to 8 threads a candidate); 2,196 (to 2); 7,824 (over 4,096 kept, so two
# weight blocks); 14,910 (separate launches)
@pytest.mark.parametrize("radix,radius,C", [
    ((2,), 1, 3), ((16, 16), 1, 7), ((16, 16, 4), 2, 33), ((11, 11, 11), 3, 64),
    ((13, 13, 13), 3, 20), ((13, 13, 13, 13), 3, 17), ((16, 16, 16, 16), 3, 5)])
def test_restricted_steps_at_split_edges(radix, radius, C):
    spec = synth.Space(list(radix), [list(range(1, r + 1)) for r in radix])
    g = synth.rng(63, *radix, radius)
    pair = NbPair(spec, synth.random_forest(g, spec.radix, 3, 6, C))
    U = synth.uniforms_u64(g, 10)
    deltas = synth.deltas(g, 4, C)
    deltas[1, ::2] = 0.0
    prof = pair.start(U[0])
    for i in range(3):                        # draws in the launch on even steps
        ref = pair.nb_step(prof, deltas[i], U[1 + 3 * i:4 + 3 * i], radius, check=i % 2 == 1)
        prof = next((p for p in ref.picks if p is not None), prof)
    pair.check_explored()
