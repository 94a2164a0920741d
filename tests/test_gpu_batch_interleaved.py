"""Draws from a batch's sessions between its steps and draws, on small and
large spaces: every session gives the picks, scores and explored
configurations of one that makes the same steps and draws by itself."""
import numpy as np
import pytest

import synth
from tests.helpers import cgs

pytestmark = pytest.mark.gpu

C = 24


def _spaces(m, radix, n):
    spec = synth.Space(list(radix), [list(range(1, r + 1)) for r in radix])
    sp = m.Space.from_spec(spec)
    model = m.ForestModel.from_spec(sp, synth.random_forest(synth.rng(120, *radix), spec.radix, 3, 6, C))
    return sp, model, [m.Session(sp) for _ in range(n)], [m.Session(sp) for _ in range(n)]


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("radix,n", [((15, 13, 7, 3), 5), ((16, 16, 16, 16), 3), ((16, 16, 16, 16, 16, 4), 2)])
def test_draws_between_batch_steps(radix, n, graph):
    m = cgs()
    sp, model, sessions, alone = _spaces(m, radix, n)
    batch = m.Batch(sessions, [model] * n, m.cgs_batch_schedule(512, 256, graph, 0))
    g = synth.rng(121, *radix)
    U = synth.uniforms_u64(g, 40 * n).reshape(40, n)
    D = synth.deltas(g, 8 * n, C).reshape(8, n, C)
    prof = [m.NO_PROFILE] * n
    for step in range(8):
        u = iter(U[5 * step:])
        first = next(u)
        raw, _, status = batch.step(prof, D[step] if step else None, first)
        assert (status == 0).all()
        for i in range(n):
            alone[i].search_step(model, prof[i], delta=D[step][i] if step else None)
            assert alone[i].sample_next(int(first[i]))[0] == raw[i], (step, i)
        own, drawn = next(u), next(u)
        for i in range(n):                    # the last thing enqueued before the batch goes on
            if step % 2:
                assert sessions[i].sample_next(int(own[i])) == alone[i].sample_next(int(own[i])), (step, i)
        raw2, _, status = batch.draw(drawn)
        assert (status == 0).all()
        for i in range(n):
            assert alone[i].sample_next(int(drawn[i]))[0] == raw2[i], (step, i)
        own = next(u)
        for i in range(n):
            assert sessions[i].sample_next(int(own[i])) == alone[i].sample_next(int(own[i])), (step, i)
        prof = [int(r) for r in raw]
    for a, b in zip(sessions, alone):
        assert (a.copy_explored() == b.copy_explored()).all()
        assert (a.copy_scores() == b.copy_scores()).all() and (a.copy_weights() == b.copy_weights()).all()
