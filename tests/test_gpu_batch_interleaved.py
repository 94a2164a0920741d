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


@pytest.mark.parametrize("radix", [(15, 13, 7, 3), (16, 16, 16, 16)])
def test_a_batch_step_after_a_restricted_step(radix):
    m = cgs()
    sp, model, sessions, alone = _spaces(m, radix, 2)
    batch = m.Batch(sessions, [model] * 2)
    g = synth.rng(122, *radix)
    U, D = synth.uniforms_u64(g, 12), synth.deltas(g, 4, C)
    raw, _, _ = batch.step([m.NO_PROFILE] * 2, None, U[:2])
    for i in range(2):
        alone[i].search_step(model, m.NO_PROFILE)
        assert alone[i].sample_next(int(U[i]))[0] == raw[i]
        for s in (sessions[i], alone[i]):
            s.search_step_neighbourhood(model, int(raw[i]), 1, delta=D[i])
        assert sessions[i].sample_next(int(U[2 + i])) == alone[i].sample_next(int(U[2 + i]))
    nxt, _, _ = batch.step([int(r) for r in raw], D[2:], U[4:6])
    for i in range(2):
        alone[i].search_step(model, int(raw[i]), delta=D[2 + i])
        assert alone[i].sample_next(int(U[4 + i]))[0] == nxt[i]
        assert (sessions[i].copy_scores() == alone[i].copy_scores()).all()
        assert (sessions[i].copy_weights() == alone[i].copy_weights()).all()
        assert sessions[i].sample_next(int(U[6 + i])) == alone[i].sample_next(int(U[6 + i]))
        assert (sessions[i].copy_explored() == alone[i].copy_explored()).all()
