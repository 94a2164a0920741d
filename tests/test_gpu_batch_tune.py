"""Runs of Alg. 1 in a batch on a small space, all iterations on the device:
each equals the run of a session of its own (which the oracle tests pin), in
its tests, its explored configurations and the steps and draws that follow;
spaces that are used up, one to 33 draws, runs that end at a good
configuration, and the two errors a run can end with."""
import numpy as np
import pytest

import synth
from oracle import space as SP
from tests.helpers import cgs

pytestmark = pytest.mark.gpu

RUNS = 64


def _setup(m, radix, key):
    spec = synth.Space(list(radix), [list(range(1, r + 1)) for r in radix])
    valid = SP.enumerate_valid(spec.radix, spec.values, spec.constraints)
    table = synth.kernel_table(synth.rng(96, key), SP.digits_of(valid, spec.radix), spec.radix)
    sp = m.Space.from_spec(spec)
    return sp, table, m.TableModel(sp, table.counters.astype(np.float32))


def _ep(m):
    return m.cgs_expert_params(inst_reaction=0.7, volta=0, reserved=0, cores=1.0, threads=1e9)


@pytest.mark.parametrize("radix,draws,tests,stop", [((3, 2), 2, 100, False), ((3, 4, 2, 5), 1, 400, False),
                                                    ((15, 13, 7, 3), 33, 150, False),
                                                    ((15, 13, 7, 3), 5, 200, True),
                                                    ((16, 16, 16), 4, 41, False),
                                                    ((16, 16, 16, 8), 5, 60, False)])
def test_runs_equal_single_ones(radix, draws, tests, stop):
    m = cgs()
    sp, table, model = _setup(m, radix, 1)
    U = np.stack([synth.uniforms_u64(synth.rng(97, i), 600) for i in range(RUNS)])
    kw = dict(draws=draws, max_tests=tests, stop_at_well=stop, expert=_ep(m))
    sessions = [m.Session(sp) for _ in range(RUNS)]
    batch = m.Batch(sessions, [model] * RUNS)
    print(f"{radix} draws {draws} tests {tests}", flush=True)
    got = batch.tuning_run(table.runtime, table.counters, U, **kw)
    lengths = set()
    for i in range(0, RUNS, 9):
        one = m.Session(sp)
        ref = one.tuning_run(model, table.runtime, table.counters, U[i], **kw)
        assert got[i][0].tolist() == ref[0].tolist() and got[i][1].tolist() == ref[1].tolist()
        assert got[i][2] == ref[2]
        lengths.add(len(ref[0]))
        assert (sessions[i].copy_explored() == one.copy_explored()).all()
        if sp.n_valid > 2 * tests:
            raw = int(sp.copy_valid(int(ref[0][-1]), 1)[0])
            delta = synth.deltas(synth.rng(98, i), 1, 24)[0]
            for s in (sessions[i], one):
                s.search_step(model, raw, delta=delta)
            assert sessions[i].sample_next(int(U[i, -1])) == one.sample_next(int(U[i, -1]))
    if stop:
        assert len(lengths) > 1


def test_draws_go_on_from_the_last_steps():
    m = cgs()
    sp, table, model = _setup(m, (15, 13, 7, 3), 1)
    U = np.stack([synth.uniforms_u64(synth.rng(97, i), 200) for i in range(RUNS)])
    batch = m.Batch([m.Session(sp) for _ in range(RUNS)], [model] * RUNS)
    got = batch.tuning_run(table.runtime, table.counters, U, draws=3, max_tests=40,
                           stop_at_well=False, expert=_ep(m))
    _, valid, status = batch.draw(U[:, -1])
    assert (status == 0).all()
    for i in range(RUNS):
        assert valid[i] not in set(got[i][0].tolist())


def test_a_run_that_cannot_go_on_names_itself():
    m = cgs()
    sp, table, model = _setup(m, (15, 13, 7, 3), 2)
    U = np.stack([synth.uniforms_u64(synth.rng(97, i), 30) for i in range(RUNS)])
    kw = dict(draws=4, stop_at_well=False, expert=_ep(m))

    def fails(counters, u, tests):
        batch = m.Batch([m.Session(sp) for _ in range(RUNS)], [model] * RUNS)
        with pytest.raises(m.CgsError) as ei:
            batch.tuning_run(table.runtime, counters, u, max_tests=tests, **kw)
        return ei.value

    e = fails(table.counters, U, 200)        # 30 numbers: the first, and 7 iterations' and one
    assert e.status == m.ERANGE and "run 0 needs more than 30" in str(e)
    batch = m.Batch([m.Session(sp) for _ in range(RUNS)], [model] * RUNS)
    good = batch.tuning_run(table.runtime, table.counters, U, max_tests=26, **kw)
    # one configuration's counters become unusable: the run that profiles it
    # first, and of those the first, is named
    bad = int(good[40][0][np.flatnonzero(good[40][1])[1]])
    first = min((int(np.flatnonzero(t[p == 1] == bad)[0]), i) for i, (t, p, _) in enumerate(good)
                if (t[p == 1] == bad).any())[1]
    counters = table.counters.copy()
    counters[bad, 3] = np.nan
    e = fails(counters, U, 26)
    assert e.status == m.EINVAL and f"run {first}: expert system rejected" in str(e)
