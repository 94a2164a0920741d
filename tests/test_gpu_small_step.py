"""Steps of small spaces (one launch up to 32,768 configurations) at the
edges of their tiles, runs and blocks against the oracle: scores, weights,
totals and picks bit-exact, with draws made in the step's launch, draws made
after it from the block sums it leaves, and steps read before any draw."""
import numpy as np
import pytest

import synth
from oracle import search as SR
from oracle import space as SP
from oracle import tuning as TU
from tests.helpers import bits_to_bool, cgs
from tests.test_gpu_step import Pair

pytestmark = pytest.mark.gpu

# 1, one workgroup and around it, a block of 4,096 and around it, runs that
# do not divide a block, the last size of the single launch and the next
RADICES = [(1,), (3, 2), (8, 8, 8), (15, 7, 5), (15, 13, 7, 3), (16, 16, 16), (14, 14, 7, 3),
           (15, 14, 13, 12), (16, 16, 16, 8), (13, 11, 11, 7, 3)]


@pytest.mark.parametrize("radix", RADICES, ids=lambda r: str(int(np.prod(r))))
def test_steps_equal_the_oracle(radix):
    spec = synth.Space(list(radix), [list(range(1, r + 1)) for r in radix])
    g = synth.rng(60, *radix)
    C = 20                                    # more counters than one round of loads
    if max(radix) == 1:
        forest = synth.Forest(1, 0, C, np.zeros((1, 0), np.uint8), np.zeros((1, 0), np.uint8),
                              g.random((1, 1, C), dtype=np.float32))
    else:
        forest = synth.random_forest(g, spec.radix, 3, 6, C)
    pair = Pair(spec, forest)
    U = synth.uniforms_u64(g, 16)
    U[3], U[4] = 0, np.iinfo(np.uint64).max
    deltas = synth.deltas(g, 4, C)
    ref, _ = pair.step(None, np.zeros(C, np.float32), U[:1], check_scores=False)
    prof = ref.picks[0]
    for i in range(4):                        # first draw in the launch on even steps
        ref, info = pair.step(prof, deltas[i], U[1 + 3 * i:4 + 3 * i], check_scores=i % 2 == 1)
        if ref.picks and ref.picks[0] is not None:
            prof = ref.picks[0]
    ex = bits_to_bool(pair.sess.copy_explored(), len(pair.prep.valid))
    assert (ex == pair.explored).all()


@pytest.mark.parametrize("radix,draws", [((16, 16, 16), 33), ((15, 14, 13, 12), 7),
                                         ((13, 11, 11, 7, 3), 4)])
def test_draw_series_equal_the_oracle(radix, draws):
    m = cgs()
    spec = synth.Space(list(radix), [list(range(1, r + 1)) for r in radix])
    valid = SP.enumerate_valid(spec.radix, spec.values, spec.constraints)
    digits = SP.digits_of(valid, spec.radix)
    table = synth.kernel_table(synth.rng(61, *radix), digits, spec.radix)
    P = table.counters
    prep = SR.Prepared(valid, digits, None, P, P.astype(np.float32))
    sp = m.Space.from_spec(spec)
    model = m.TableModel(sp, P.astype(np.float32))
    U = synth.uniforms_u64(synth.rng(62, *radix), 200)
    ep = m.cgs_expert_params(inst_reaction=0.7, volta=0, reserved=0, cores=1.0, threads=1e9)
    n = 3 * (draws + 1) + 2
    got = m.Session(sp).tuning_run(model, table.runtime, P, U, draws=draws, max_tests=n,
                                   stop_at_well=False, expert=ep)
    ref = TU.run(prep, table.runtime, P, U, draws=draws, max_tests=n, stop_at_well=False,
                 cores=1.0, threads=1e9)
    assert got[0].tolist() == ref.tested and got[1].tolist() == ref.profiled


# one workgroup a session (more sessions than workgroups, a space of one
# tile), several, and one per tile
@pytest.mark.parametrize("radix,runs,draws", [((15, 7, 5), 3, 2), ((15, 13, 7, 3), 130, 5),
                                              ((15, 14, 13, 12), 9, 5), ((16, 16, 16), 1, 33)])
def test_batched_runs_equal_the_oracle(radix, runs, draws):
    m = cgs()
    spec = synth.Space(list(radix), [list(range(1, r + 1)) for r in radix])
    valid = SP.enumerate_valid(spec.radix, spec.values, spec.constraints)
    digits = SP.digits_of(valid, spec.radix)
    table = synth.kernel_table(synth.rng(64, *radix), digits, spec.radix)
    P = table.counters
    prep = SR.Prepared(valid, digits, None, P, P.astype(np.float32))
    sp = m.Space.from_spec(spec)
    model = m.TableModel(sp, P.astype(np.float32))
    sessions = [m.Session(sp) for _ in range(runs)]
    U = np.stack([synth.uniforms_u64(synth.rng(65, i), 200) for i in range(runs)])
    ep = m.cgs_expert_params(inst_reaction=0.7, volta=0, reserved=0, cores=1.0, threads=1e9)
    n = 2 * (draws + 1) + 2
    batch = m.Batch(sessions, [model] * runs)
    got = batch.tuning_run(table.runtime, P, U, draws=draws, max_tests=n, stop_at_well=False,
                           expert=ep)
    for i in sorted({0, runs // 2, runs - 1}):
        ref = TU.run(prep, table.runtime, P, U[i], draws=draws, max_tests=n, stop_at_well=False,
                     cores=1.0, threads=1e9)
        assert got[i][0].tolist() == ref.tested and got[i][1].tolist() == ref.profiled
    # the sessions go on from the batch's last step, one draw each
    more = batch.draw(U[:, -1])
    assert (more[2] == 0).all()
    for i in range(runs):
        assert more[1][i] not in set(got[i][0].tolist())
