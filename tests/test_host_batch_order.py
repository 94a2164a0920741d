"""A batch runs on a stream of its own.  What its sessions enqueued on their
space's stream (a draw returns when its result is published, not when its
kernel has ended) is waited for before the batch touches the sessions' arrays.
On the runtime in host memory: the order of launches and waits."""
import pytest

from tests import fake

SETUP = """
def kinds(l):
    return [e[0] + (" " + e[2] if len(e) > 2 else "") for e in l]

def ordered(call, own, what):
    # own launches on the space's stream, then the batch's `what` after a wait for that stream
    fake.fake_clear()
    own()
    call()
    l = log()
    first = next(i for i, e in enumerate(l) if e[0] == "launch" and what in e[2])
    mine = [i for i, e in enumerate(l[:first]) if e[0] == "launch" and e[1] != l[first][1]]
    assert mine, l
    stream = l[mine[-1]][1]
    copies = [i for i, e in enumerate(l) if e[0] == "copy" and e[1] == l[first][1]]
    start = min([first] + [i for i in copies if i > mine[-1]])
    assert ["wait", stream] in l[mine[-1]:start], kinds(l)

sp = space(*RADIX)
f = forest(sp, 24)
sessions = [m.Session(sp) for _ in range(3)]
b = m.Batch(sessions, [f] * 3, m.cgs_batch_schedule(4, 4, 0, 0))
b.step([m.NO_PROFILE] * 3, None, U[:3])
step = lambda: b.step([m.NO_PROFILE] * 3, None, U[:3])
draw = lambda: sessions[1].sample_next(7)
restricted = lambda: (sessions[2].search_step_neighbourhood(f, 0, 1, delta=np.full(24, 0.5, np.float32)),
                      sessions[2].sample_next(8))
"""

TUNE = """
rt, ct = np.ones(sp.n_valid, np.float32), np.ones((sp.n_valid, 24))
def tune(batch, n, tests):
    batch.tuning_run(rt, ct, U[:30 * n].reshape(n, 30), draws=1, max_tests=tests, stop_at_well=True)
"""


@pytest.mark.parametrize("radix", ["(16, 16, 3)", "(16, 16, 16, 16)"])
@pytest.mark.parametrize("script", [
    "ordered(step, draw, 'batch_score')",
    "ordered(lambda: b.draw(U[:3]), draw, 'batch_draw')",
    "ordered(step, restricted, 'batch_score')",
    "ordered(b.autotune, draw, 'batch_score')",
    TUNE + "ordered(lambda: tune(b, 3, 1), draw, 'batch_s')",    # batch_small, or batch_score on the large space
    TUNE + "b = m.Batch([sessions[1]] + [m.Session(sp) for _ in range(63)], [f] * 64)\n"
           "ordered(lambda: tune(b, 64, 30), draw, 'batch_tune' if sp.n_valid <= 32768 else 'graph')",
], ids=["step", "draw", "restricted", "autotune", "tuning", "tuning-64"])
def test_the_batch_waits_for_its_sessions_own_work(radix, script):
    fake.run(SETUP.replace("RADIX", radix) + script)
