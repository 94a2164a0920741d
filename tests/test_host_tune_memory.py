"""Batched runs of Alg. 1 where the device has no room for the buffers that
runs made on the device need: they are made with a launch per iteration, which
needs none.  On the runtime in host memory."""
from tests import fake


def test_without_room_the_runs_are_made_with_the_host():
    fake.run("""
sp = space(16, 16, 3)
f = forest(sp, 24)
sessions = [m.Session(sp) for _ in range(64)]
b = m.Batch(sessions, [f] * 64)
rt, ct = np.ones(sp.n_valid, np.float32), np.ones((sp.n_valid, 24))
def run():
    fake.fake_clear()
    r = b.tuning_run(rt, ct, U[:3200].reshape(64, 50), draws=1, max_tests=30, stop_at_well=True)
    kernels = {k for e in log() if e[0] == "launch" for k in ("batch_tune", "batch_small") if k in e[2]}
    return kernels, r
assert run()[0] == {"batch_tune"}
m.cgs_release_memory()
fake.fake_limit(100_000)                       # not the counters' 147 kB
kernels, r = run()
assert kernels == {"batch_small"}, kernels
assert all(t.tolist() == [0] and p.tolist() == [1] and w == 1 for t, p, w in r)
m.cgs_release_memory()
fake.fake_limit(1 << 30)
assert run()[0] == {"batch_tune"}
""")
