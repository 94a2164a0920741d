"""Whether a batch's runs of Alg. 1 are made on the device or with a launch per
iteration, on the runtime in host memory, where the draws of an iteration
decide."""
import pytest

from tests import fake


@pytest.mark.parametrize("radix,runs,draws,tests,device", [
    ((16, 16, 16, 8), 64, 33, 150, True), ((14, 14, 14, 9), 64, 33, 40, True), ((15, 10, 9, 5), 16, 33, 150, True),
    ((15, 10, 9, 5), 64, 5, 150, True), ((14, 14, 14, 9), 64, 1, 8, False), ((3, 4, 2, 5, 10), 1, 5, 40, False),
    ((16, 16, 16, 8), 16, 5, 150, False), ((3, 4, 2, 5, 10), 64, 1, 400, True), ((16, 16, 3), 2, 4, 1, False)])
def test_the_form_follows_the_work(radix, runs, draws, tests, device):
    fake.run(f"""
sp = space(*{radix})
f = forest(sp, 24)
b = m.Batch([m.Session(sp) for _ in range({runs})], [f] * {runs})
fake.fake_clear()
b.tuning_run(np.ones(sp.n_valid, np.float32), np.ones((sp.n_valid, 24)), U[:30 * {runs}].reshape({runs}, 30),
             draws={draws}, max_tests={tests}, stop_at_well=True)
assert {{k for e in log() if e[0] == "launch" for k in ("batch_tune", "batch_small") if k in e[2]}} == \\
    {{"batch_tune" if {device} else "batch_small"}}
""")
