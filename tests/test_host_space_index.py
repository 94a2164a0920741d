"""The host's side of raw <-> valid indices: a list where few configurations
are valid, the validity mask where many are; what a space takes from the
driver.  On the runtime in host memory."""
import pytest

from tests import fake


@pytest.mark.parametrize("every", [1, 2, 31, 32, 33, 100, 5000, 1 << 30])
@pytest.mark.parametrize("radix", [(2,), (16, 16, 16, 5), (13, 11, 7, 3)])
def test_both_forms_agree_with_the_list(every, radix):
    fake.run(f"""
fake.fake_every({every})
fake.fake_clear()
sp = space(*{radix})
n = int(np.prod({radix}))
valid = list(range(0, n, {every}))
assert sp.n_valid == len(valid)
assert [i for i in range(n) if sp.valid_index(i) >= 0] == valid
assert [sp.valid_index(k) for k in valid] == list(range(len(valid)))
assert sp.valid_index(n) == sp.valid_index(1 << 40) == -1
pins = [int(e[2]) for e in log() if e[0] == "pin"]
words = -(-n // 32)
assert len(pins) == 1                              # one block: the shorter form and a draw's result
assert pins[0] <= 1.2 * 4 * min(len(valid), words + -(-n // 2048)) + 300, pins
assert len([e for e in log() if e[0] == "malloc"]) <= 5
f = forest(sp, 24)                                 # an index from the host's form to the device and back
s = m.Session(sp)
s.tuning_run(f, np.ones(sp.n_valid, np.float32), np.ones((sp.n_valid, 24)), U[:9], draws=1, max_tests=1)
""")
