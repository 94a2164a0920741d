"""Host memory that runs out inside an entry point is a status, not an
exception that ends the process.  On the runtime in host memory, whose host
allocations can fail too."""
import pytest

from tests import fake

CALLS = {
    "forest": "z = np.zeros((4, 1023), np.uint8)\ncall = lambda: m.ForestModel(sp, z, z, np.ones((4, 1024, 24), np.float32))",
    "poly": "pts, y = np.zeros(4096, np.uint32), np.ones((4096, 24), np.float32)\ncall = lambda: m.PolyModel(sp, pts, y, 2)",
    "batch": "call = lambda: m.Batch([s] * 200, [f] * 200)",
    "tune": "b = m.Batch([m.Session(sp) for _ in range(64)], [f] * 64)\n"
            "call = lambda: b.tuning_run(np.ones(768, np.float32), np.ones((768, 24)), U[:128].reshape(64, 2), draws=1,\n"
            "                            max_tests=1)",
    "search": "call = lambda: s.search_run(f, np.ones((100, 24)), [m.cgs_default_expert_params()] * 100, U[:101])",
    "near": "call = lambda: s.search_step_neighbourhood(f, 0, 3, delta=np.ones(24, np.float32))",
    "timed": "p = m.cgs_default_params(); p.timing = 1\ncall = lambda: m.Session(sp, p).close()",
    "read": "call = lambda: f.copy_predictions()",
}


@pytest.mark.parametrize("name", CALLS)
def test_a_lack_of_host_memory_is_a_status(name):
    fake.run(f"""
sp = space(16, 16, 3)
f = forest(sp, 24)
s = m.Session(sp)
{CALLS[name]}
assert status(call) == 0
m.cgs_release_memory()
used = fake.fake_used()
for limit in (1 << 11, 1 << 9, 64, 8):
    fake.fake_host_limit(limit)
    st = status(call)
    fake.fake_host_limit((1 << 64) - 1)
    assert st in (0, m.ENOMEM), st
    m.cgs_release_memory()
    assert fake.fake_used() <= used, limit     # nothing is left behind
assert st == m.ENOMEM
assert status(call) == 0
""")
