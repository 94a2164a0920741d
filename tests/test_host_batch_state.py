"""What a session is after its batch's step: as after a full step of its own,
also where its own last step was restricted.  On the runtime in host memory."""
import pytest

from tests import fake


@pytest.mark.parametrize("radix", ["(16, 16, 3)", "(16, 16, 16, 16)"])
@pytest.mark.parametrize("pending", [True, False])
def test_a_batch_step_ends_a_restricted_one(radix, pending):
    fake.run(f"""
sp = space(*{radix})
f = forest(sp, 24)
s = m.Session(sp)
b = m.Batch([s], [f], m.cgs_batch_schedule(4, 4, 0, 0))
s.search_step_neighbourhood(f, 0, 1, delta=np.full(24, 0.5, np.float32))
if not {pending}:
    s.sample_next(1)
b.step([m.NO_PROFILE], None, U[:1])
assert status(s.copy_scores) == 0 and status(s.copy_weights) == 0
fake.fake_clear()
s.sample_next(2)
drawn = [e[2] for e in log() if e[0] == "launch"]
assert len(drawn) == 1 and "draw_scores" in drawn[0], drawn
""")
