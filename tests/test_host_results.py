"""A draw's result counts only when that draw has published it: words that an
earlier draw, sampler call or batch left in the same place are not taken.  On
the runtime in host memory, whose draws can be kept from publishing."""
from tests import fake


def test_a_sampler_draw_that_does_not_publish_is_an_error():
    fake.run("""
sp = space(4, 4)
q = np.ones(100, np.uint32)
assert sp.sample_weights(q, U[:3]).tolist() == [0, 0, 0]
assert sp.sample_weights_noalloc(q, U[:3]).tolist() == [0, 0, 0]
fake.fake_publish(0)
assert status(lambda: sp.sample_weights(q, U[:1])) == m.EDEVICE
assert status(lambda: sp.sample_weights_noalloc(q, U[:1])) == m.EDEVICE
fake.fake_publish(1)
assert sp.sample_weights(q, U[:1]).tolist() == [0]
sp2 = space(4, 4)                              # on the block of a space that is gone
sp.close()
sp3 = space(4, 4)
fake.fake_publish(0)
for s in (sp2, sp3):
    assert status(lambda: s.sample_weights(q, U[:1])) == m.EDEVICE
""")


def test_a_batch_does_not_take_an_earlier_ones_results():
    fake.run("""
sp = space(16, 16, 3)
f = forest(sp, 24)
s = m.Session(sp)
one = lambda: m.Batch([s], [f], m.cgs_batch_schedule(4, 4, 0, 0))
b = one()
b.step([m.NO_PROFILE], None, U[:1])
b.close()
b = one()                                      # the same pinned block
fake.fake_publish(0)
assert status(lambda: b.step([m.NO_PROFILE], None, U[:1])) == m.EDEVICE
""")


def test_a_batch_draws_only_from_a_step_of_its_own():
    fake.run("""
sp = space(16, 16, 3)
f = forest(sp, 24)
s = m.Session(sp)
one = lambda: m.Batch([s], [f], m.cgs_batch_schedule(4, 4, 0, 0))
b = one()
assert status(lambda: b.draw(U[:1])) == m.ESTATE
for steps in (1, 2):                           # either accumulator set
    for _ in range(steps):
        b.step([m.NO_PROFILE], None, U[:1])
    b.draw(U[:1])
    b.close()
    b = one()                                  # the step was another batch's
    assert status(lambda: b.draw(U[:1])) == m.ESTATE
""")
