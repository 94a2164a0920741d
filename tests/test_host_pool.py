"""Memory kept between handles: given back on request and with the last
space.  On the runtime in host memory."""
from tests import fake


def test_what_is_kept_is_given_back():
    fake.run("""
sp = space(16, 16, 16, 16, 16)
f = forest(sp, 8)
m.cgs_release_memory()
live = fake.fake_used()
forest(sp, 64).close()
m.Session(sp).close()
assert fake.fake_used() > live + (1 << 28)
m.cgs_release_memory()
assert fake.fake_used() == live                # only what the open handles hold
f.close(); sp.close()
assert fake.fake_used() == 0
m.cgs_release_memory()                         # nothing is kept without a space
""")
