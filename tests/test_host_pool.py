"""Memory kept between handles: bounded, the longest unused goes first, and
given back on request and with the last space.  On the runtime in host
memory."""
from tests import fake


def test_blocks_nobody_asks_for_make_room():
    fake.run("""
sp = space(16, 16, 16, 16, 16)                 # 2^20 configurations: 4 MiB a counter
def use(C):
    fake.fake_clear()
    forest(sp, C).close()
    return [int(e[2]) for e in log() if e[0] == "malloc" and int(e[2]) >= 1 << 22]
base = fake.fake_used()
for C in (64, 63, 62, 61):                     # 1,000 MiB, each size used once
    assert use(C)
for C in (20, 21, 40):                         # each does not fit beside what is kept
    assert use(C)
    for _ in range(3):
        assert use(C) == []                    # but is kept now
    assert fake.fake_used() - base <= 1 << 30
for _ in range(2):
    for C in (20, 21, 40):
        assert use(C) == []                    # all three are
assert use(64)                                 # and what made room is gone
big = space(16, 16, 16, 16, 16, 16)
for _ in range(2):
    fake.fake_clear()
    forest(big, 24).close()                    # 1.5 GiB: larger than what may be kept
    assert fake.fake_used() - base <= (1 << 30) + (1 << 28)
    assert [int(e[2]) for e in log() if e[0] == "malloc" and int(e[2]) > 1 << 30]
assert use(40) == []                           # and makes nothing go
""")


def test_pinned_blocks_make_room():
    fake.run("""
keep = space(4)
def use(*radix):                               # the space's mask is pinned: n_raw / 8 bytes
    fake.fake_clear()
    space(*radix).close()
    return [int(e[2]) for e in log() if e[0] == "pin" and int(e[2]) >= 1 << 20]
assert use(*(16,) * 6, 6) and use(*(16,) * 6, 2) # 12 and 4 MiB: all that may be kept
assert use(*(16,) * 6, 3)                      # 6 MiB: the 12 go
for _ in range(3):
    assert use(*(16,) * 6, 3) == [] and use(*(16,) * 6, 2) == []
""")


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
