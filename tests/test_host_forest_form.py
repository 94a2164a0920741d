"""Which evaluation a forest takes, at the edges of the rule, on the runtime in
host memory: byte nodes with 24, 32, 40, 48 or 64 trees walked, or nodes as
(feature, threshold) where bytes do not pay."""
import pytest

from tests import fake

BYTES, WIDE, GENERAL = "forest_eval_residentILi{}ELb1E", "forest_eval_residentILi{}ELb0E", "11forest_evalE"


@pytest.mark.parametrize("T,D,C,kernel", [
    (1, 3, 24, WIDE.format(1)), (1, 4, 24, BYTES.format(1)),
    (2, 7, 8, WIDE.format(2)), (2, 8, 8, BYTES.format(2)), (2, 8, 9, WIDE.format(2)),
    (3, 1, 64, BYTES.format(4)), (16, 6, 64, BYTES.format(16)), (17, 6, 24, BYTES.format(24)),
    (24, 6, 24, BYTES.format(24)), (25, 6, 64, BYTES.format(32)), (32, 6, 5, BYTES.format(32)),
    (33, 6, 8, BYTES.format(40)), (33, 6, 2, BYTES.format(40)), (33, 6, 5, GENERAL), (33, 6, 24, GENERAL),
    (41, 6, 4, BYTES.format(48)), (48, 6, 12, GENERAL), (49, 6, 1, BYTES.format(64)), (56, 6, 24, GENERAL),
    (57, 6, 24, BYTES.format(64)), (57, 6, 28, GENERAL), (64, 6, 6, BYTES.format(64)), (64, 2, 64, GENERAL)])
def test_the_form_follows_the_work(T, D, C, kernel):
    fake.run(f"""
sp = space(8, 8, 8)
z = np.zeros(({T}, {(1 << D) - 1}), np.uint8)
fake.fake_clear()
m.ForestModel(sp, z, z, np.ones(({T}, {1 << D}, {C}), np.float32))
assert [{kernel!r} in e[2] for e in log() if e[0] == "launch" and "forest" in e[2]] == [True], log()
""")
