"""Which evaluation a polynomial model takes, on the runtime in host memory:
nested where many terms meet many valid configurations of each tile, every
configuration by itself where not."""
import pytest

from tests import fake


@pytest.mark.parametrize("radix,order,C,nested", [
    ([4] * 9, 3, 24, True), ([4] * 10, 2, 24, True), ([4] * 10, 1, 24, False),
    ([8] * 7, 2, 24, True), ([8] * 7, 1, 24, False), ([16] * 5, 2, 64, False), ([16] * 5, 3, 8, True),
    ([3] * 12, 2, 64, True), ([2, 2] + [8] * 6, 2, 4, False), ([5] * 8, 3, 1, True),
    ([4] * 8, 3, 8, True), ([4] * 8, 2, 8, False), ([4] * 4, 2, 8, False), ([2, 2, 2, 4, 4], 2, 24, False)])
def test_the_form_follows_the_work(radix, order, C, nested):
    fake.run(f"""
sp = space(*{radix})
fake.fake_clear()
m.PolyModel(sp, np.arange(32, dtype=np.uint32), np.ones((32, {C}), np.float32), {order})
k = [e[2] for e in log() if e[0] == "launch" and "poly_eval" in e[2]]
assert ["nested" in x for x in k] == [{nested}], k
""")
