"""What a small polynomial fit asks of the device before its points can be
sorted by subspace: nothing where there is one subspace, one launch and a wait
(no copy) where there are several.  On the runtime in host memory."""
import pytest

from tests import fake


@pytest.mark.parametrize("radix,several", [([3, 4, 5], False), ([4] * 5, False), ([2, 2, 2, 4, 4], True)])
def test_the_points_need_no_copy(radix, several):
    fake.run(f"""
sp = space(*{radix})
pts, y = np.arange(40, dtype=np.uint32), np.ones((40, 24), np.float32)
m.PolyModel(sp, pts, y, 2).close()
fake.fake_clear()
m.PolyModel(sp, pts, y, 2).close()
l = log()
fit = next(i for i, e in enumerate(l) if e[0] == "launch" and "poly_features" in e[2])
sort = [i for i, e in enumerate(l[:fit]) if e[0] == "launch" and "poly_subspaces" in e[2]]
waits = [i for i, e in enumerate(l[:fit]) if e[0] == "wait"]
assert len(sort) == len(waits) == {int(several)}, l[:fit]
if sort:
    assert l[sort[0] + 1][0] == "wait", l[:fit]
""")
