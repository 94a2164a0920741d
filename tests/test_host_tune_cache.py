"""The batch autotuner's cache: an entry is for the kernels that it was timed
with.  On the runtime in host memory."""
import pytest

from tests import fake


@pytest.mark.parametrize("old", [False, True])
def test_entries_name_the_kernels_they_were_timed_with(tmp_path, old):
    fake.run(f"""
path = {str(tmp_path / "cache.txt")!r}
sp = space(16, 16, 16, 16, 4)
shared = forest(sp, 64)                             # 67 MB of predictions
models = [forest(sp, 64) for _ in range(9)]
sessions = [m.Session(sp) for _ in range(9)]
one = m.Batch(sessions, [shared] * 9)               # read from the caches
each = m.Batch(sessions, models)                    # 604 MB: streamed
def kernels(b):
    fake.fake_clear()
    b.autotune(path)
    b.set_schedule(m.cgs_batch_schedule(8, 8, 0, 0))
    b.step([m.NO_PROFILE] * 9, None, U[:9])
    return [e[2] for e in log() if e[0] == "launch" and "batch_score" in e[2]]
if {old}:                                           # an entry as it was before the streamed kernel
    open(path, "w").write(f"gfx950 n=9 tiles={{9 * 256}} blocks={{9 * 64}} counters={{9 * 64}} -> 128 128 1 0\\n")
a, b = kernels(one), kernels(each)
assert len(a) == 1 if {old} else len(a) > 2         # the plain kernel's old entry still holds
assert len(b) > 2                                   # timed: it took neither entry
assert a[-1] != b[-1]                               # with different kernels
assert len(kernels(one)) == len(kernels(each)) == 1 # and now taken from the file
""")
