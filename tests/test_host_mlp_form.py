"""Which kernels a perceptron's rows take, on the runtime in host memory: steps
of a run are split over columns at 512 hidden units and up to 1,024 rows, a
step by itself is not."""
import pytest

from tests import fake


@pytest.mark.parametrize("H,n,split", [(512, 1, True), (512, 1024, True), (512, 1025, False), (256, 64, False)])
def test_the_form_follows_the_work(H, n, split):
    fake.run(f"""
sp = space(16, 16, 16)
H, C = {H}, 24
z = lambda *s: np.zeros(s, np.float32)
mo = m.MLPModel(sp, [z(H, 3), z(H), z(H, H), z(H), z(C, H), z(C)])
cfg, y = np.arange({n}, dtype=np.uint32), np.ones(({n}, C), np.float32)
def kernels(call):
    fake.fake_clear()
    call()
    return {{k for e in log() if e[0] == "launch" for k in ("mlp_split_forward", "mlp_split_backward", "mlp_train_rows")
            if k in e[2]}}
assert kernels(lambda: mo.gradients(cfg, y)) == {{"mlp_train_rows"}}
want = {{"mlp_split_forward", "mlp_split_backward"}} if {split} else {{"mlp_train_rows"}}
assert kernels(lambda: mo.train(cfg, y, np.arange({n}, dtype=np.int32)[None])) == want
""")
