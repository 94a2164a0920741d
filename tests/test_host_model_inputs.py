"""A model's bad values are refused first: before the predictions are
allocated (bad values are reported also where those do not fit) and before
anything is evaluated.  On the runtime in host memory."""
import pytest

from tests import fake

MODELS = {
    "forest": """
def load(bad):
    leaves = np.ones((2, 16, C), np.float32)
    if bad: leaves[1, 3, 2] = bad
    z = np.zeros((2, 15), np.uint8)
    return m.ForestModel(sp, z, z, leaves)
values, where = (np.nan, -1.0, np.inf), f"leaf value {(16 + 3) * C + 2} is negative or not finite"
""",
    "table": """
def load(bad):
    p = np.ones((sp.n_valid, C), np.float32)
    if bad: p[77, 5] = bad
    return m.TableModel(sp, p)
values, where = (np.nan, -1.0, np.inf), f"prediction {77 * C + 5} is negative or not finite"
""",
    "mlp": """
def load(bad):
    flat = np.zeros(m._lib.cgs_mlp_param_count(ctypes.byref(m.cgs_mlp_desc(3, 64, C, 0))), np.float32)
    if bad: flat[1234] = bad
    h = ctypes.c_void_p()
    m._check(m._lib.cgs_model_load_mlp(sp.h, ctypes.byref(m.cgs_mlp_desc(3, 64, C, 0)), m._ptrof(flat),
                                       ctypes.byref(h)), "cgs_model_load_mlp")
    m._lib.cgs_model_destroy(h)
values, where = (np.nan, np.inf), "parameter 1234 not finite"
""",
}


@pytest.mark.parametrize("kind", MODELS)
def test_bad_values_are_refused_before_all_else(kind):
    fake.run("C = 24\nsp = space(16, 16, 16)\n" + MODELS[kind] + """
load(None)
for bad in values:
    # room for all, for the inputs but not the predictions, and for nothing
    for room in (1 << 40, 395_000, 0):
        sp.close()
        sp = space(16, 16, 16)                 # a pool without blocks
        fake.fake_limit(room)
        fake.fake_clear()
        try:
            load(bad)
            raise SystemExit("accepted")
        except m.CgsError as e:
            assert e.status == m.EINVAL and where in str(e), (room, str(e))
        launched = [e[2] for e in log() if e[0] == "launch"]
        assert all("check_" in k for k in launched), launched
        if room < 1 << 40:
            fake.fake_limit(1000)
            assert status(lambda: load(None)) == m.ENOMEM, room
        fake.fake_limit(1 << 40)
load(None)
""")


@pytest.mark.parametrize("depth,C,device", [(0, 24, False), (10, 16, False), (10, 17, True)])   # up to 16,384 values
def test_few_values_are_looked_through_on_the_host(depth, C, device):
    fake.run(f"""
sp = space(4, 4, 4)
z = np.zeros((1, (1 << {depth}) - 1), np.uint8)
leaves = np.ones((1, 1 << {depth}, {C}), np.float32)
fake.fake_clear()
m.ForestModel(sp, z, z, leaves)
assert any("check_" in e[2] for e in log() if e[0] == "launch") == {device}
leaves[0, -1, -1] = np.nan
assert status(lambda: m.ForestModel(sp, z, z, leaves)) == m.EINVAL
""")
