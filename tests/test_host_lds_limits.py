"""The LDS that a kernel may use is set once and for all of its launches: a
limit set for a smaller launch on one thread must not stand in the way of a
larger one on another.  On the runtime in host memory, which logs the limits."""
from tests import fake

PROLOGUE = """
limits = {}
def note():
    for e in log():
        if e[0] == "attr": limits.setdefault(e[2], set()).add(int(e[3]))
"""


def test_limits_do_not_depend_on_the_launch():
    fake.run(PROLOGUE + """
def tune(sp):
    f = forest(sp, 24)
    b = m.Batch([m.Session(sp) for _ in range(64)], [f] * 64)
    b.tuning_run(np.ones(sp.n_valid, np.float32), np.ones((sp.n_valid, 24)), U[:3200].reshape(64, 50), draws=1,
                 max_tests=30, stop_at_well=True)
    b = m.Batch([m.Session(sp) for _ in range(2)], [f] * 2)
    b.tuning_run(np.ones(sp.n_valid, np.float32), np.ones((sp.n_valid, 24)), U[:100].reshape(2, 50), draws=1,
                 max_tests=1, stop_at_well=True)
for radix in ((16, 16, 3), (16, 16, 16, 5), (16, 16, 16, 8)):
    sp = space(*radix)
    tune(sp)
    f = forest(sp, 4)
    s = m.Session(sp)
    s.search_step(f, m.NO_PROFILE)
    s.sample_next(1)
    sp.close()
for radix in ((16, 16, 15, 7), (13, 13, 13, 13)):
    sp = space(*radix)
    f = forest(sp, 64)
    s = m.Session(sp)
    s.search_step_neighbourhood(f, 0, 3, delta=np.full(64, 0.5, np.float32))
    s.sample_next(1)
sp = space(8, 8, 8)
for T, D in ((9, 13), (16, 13), (12, 13)):
    z = np.zeros((T, (1 << D) - 1), np.uint8)
    m.ForestModel(sp, z, z, np.ones((T, 1 << D, 4), np.float32))
for radix in ((4, 4, 4, 4), (16,) * 4, (16,) * 5):
    sp = space(*radix)
    pts = np.arange(200, dtype=np.uint32)
    for C in (8, 24, 64):
        status(lambda: m.PolyModel(sp, pts, np.ones((200, C), np.float32), 2))
        status(lambda: m.ForestModel.fit(sp, pts, np.ones((200, C), np.float32), U[:200], 4))
note()
names = ("batch_tune", "batch_small", "small_step", "nb_step", "forest_eval_resident", "fit_split")
for n in names:
    assert any(n in k for k in limits), (n, sorted(limits))
for k, v in limits.items():
    assert len(v) == 1 or not any(n in k for n in (*names, "poly_")), (k, v)
""")
