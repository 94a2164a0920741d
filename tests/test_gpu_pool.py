"""Buffers and streams kept between handles (released by one, used by the
next, on other streams and threads): every handle starts from its own state
and gives the results it gives alone."""
import threading

import numpy as np
import pytest

import synth
from tests.helpers import cgs

pytestmark = pytest.mark.gpu


def _search(m, key, radix, sizes):
    """Searches, a batch and a fitted tree on a space of its own; everything
    opened is closed again, so that the next handles use its buffers."""
    spec = synth.Space(list(radix), [list(range(1, r + 1)) for r in radix])
    g = synth.rng(70, key)
    forest = synth.random_forest(g, spec.radix, 2, 5, 24)
    pcs, U = synth.profiler_counters(g, 6), synth.uniforms_u64(g, 8)
    eps = [m.cgs_default_expert_params() for _ in range(6)]
    sp = m.Space.from_spec(spec)
    out = []
    for n in sizes:
        model = m.ForestModel.from_spec(sp, forest)
        sessions = [m.Session(sp) for _ in range(n)]
        for s in sessions[:2]:
            out.append(s.search_run(model, pcs, eps, U)[1].tolist())
            out.append(int(s.copy_explored().view(np.uint8).sum()))
        batch = m.Batch(sessions[2:], [model] * (n - 2))
        out.append(batch.step([m.NO_PROFILE] * (n - 2), None, U[:n - 2])[1].tolist())
        batch.close()
        pts = synth.uniform_indices(g, 300, sp.n_valid).astype(np.uint32)
        fit, rep = m.ForestModel.fit(sp, pts, model.gather_predictions(pts),
                                     synth.uniforms_u64(g, 300), 4)
        out.append((rep["depth"], rep["abs_err"]))
        for h in sessions + [model, fit]:
            h.close()
    sp.close()
    return out


def test_threads_share_released_buffers():
    m = cgs()
    shapes = [(1, (16, 16, 16), (4, 9, 3)), (2, (15, 14, 13, 12, 2), (3, 5, 8))]
    alone = [_search(m, *a) for a in shapes]
    got = [[], []]

    def work(i):
        for _ in range(3):
            got[i].append(_search(m, *shapes[i]))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i in range(2):
        assert got[i] == [alone[i]] * 3
