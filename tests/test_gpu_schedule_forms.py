"""The device schedule at the orbital counts where its packing changes form
(one, two and four bit words per batch, then LDS) and the round-robin
fallback with more rounds than a workgroup has threads."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
from paper_1801_09263_amd import lace  # noqa: E402
from paper_1801_09263_amd.session import CellSession  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fallback", [False, True], ids=["first-fit", "round-robin"])
@pytest.mark.parametrize("prec", [lace.LACE_FP32, lace.LACE_FP32_GAMMA],
                         ids=["complex", "gamma"])
@pytest.mark.parametrize("n_orb", [1, 2, 63, 64, 65, 128, 129, 256, 257, 300])
def test_schedule(n_orb, prec, fallback, monkeypatch):
    monkeypatch.setenv("LACE_SCHEDULE_FALLBACK", "1" if fallback else "0")
    L, n_grid, ppb = 4.0, 8, 24
    miller = synth.miller_sphere(L, 6.0)
    rng = np.random.default_rng(n_orb)
    pairs = np.array([(i, j) for j in range(n_orb) for i in range(j + 1)
                      if i == j or rng.random() < 0.6])
    s = CellSession(dict(L=L, n=n_grid, miller=miller), n_orb, prec)
    lace.lace_set_tuning(s.plan, 0, ppb, 2)
    s.psi.fill_(0.01)
    s.apply_exchange(0.0, pairs=pairs)
    bo, so, nb = lace.lace_read_schedule(s.plan, 0, n_orb, s.ws, pairs)
    kept = s.n_kept
    s.close()
    assert kept == len(pairs)
    assert bo.min() >= 0 and so.min() >= 0 and bo.max() == nb - 1
    assert np.bincount(bo).max() <= ppb
    for b in range(nb):   # no orbital in two slots of a batch
        k = np.nonzero(bo == b)[0]
        seen = {}
        for t in k:
            for o in set(pairs[t].tolist()):
                assert seen.setdefault(o, so[t]) == so[t]
    if not fallback:
        if prec == lace.LACE_FP32_GAMMA:
            bh, sh, nh = lace.lace_schedule_slots(pairs, n_orb, ppb)
            assert np.array_equal(so, sh)
        else:
            bh, nh = lace.lace_schedule_pairs(pairs, n_orb, ppb)
        assert nb == nh and np.array_equal(bo, bh)
    else:                 # batches of one round each, rounds in order
        m = n_orb + (n_orb & 1) - 1

        def round_of(i, j):
            if i == j:
                return m
            if j == m:
                return i
            return ((i + j) * ((m + 1) // 2)) % m

        r = np.array([round_of(int(i), int(j)) for i, j in pairs])
        order = np.array([r[bo == b][0] for b in range(nb)])
        assert all((r[bo == b] == order[b]).all() for b in range(nb))
        assert (np.diff(order) >= 0).all()
