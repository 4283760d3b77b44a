"""Batches run in groups (one launch for several batches' passes A and B)
against the same schedule run batch by batch, as a profiled call runs it."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
from paper_1801_09263_amd import lace  # noqa: E402
from paper_1801_09263_amd.session import CellSession  # noqa: E402

pytestmark = pytest.mark.gpu


# small grids, group sizes that do not divide the batch count, one-pair
# batches, both xy schedules, every z tile and radix order
@pytest.mark.parametrize("prec,n,L,n_orb,virt,tuning", [
    ("fp32", 8, 4.0, 1, 0, (32, 1, 0, 0)),
    ("fp32g", 12, 5.0, 3, 1, (32, 1, 0, 0)),
    ("fp32", 24, 10.0, 9, 2, (5, 1, 1, 0)),
    ("fp32g", 24, 10.0, 17, 0, (1, 2, 0, 0)),
    ("fp32g", 24, 10.0, 20, 3, (32, 2, 2, 1)),
    ("fp64", 32, 13.0, 7, 0, (32, 1, 0, 1)),
    ("fp64g", 48, 12.0, 13, 2, (16, 2, 1, 0)),
    ("fp32", 48, 12.0, 21, 0, (64, 2, 0, 0)),
    ("fp32g", 80, 20.0, 12, 0, (128, 1, 2, 0)),
])
def test_group_equals_batches(prec, n, L, n_orb, virt, tuning):
    p = {"fp32": lace.LACE_FP32, "fp64": lace.LACE_FP64,
         "fp32g": lace.LACE_FP32_GAMMA, "fp64g": lace.LACE_FP64_GAMMA}[prec]
    miller = synth.miller_sphere(L, min(40.0, 0.5 * (2 * np.pi * 0.36 * n / L) ** 2))
    c = synth.virtual_orbitals(miller, L, np.zeros((0, miller.shape[0]), complex),
                               n_orb, synth.rng_for(81, n_orb), real=prec.endswith("g"))
    s = CellSession(dict(L=L, n=n, miller=miller), n_orb, p)
    lace.lace_set_tuning(s.plan, 0, *tuning)
    s.set_orbitals(c)
    s.ws.fill_(0xff)   # no value of an earlier call is used
    out = []
    for profiled in (False, True, False):
        lace.lace_profile_enable(s.plan, profiled)
        s.w.fill_(float("nan"))
        s.apply_exchange(0.05, n_occ=n_orb - virt)
        torch.cuda.synchronize()
        out.append((s.w.clone(), s.e_x.item(), s.n_kept))
    s.close()
    for w, e, kept in out[1:]:
        assert torch.equal(w, out[0][0])
        assert kept == out[0][2]
        assert e == out[0][1]
    assert torch.isfinite(torch.view_as_real(out[0][0])).all()
