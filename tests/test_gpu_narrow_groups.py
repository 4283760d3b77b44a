"""ACE application to 17 ... 32 functions on both sides of the line between one
and two groups of columns, against plain torch in FP64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_1801_09263_amd import lace  # noqa: E402

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


# few plane waves; the first count beyond 16384; a side below and above 300 MB
@pytest.mark.parametrize("n_vec", [17, 31, 32])
@pytest.mark.parametrize("n_orb,n_pw", [(130, 300), (40, 16384), (40, 16385),
                                        (1139, 16400), (1150, 16400)])
def test_apply(n_orb, n_vec, n_pw):
    r = np.arange(-15, 16)
    mz, my, mx = np.meshgrid(r, r, r, indexing="ij")
    miller = np.stack([mx.ravel(), my.ravel(), mz.ravel()], 1).astype(np.int32)[:n_pw]
    plan = lace.lace_plan_create([dict(L=10.0, n=32, miller=miller)], lace.LACE_FP64)
    gen = torch.Generator(device="cuda").manual_seed(n_orb + n_vec)
    xi, x = (torch.complex(*(torch.randn((k, n_pw), generator=gen, device="cuda",
                                         dtype=torch.float64) for _ in range(2)))
             for k in (n_orb, n_vec))
    # room past the end of y that no store may touch
    guard = torch.full((n_vec * n_pw + 64,), 7.0, dtype=torch.complex128, device="cuda")
    y = guard[: n_vec * n_pw]
    lace.lace_apply_ace_noalloc(plan, 0, xi, n_orb, x, n_vec, y)
    torch.cuda.synchronize()
    plan.close()
    xh, vh = xi.cpu(), x.cpu()
    ref = -((xh.conj() @ vh.t()).t() @ xh)
    # each element: n_orb products of n_pw-term sums; the bound is on the
    # sums of moduli
    mag = (xh.abs() @ vh.abs().t()).t() @ xh.abs()
    err = (y.view(n_vec, n_pw).cpu() - ref).abs()
    tol = 4 * EPS * (np.sqrt(n_pw) + np.sqrt(n_orb) + 4) * mag
    assert bool((err <= tol).all()), float((err / tol).max())
    assert bool((guard[n_vec * n_pw:] == 7.0).all())
