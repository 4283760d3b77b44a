"""The polar factor of the alignment at the edges of its tiles and of its
one-workgroup form, against the oracle's SVD."""
import numpy as np
import pytest

import oracle as O

torch = pytest.importorskip("torch")
from paper_1801_09263_amd import lace  # noqa: E402

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


def orthonormal(rng, n_pw, n):
    z = rng.standard_normal((n_pw, n)) + 1j * rng.standard_normal((n_pw, n))
    return np.ascontiguousarray(np.linalg.qr(z)[0].T)


@pytest.mark.parametrize("n", [1, 3, 16, 17, 32, 33, 48, 49, 64, 65, 130, 256, 257])
@pytest.mark.parametrize("related", [True, False])
def test_polar_factor(n, related):
    r = np.arange(-5, 6)
    mz, my, mx = np.meshgrid(r, r, r, indexing="ij")
    miller = np.stack([mx.ravel(), my.ravel(), mz.ravel()], 1).astype(np.int32)
    rng = np.random.default_rng(1000 + n)
    old = orthonormal(rng, miller.shape[0], n)
    new = orthonormal(rng, miller.shape[0], n)
    if related:
        new = np.ascontiguousarray(
            np.linalg.qr((old + 0.02 * new).T @ np.linalg.qr(
                rng.standard_normal((n, n)))[0])[0].T)
    plan = lace.lace_plan_create([dict(L=10.0, n=24, miller=miller)], lace.LACE_FP64)
    ws = torch.empty(lace.lace_workspace_size(plan, 0, n, n), dtype=torch.uint8,
                     device="cuda")
    tn, to = torch.tensor(new, device="cuda"), torch.tensor(old, device="cuda")
    out = torch.empty_like(tn)
    resid = torch.full((1,), -1.0, dtype=torch.float64, device="cuda")
    again = torch.empty_like(tn)
    lace.lace_align(plan, 0, tn, to, n, out, resid, ws)
    lace.lace_align(plan, 0, tn, to, n, again, None, ws)
    torch.cuda.synchronize()
    plan.close()
    s = np.linalg.svd(np.conj(new) @ old.T, compute_uv=False)
    ref = O.align_orbitals(new, old)
    err = np.linalg.norm(out.cpu().numpy() - ref) / np.linalg.norm(ref)
    # a perturbation d of A moves its polar factor by at most 2 d / s_min;
    # d is the rounding of n_pw-term sums (64 eps leaves room for both sides)
    tol = 64 * EPS * np.sqrt(n) * s[0] / s[-1]
    print(f"n {n} related {related}: err {err:.1e} tol {tol:.1e} "
          f"resid {resid.item():.1e}", flush=True)
    assert err <= tol
    assert resid.item() <= 64 * EPS * np.sqrt(n)
    assert torch.equal(out, again)
