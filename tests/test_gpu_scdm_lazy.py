"""SCDM point selection on grids large enough for the lazy selection: every
pick has to be a greedy pick by definition, checked against residuals that
plain FP64 torch computes from the same coefficients."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
from paper_1801_09263_amd import lace  # noqa: E402

pytestmark = pytest.mark.gpu

N = 80
L = 20.0


def grids(coeffs, miller):
    """psi on the grid up to a constant factor, (n_orb, N^3), FP64."""
    m = torch.as_tensor(miller, device="cuda", dtype=torch.int64) % N
    idx = (m[:, 2] * N + m[:, 1]) * N + m[:, 0]
    out = torch.zeros((coeffs.shape[0], N ** 3), dtype=torch.complex128, device="cuda")
    for k in range(coeffs.shape[0]):
        out[k, idx] = torch.as_tensor(coeffs[k], device="cuda")
        out[k] = torch.fft.ifftn(out[k].view(N, N, N)).reshape(-1)
    return out


def check_greedy(coeffs, miller, points, tol):
    psi = grids(coeffs, miller)
    d = (psi.real ** 2 + psi.imag ** 2).sum(0)
    top = float(d.max())
    q = torch.zeros((len(points),) * 2, dtype=torch.complex128, device="cuda")
    worst = 0.0
    for k, r in enumerate(points):
        worst = max(worst, (float(d.max()) - float(d[r])) / top)
        u = psi[:, r].conj().resolve_conj()
        for _ in range(2):
            u = u - q[:k].t() @ (q[:k].conj() @ u)
        q[k] = u / torch.linalg.vector_norm(u)
        t = (q[k:k + 1] @ psi)[0]
        d = d - (t.real ** 2 + t.imag ** 2)
        d[r] = -top
    print(f"greedy: worst shortfall {worst:.1e} of the density (tol {tol:.1e})",
          flush=True)
    assert worst <= tol


def run(coeffs, miller, prec):
    n = coeffs.shape[0]
    plan = lace.lace_plan_create([dict(L=L, n=N, miller=miller)], prec)
    ws = torch.empty(lace.lace_workspace_size(plan, 0, n, n), dtype=torch.uint8,
                     device="cuda")
    psi = torch.tensor(coeffs, device="cuda")
    phi = torch.empty_like(psi)
    pts = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    resid = torch.zeros(1, dtype=torch.float64, device="cuda")
    out = []
    for _ in range(2):
        lace.lace_scdm(plan, 0, psi, n, phi, pts, resid, ws)
        torch.cuda.synchronize()
        out.append((pts.cpu().numpy().copy(), phi.cpu().numpy().copy()))
    plan.close()
    assert np.array_equal(out[0][0], out[1][0])
    assert np.array_equal(out[0][1], out[1][1])
    points = out[0][0]
    assert len(set(points.tolist())) == n
    assert points.min() >= 0 and points.max() < N ** 3
    return points, resid.item()


# one orbital fewer than takes the lazy form, and odd counts above it; the
# values differ from exact ones by the rounding of the grids' precision
@pytest.mark.parametrize("prec,n_orb,tol", [
    ("fp32g", 93, 1e-6), ("fp32g", 97, 1e-6), ("fp64g", 49, 1e-13),
    ("fp32", 47, 1e-6), ("fp64", 25, 1e-13)])
def test_picks_are_greedy(prec, n_orb, tol):
    miller = synth.miller_sphere(L, 40.0)
    c = synth.gaussian_orbitals(miller, L, n_orb, (n_orb + 1) // 2, synth.rng_for(71))
    rng = np.random.default_rng(72)
    a = rng.standard_normal((n_orb, n_orb))
    if not prec.endswith("g"):
        a = a + 1j * rng.standard_normal((n_orb, n_orb))
    c = np.ascontiguousarray(np.linalg.qr(a)[0] @ c)
    p = {"fp32g": lace.LACE_FP32_GAMMA, "fp64g": lace.LACE_FP64_GAMMA,
         "fp32": lace.LACE_FP32, "fp64": lace.LACE_FP64}[prec]
    points, resid = run(c, miller, p)
    check_greedy(c, miller, points, tol)
    assert resid <= 1e-12


def test_uniform_density():
    """Plane waves: every point has the same density, so no histogram bin
    separates them and every point is downdated in every step."""
    miller = synth.miller_sphere(L, 40.0)
    c = np.zeros((26, miller.shape[0]), dtype=np.complex128)
    c[np.arange(26), np.random.default_rng(73).permutation(miller.shape[0])[:26]] = 1.0
    points, _ = run(c, miller, lace.LACE_FP64)
    check_greedy(c, miller, points, 1e-12)
