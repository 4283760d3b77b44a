"""SCDM with many complex orbitals on a small grid: the 1024-thread pick, whose
column and partial sums take more than 64 KB of LDS, up to the limit of the
call.  Every pick has to be a greedy one."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_1801_09263_amd import lace  # noqa: E402

pytestmark = pytest.mark.gpu

N = 16


@pytest.mark.parametrize("n_orb", [200, 1600, 3072])
def test_picks_are_greedy(n_orb):
    r = np.arange(-7, 8)
    mz, my, mx = np.meshgrid(r, r, r, indexing="ij")
    miller = np.stack([mx.ravel(), my.ravel(), mz.ravel()], 1).astype(np.int32)
    gen = torch.Generator(device="cuda").manual_seed(n_orb)
    z = torch.randn((miller.shape[0], n_orb, 2), generator=gen, device="cuda",
                    dtype=torch.float64)
    c = torch.linalg.qr(torch.view_as_complex(z))[0].t().contiguous()
    plan = lace.lace_plan_create([dict(L=8.0, n=N, miller=miller)], lace.LACE_FP64)
    ws = torch.empty(lace.lace_workspace_size(plan, 0, n_orb, 0), dtype=torch.uint8,
                     device="cuda")
    phi = torch.empty_like(c)
    pts = torch.full((n_orb,), -1, dtype=torch.int32, device="cuda")
    lace.lace_scdm(plan, 0, c, n_orb, phi, pts, None, ws)
    torch.cuda.synchronize()
    plan.close()
    points = pts.cpu().numpy()
    assert len(set(points.tolist())) == n_orb
    assert points.min() >= 0 and points.max() < N ** 3
    m = torch.as_tensor(miller, device="cuda", dtype=torch.int64) % N
    psi = torch.zeros((n_orb, N ** 3), dtype=torch.complex128, device="cuda")
    psi[:, (m[:, 2] * N + m[:, 1]) * N + m[:, 0]] = c
    psi = torch.fft.ifftn(psi.view(-1, N, N, N), dim=(1, 2, 3)).reshape(n_orb, -1)
    d = (psi.real ** 2 + psi.imag ** 2).sum(0)
    top = d.max()
    q = torch.zeros((n_orb, n_orb), dtype=torch.complex128, device="cuda")
    worst = torch.zeros((), dtype=torch.float64, device="cuda")
    for k, p in enumerate(points.tolist()):
        worst = torch.maximum(worst, (d.max() - d[p]) / top)
        u = psi[:, p].conj().resolve_conj()
        for _ in range(2):
            u = u - torch.mv(q[:k].t(), torch.mv(q[:k].conj().resolve_conj(), u))
        q[k] = u / torch.linalg.vector_norm(u)
        t = torch.mv(psi.t(), q[k])
        d = d - (t.real ** 2 + t.imag ** 2)
        d[p] = -top
    # each of the k differences rounds once on either side
    tol = 8 * n_orb * np.finfo(np.float64).eps
    print(f"greedy: worst shortfall {worst.item():.1e} of the density (tol {tol:.1e})",
          flush=True)
    assert worst.item() <= tol
