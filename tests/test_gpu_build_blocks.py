"""ACE build at the edges of the Cholesky factor's 64-wide blocks and past the
256 entries that the triangular inverse prefetches, against numpy in FP64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_1801_09263_amd import lace  # noqa: E402
from paper_1801_09263_amd.session import CellSession  # noqa: E402

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


def session(n):
    r = np.arange(-5, 6)
    mz, my, mx = np.meshgrid(r, r, r, indexing="ij")
    miller = np.stack([mx.ravel(), my.ravel(), mz.ravel()], 1).astype(np.int32)
    rng = np.random.default_rng(500 + n)

    def ortho(rows, cols):
        z = rng.standard_normal((rows, cols)) + 1j * rng.standard_normal((rows, cols))
        return np.linalg.qr(z)[0]

    s = CellSession(dict(L=10.0, n=24, miller=miller), n, lace.LACE_FP64)
    psi = np.ascontiguousarray(ortho(miller.shape[0], n).T)
    s.set_orbitals(psi)
    return s, psi, ortho(n, n)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 127, 128, 129, 256, 257, 258, 321])
def test_build(n):
    s, psi, u = session(n)
    # -M has eigenvalues 1 ... 2, so that the bounds below need no conditioning
    h = (u * np.linspace(1.0, 2.0, n)) @ u.conj().T
    w = -(h.T @ psi)
    s.w.copy_(torch.tensor(np.ascontiguousarray(w)))
    s.build_ace("avg")
    torch.cuda.synchronize()
    assert s.info() == 0
    m = psi.conj() @ w.T
    chol = np.linalg.cholesky(-0.5 * (m + m.conj().T))
    xi = np.linalg.solve(chol.conj(), w)   # rows: xi = W L^-H, transposed
    got = s.xi.cpu().numpy()
    s.close()
    # sums of n_pw terms in M, of up to n in the factor and its inverse
    tol = 8 * EPS * (np.sqrt(psi.shape[1]) + n)
    err = np.linalg.norm(got - xi) / np.linalg.norm(xi)
    print(f"n {n}: err {err:.1e} tol {tol:.1e}", flush=True)
    assert err <= tol


@pytest.mark.parametrize("n,bad", [(65, 0), (65, 63), (65, 64), (130, 70), (300, 128),
                                   (300, 299)])
def test_first_failing_pivot(n, bad):
    s, psi, _ = session(n)
    f = np.ones(n)
    f[bad] = -1.0
    s.w.copy_(torch.tensor(-f[:, None] * psi))
    s.build_ace("avg")
    torch.cuda.synchronize()
    assert s.info() == bad + 1
    s.close()
