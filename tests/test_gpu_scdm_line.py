"""SCDM on both sides of the line between downdating every point and the lazy
selection, in every grid form; and an input that makes the lazy selection give
up.  The picks are checked as in test_gpu_scdm_lazy."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
from paper_1801_09263_amd import lace  # noqa: E402
from test_gpu_scdm_lazy import L, check_greedy, run  # noqa: E402

pytestmark = pytest.mark.gpu


# the last count that downdates every point and one that is lazy, at 80^3; the
# tolerances are the rounding of the grids' precision, as for the other picks
@pytest.mark.parametrize("prec,n_orb,tol", [
    ("fp32g", 94, 1e-6), ("fp64g", 51, 1e-13), ("fp64g", 53, 1e-13),
    ("fp32", 62, 1e-6), ("fp32", 63, 1e-6), ("fp64", 36, 1e-13),
    ("fp64", 37, 1e-13), ("fp64", 66, 1e-13)])
def test_picks_are_greedy(prec, n_orb, tol):
    miller = synth.miller_sphere(L, 40.0)
    c = synth.gaussian_orbitals(miller, L, n_orb, (n_orb + 1) // 2, synth.rng_for(74))
    rng = np.random.default_rng(75)
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
    """Plane waves: no histogram bin separates the points."""
    miller = synth.miller_sphere(L, 40.0)
    c = np.zeros((40, miller.shape[0]), dtype=np.complex128)
    c[np.arange(40), np.random.default_rng(76).permutation(miller.shape[0])[:40]] = 1.0
    points, _ = run(c, miller, lace.LACE_FP64)
    check_greedy(c, miller, points, 1e-12)


@pytest.mark.parametrize("prec,n_orb", [("fp64g", 55), ("fp64", 39)])
def test_gives_up_after_refreshes_without_a_pick(prec, n_orb):
    """Two orbitals hold almost all of the density, everywhere: their picks
    leave nothing of the points that each following refresh selects by their
    old values, and there are more such refreshes (the same selection in numpy
    counts 9) than are allowed before every point is updated.  The other
    orbitals are picked after that."""
    miller = synth.miller_sphere(L, 40.0)
    c = 1e-4 * synth.gaussian_orbitals(miller, L, n_orb, (n_orb + 1) // 2,
                                       synth.rng_for(77))
    # f(x) f(y) f(z) with f = 1.2 + cos, of one and two periods: each density
    # over 20 octaves
    for k, amp in ((1, 1.0), (2, 1e-2)):
        w = {0: 1.2, k: 0.5, -k: 0.5}
        c[k - 1] = [amp * np.prod([w.get(int(v), 0.0) for v in m]) for m in miller]
    p = lace.LACE_FP64_GAMMA if prec.endswith("g") else lace.LACE_FP64
    points, _ = run(c, miller, p)
    check_greedy(c, miller, points, 1e-13)
