"""Products whose slices are shared by two or four wavefronts (the choice
follows the number of rows and the width) against SciPy products with the
exported FP64 matrices, and the velocity preconditioner against the Chebyshev
iteration with them.  Tolerances as in the parity tests of the same operators: products 1e-13
(FP64) and 1e-6 (FP32), the degree-6 polynomial 1e-11 and 2e-3.
"""

import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _problem(dim, n, **kw):
    from paper_2407_01783_amd.stokes import StokesProblem
    print(f"[case] dim={dim} n={n} {kw}", flush=True)
    return StokesProblem(dim, n, mesh_seed=4, jitter=0.1, mu=0.02, alpha=50.0, **kw)


def _csr(P, which, ncols):
    rp, cols, vals = P.export_csr(which)
    return sp.csr_matrix((vals, cols, rp), shape=(len(rp) - 1, ncols))


def _chebyshev(A, lo, hi, steps, r):
    """Chebyshev iteration for D^-1 A z = D^-1 r from 0 (Saad, Iterative
    Methods for Sparse Linear Systems, Alg. 12.1), r: [n, columns]."""
    dinv = (1.0 / A.diagonal())[:, None]
    theta, delta = 0.5 * (hi + lo), 0.5 * (hi - lo)
    rho = delta / theta
    res, d = r.copy(), dinv * r / theta
    z = d.copy()
    for _ in range(steps - 1):
        res -= A @ d
        rho_next = 1.0 / (2.0 * theta / delta - rho)
        d = rho_next * rho * d + 2.0 * rho_next / delta * (dinv * res)
        rho = rho_next
        z += d
    return z


def _rel(y, ref):
    return np.linalg.norm(y.ravel() - ref.ravel()) / max(np.linalg.norm(ref), 1e-300)


# width 3: four wavefronts below 87,382 rows, two below 524,288, one from there
# on; width 1: four below 131,072, then one.  n = 1 and 2: one slice, 1 and 27
# rows; 22: 79,507 rows; 23: 91,125; 41: 531,441 and 74,088; 51: 140,608
# pressure rows.  Two and four right-hand sides and 2D: never shared.
@pytest.mark.parametrize("dim,n,nrhs,p3", [(3, 1, 1, False), (3, 2, 1, False), (3, 5, 1, False), (3, 22, 1, False),
                                           (3, 23, 1, False), (3, 41, 1, False), (3, 51, 1, False), (3, 5, 2, False),
                                           (2, 9, 1, False), (2, 5, 4, False), (3, 3, 1, True), (3, 16, 1, True)])
def test_shared_slices(gpu_lib, dim, n, nrhs, p3):
    P = _problem(dim, n, p3=p3)
    rng = np.random.default_rng(n)
    k = (3 if p3 else 2) * n
    idx = np.indices((k + 1,) * dim).reshape(dim, -1)
    inside = ((idx > 0) & (idx < k)).all(0)
    xu = rng.standard_normal((nrhs, dim, P.n_p2)) * inside
    xp = rng.standard_normal((nrhs, P.n_p1))
    A = 50.0 * _csr(P, 0, P.n_p2) + 0.02 * _csr(P, 1, P.n_p2)
    B = [_csr(P, 2 + c, P.n_p2) for c in range(dim)]
    ref = {0: np.stack([[(A @ xu[r, c]) * inside for c in range(dim)] for r in range(nrhs)]),
           2: np.stack([[(B[c].T @ xp[r]) * inside for c in range(dim)] for r in range(nrhs)])}
    for op, which in ((3, 5), (4, 6), (7, 9)):
        S = _csr(P, which, P.n_p1)
        ref[op] = np.stack([S @ xp[r] for r in range(nrhs)])
    lo, hi = P.bounds()[:2]
    I = np.flatnonzero(inside)
    A_II = A[I][:, I]
    ref[10] = np.zeros_like(xu)
    for r in range(nrhs):
        ref[10][r][:, I] = _chebyshev(A_II, lo, hi, 6, xu[r][:, I].T).T
    for op, want in ref.items():
        x = xu if op in (0, 10) else xp
        for precision in (0, 1):
            tol = ((1e-11, 2e-3) if op == 10 else (1e-13, 1e-6))[precision]
            y = P.apply(op, torch.tensor(x.ravel(), device="cuda"), precision=precision, nrhs=nrhs).cpu().numpy()
            assert _rel(y, want) <= tol, (op, precision)


# the dot products of the inner CGs over shared slices
@pytest.mark.parametrize("n,precision", [(9, 0), (9, 1), (23, 0), (23, 1)])
def test_tolerance_driven_solve(gpu_lib, monkeypatch, n, precision):
    from paper_2407_01783_amd import inputs
    monkeypatch.setenv("STOKES_PCG_SMALL", "0")
    P = _problem(3, n)
    xy, _ = P.mesh()
    f = torch.tensor(inputs.fourier_forcing(xy, inputs.forcing_seed(4, 0)), device="cuda")
    u, p, info = P.solve(f, method="coupled", precision=precision, rtol=1e-8, inner_mode=0)
    assert info["status"] == 0, info
    assert P.residual(f, u, p).max() <= 1.01e-8
