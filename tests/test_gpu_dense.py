"""Dense inverse of a coarsest multigrid level, formed on the device: one-level
hierarchies, where the pressure V-cycle (op 8) is exactly the inverse of
B_I Lambda_V^-1 B_I^T + M_Q, against SciPy's solve with the exported matrices.

Sizes are whole 64-row tiles (64 and 4,096 rows) and ragged ones, up to the
largest odd meshes that take the dense inverse.  Tolerances: FP64 1e-10 (the
condition number, below 1e5 here, times the rounding of a few thousand
operations per entry), FP32 1e-5 (the rounding of the stored inverse, 6e-8,
times the cancellation of its rows)."""

import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg as spl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dim,n,nrhs", [(2, 2, 1), (2, 7, 1), (3, 3, 2), (2, 8, 8), (3, 9, 4), (3, 13, 1), (2, 63, 2),
                                        (3, 17, 1), (2, 93, 1)])
def test_one_level_cycle_is_the_inverse(gpu_lib, dim, n, nrhs):
    from paper_2407_01783_amd.stokes import StokesProblem
    print(f"[case] dense dim={dim} n={n} nrhs={nrhs}", flush=True)
    P = StokesProblem(dim, n, mesh_seed=6, jitter=0.1, mu=0.02, alpha=50.0)
    mats = []
    for which in (9, 5):
        rp, cols, vals = P.export_csr(which)
        mats.append(sp.csr_matrix((vals, cols, rp), shape=(P.n_p1, P.n_p1)))
    X = (mats[0] + mats[1]).tocsc()
    x = np.random.default_rng(n).standard_normal((nrhs, P.n_p1))
    ref = spl.splu(X).solve(x.T).T
    for precision, tol in ((0, 1e-10), (1, 1e-5)):
        y = P.apply(8, torch.tensor(x.ravel(), device="cuda"), precision=precision, nrhs=nrhs).cpu().numpy()
        assert np.linalg.norm(y - ref.ravel()) <= tol * np.linalg.norm(ref), precision
