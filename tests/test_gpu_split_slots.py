"""Pressure products and V-cycles around the sizes where the number of
wavefronts per slice changes: rows of fewer than 24 slots share a slice by four
below 49,152 rows (of fewer than 10 in 2D, 28,672) and, in 3D, by two up to
65,536; longer rows by four up to 131,072.

Products of M_Q, L_Q and B_I Lambda_V^-1 B_I^T against SciPy with the exported
matrices, tolerances as in the tests of shared slices (1e-13 and 1e-6); cycles
against the same cycle in FP64 at a batch of two, which never shares a slice:
the order of the sums of some ten products of rows of up to 200 entries is all
that differs, 1e-11."""

import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dim,n,p3", [(3, 35, False), (3, 36, False), (3, 39, False), (3, 40, False), (3, 50, False), (2, 168, False), (2, 169, False), (2, 220, False), (2, 221, False),
                                      (2, 110, True), (2, 111, True), (3, 18, True)])
def test_products_and_cycles(gpu_lib, dim, n, p3):
    from paper_2407_01783_amd.stokes import StokesProblem
    print(f"[case] dim={dim} n={n} p3={p3}", flush=True)
    P = StokesProblem(dim, n, mesh_seed=4, jitter=0.1, mu=0.02, alpha=50.0, p3=p3)
    x = np.random.default_rng(n).standard_normal(P.n_p1)
    t = torch.tensor(x, device="cuda")
    for op, which in ((3, 5), (4, 6), (7, 9)):
        rp, cols, vals = P.export_csr(which)
        want = sp.csr_matrix((vals, cols, rp), shape=(P.n_p1, P.n_p1)) @ x
        for precision, tol in ((0, 1e-13), (1, 1e-6)):
            y = P.apply(op, t, precision=precision).cpu().numpy().ravel()
            assert np.linalg.norm(y - want) <= tol * np.linalg.norm(want), (op, precision)
    for op in (6, 8):
        one = P.apply(op, t).ravel()
        two = P.apply(op, torch.stack([t, -t]), nrhs=2).reshape(2, -1)
        assert float((two[0] - one).norm()) <= 1e-11 * float(one.norm()), op
        assert float((two[1] + one).norm()) <= 1e-11 * float(one.norm()), op
