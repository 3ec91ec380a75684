"""The pressure V-cycle M is symmetric, as the conjugate gradients that it
preconditions assume: M_ij = M_ji for neighbouring nodes, on hierarchies of
two and three levels.

Bound: the stored values of a level are symmetric in every precision, so only
the order of the roundings differs.  An entry is a sum of some tens of
products of either sign whose parts are no larger than the diagonal; with
random signs their roundings add up to a few units, so 16 (FP64: 2^-49, FP32:
2^-20 of sqrt(M_ii M_jj)) are out of reach, while an entry-by-entry half
rounding that is not symmetric (2^-12 a value, weighed by the part of the
cycle that uses it) is not."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dim,n,p3", [(2, 80, False), (2, 150, False), (3, 18, False), (3, 36, False), (2, 40, True),
                                      (3, 12, True)])
@pytest.mark.parametrize("op", [6, 8])
def test_cycle_is_symmetric(gpu_lib, dim, n, p3, op):
    from paper_2407_01783_amd.stokes import StokesProblem
    print(f"[case] dim={dim} n={n} p3={p3} op={op}", flush=True)
    P = StokesProblem(dim, n, mesh_seed=5, jitter=0.2, mu=0.01, alpha=100.0, p3=p3)
    m = (2 if p3 else 1) * n + 1
    corners = np.indices((2,) * dim).reshape(dim, -1)  # of a cell
    for precision, tol in ((0, 2.0 ** -49), (1, 2.0 ** -20)):
        worst = 0.0
        for cell in (m // 2, m // 3, m // 4 + 1):
            ids = ((corners + cell) * (m ** np.arange(dim))[:, None]).sum(0)
            M = np.empty((len(ids), len(ids)))
            for j, node in enumerate(ids):
                e = torch.zeros(P.n_p1, dtype=torch.float64, device="cuda")
                e[node] = 1.0
                M[:, j] = P.apply(op, e, precision=precision).ravel()[torch.from_numpy(ids).cuda()].cpu().numpy()
            d = np.sqrt(np.diag(M))
            worst = max(worst, np.abs((M - M.T) / np.outer(d, d)).max())
        print(f"  precision {precision}: {worst:.2e} of at most {tol:.2e}", flush=True)
        assert worst <= tol, precision
