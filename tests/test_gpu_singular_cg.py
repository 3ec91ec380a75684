"""Pressure CG in FP32 on operators that are singular on constants (the
Laplacian of a projection step, the Cahouet-Chabard operators of a coupled
solve), preconditioned by V-cycles that are largest on constants: it must not
break down on the rounding of a mean.

The meshes are 2D ones whose constants weigh most (many pressure nodes), with
coarsest levels of 1,296 to 8,100 rows.  A step solves each of its systems to a
true relative residual of 1e-11 (1e-10 for the coupled solve) in either
precision; with condition numbers of at most 1e5 the two answers agree to
2e-6 (2e-5)."""

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _data(n, seed, k):
    from paper_2407_01783_amd import inputs
    from paper_2407_01783_amd.stokes import StokesProblem
    P = StokesProblem(2, n, mesh_seed=seed, jitter=0.1, mu=1e-3, alpha=200.0)
    f = torch.tensor(inputs.fourier_forcing(P.mesh()[0], 1002 + k + 7 * seed)[None], device="cuda")
    return P, f


@pytest.mark.parametrize("n,seed", [(70, 1), (100, 1), (100, 2), (140, 2), (150, 1), (220, 1), (252, 1), (300, 1), (300, 2),
                                    (340, 2), (356, 1), (360, 1)])
def test_projection_step(gpu_lib, n, seed):
    for k in (0, 1, 2):
        P, f = _data(n, seed, k)
        print(f"[case] projection n={n} seed={seed} forcing={k}", flush=True)
        kw = dict(rtol=1e-11, max_refine=30, max_inner=5000)
        u, p, info = P.projection_step(f, precision=1, **kw)
        v, q, ref = P.projection_step(f, precision=0, **kw)
        assert info["status"] == 0 and ref["status"] == 0
        assert float((u - v).norm()) <= 2e-6 * float(v.norm())
        assert float((p - q).norm()) <= 2e-6 * float(q.norm())


@pytest.mark.parametrize("n,seed,schur_pc", [(300, 1, 0), (340, 2, 0), (360, 1, 0), (320, 1, 1), (340, 2, 1), (40, 1, 2)])
def test_coupled_solve(gpu_lib, n, seed, schur_pc):
    for k in (0, 1, 2):
        P, f = _data(n, seed, k)
        print(f"[case] coupled n={n} seed={seed} forcing={k} schur_pc={schur_pc}", flush=True)
        kw = dict(rtol=1e-10, max_refine=30, max_inner=5000, max_outer=300, schur_pc=schur_pc)
        u, p, info = P.solve(f, precision=1, **kw)
        assert info["status"] == 0
        assert P.residual(f, u, p).max() <= 1.01e-10
        if n <= 300:
            v, q, _ = P.solve(f, precision=0, **kw)
            assert float((u - v).norm()) <= 2e-5 * float(v.norm())
            assert float((p - q).norm()) <= 2e-5 * float(q.norm())
