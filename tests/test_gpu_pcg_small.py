"""Inner velocity CG of a small system in one launch against the same CG in
separate launches (STOKES_PCG_SMALL=0): the arithmetic of an iteration is the
same up to the order of the sums.

Sizes: one interior node, less than one 64-row slice, matrices that stay in
the LDS and matrices that stream, up to the largest meshes that take the path;
both precisions, the strain form, degree 1 (Jacobi), fixed iteration counts.
Tolerances: solutions solved to a true relative residual of 1e-11 agree to
1e-9; the iteration counts agree."""

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _solve(monkeypatch, small, dim, n, strain, method="coupled", **opts):
    from paper_2407_01783_amd import inputs
    from paper_2407_01783_amd.stokes import StokesProblem
    monkeypatch.setenv("STOKES_PCG_SMALL", "1" if small else "0")
    print(f"[case] small={small} dim={dim} n={n} strain={strain} {method} {opts}", flush=True)
    P = StokesProblem(dim, n, mesh_seed=2, jitter=0.1, mu=0.05, alpha=100.0, strain=strain)
    f = torch.tensor(inputs.fourier_forcing(P.mesh()[0], 1002)[None], device="cuda")
    u, p, info = P.solve(f, method=method, rtol=1e-11, max_refine=20, **opts)
    assert info["status"] == 0
    return u, p, info


@pytest.mark.parametrize("dim,n,strain,precision,opts", [
    (2, 2, False, 0, {}), (2, 4, False, 1, {}), (2, 5, True, 0, {}), (2, 16, False, 0, {}), (2, 17, False, 0, {}),
    (2, 24, False, 0, {}), (2, 33, False, 1, {}), (2, 15, True, 1, {}), (3, 2, False, 0, {}), (3, 3, True, 1, {}),
    (3, 4, False, 0, {}), (3, 5, False, 1, {}), (3, 6, False, 1, {}), (2, 9, False, 0, {"cheb_degree": 1}),
    (2, 20, False, 1, {"cheb_degree": 2}), (3, 4, False, 0, {"cheb_degree": 16}), (2, 12, False, 0, {"inner_its_u": 5}),
    (3, 3, False, 0, {"method": "schur"})])
def test_one_launch_equals_separate_launches(gpu_lib, monkeypatch, dim, n, strain, precision, opts):
    a = _solve(monkeypatch, True, dim, n, strain, precision=precision, **opts)
    b = _solve(monkeypatch, False, dim, n, strain, precision=precision, **opts)
    for x, y in zip(a[:2], b[:2]):
        assert float((x - y).norm()) <= 1e-9 * max(float(y.norm()), 1e-300)
    assert a[2]["outer_iters"] == b[2]["outer_iters"]
    assert abs(a[2]["inner_iters_u"] - b[2]["inner_iters_u"]) <= 2 * a[2]["outer_iters"]


def test_one_launch_is_reproducible(gpu_lib, monkeypatch):
    a = _solve(monkeypatch, True, 2, 16, False, precision=0)
    b = _solve(monkeypatch, True, 2, 16, False, precision=0)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
