"""Iteration counts of the single-launch inner CG: those that ran, whatever the
interval at which the host would look at separate launches (STOKES_CG_CHECK).
With an interval of 50 the counts of separate launches are multiples of 50, so
they also tell which path a solve took: matrices in the LDS, matrices that
stream, the strain form, and meshes just past the limit.

The two paths sum in different orders, which may shift the last iteration of a
solve: one per velocity solve, two solves per outer iteration."""

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _count(monkeypatch, small, check, dim, n, precision, strain):
    from paper_2407_01783_amd import inputs
    from paper_2407_01783_amd.stokes import StokesProblem
    monkeypatch.setenv("STOKES_PCG_SMALL", str(small))
    monkeypatch.setenv("STOKES_CG_CHECK", str(check))
    print(f"[case] small={small} check={check} dim={dim} n={n} precision={precision} strain={strain}", flush=True)
    P = StokesProblem(dim, n, mesh_seed=2, jitter=0.1, mu=0.05, alpha=100.0, strain=strain)
    f = torch.tensor(inputs.fourier_forcing(P.mesh()[0], 1002)[None], device="cuda")
    info = P.solve(f, rtol=1e-9, max_refine=20, precision=precision)[2]
    assert info["status"] == 0
    return info["inner_iters_u"], info["outer_iters"]


@pytest.mark.parametrize("dim,n,precision,strain", [
    (2, 4, 0, False), (2, 16, 0, False), (2, 15, 1, True), (2, 22, 0, False), (2, 30, 1, False), (3, 4, 0, False),
    (3, 5, 1, False)])
def test_counts_that_ran(gpu_lib, monkeypatch, dim, n, precision, strain):
    one, outer = _count(monkeypatch, 1, 2, dim, n, precision, strain)
    assert _count(monkeypatch, 1, 50, dim, n, precision, strain) == (one, outer)
    apart, outer_apart = _count(monkeypatch, 0, 1, dim, n, precision, strain)
    assert outer == outer_apart and abs(one - apart) <= 2 * outer


@pytest.mark.parametrize("dim,n,precision,strain", [(2, 32, 0, False), (2, 48, 1, False), (3, 8, 0, False), (3, 9, 1, True)])
def test_larger_systems_take_launches(gpu_lib, monkeypatch, dim, n, precision, strain):
    count, _ = _count(monkeypatch, 1, 50, dim, n, precision, strain)
    assert count % 50 == 0
