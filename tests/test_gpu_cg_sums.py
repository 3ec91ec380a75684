"""Inner velocity CG whose scalars are formed by the kernels that use them
(single right-hand sides of a few ten thousand rows) against the same solves in
a batch of eight, whose sums are launches of their own; the strain operator's
product inside the CG's with one, two and four wavefronts per slice.

Sizes: below and above the limit of the first form (2D: 90,601 rows below,
210,681 above; 3D: 103,823 below, 132,651 above), matrices small enough for a single-launch CG excluded by
STOKES_PCG_SMALL=0.  Both sides solve to a true relative residual of 1e-11, so
they agree to 1e-9 as in the tests of the single-launch CG."""

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dim,n,strain,precision,opts", [
    (2, 3, True, 0, {}), (2, 20, True, 1, {}), (2, 20, False, 0, {}), (2, 150, True, 1, {}), (2, 230, True, 1, {}),
    (3, 2, True, 0, {}), (3, 5, True, 1, {}), (3, 9, False, 0, {}), (3, 20, False, 1, {}), (3, 24, False, 1, {}), (3, 26, True, 1, {}), (3, 13, True, 0, {}),
    (2, 24, True, 0, {"method": "schur"}), (2, 12, True, 0, {"method": "schur", "gamma": 1.0}),
    (3, 4, False, 0, {"method": "schur", "gamma": 1.0})])
def test_single_equals_batch(gpu_lib, monkeypatch, dim, n, strain, precision, opts):
    from paper_2407_01783_amd import inputs
    from paper_2407_01783_amd.stokes import StokesProblem
    monkeypatch.setenv("STOKES_PCG_SMALL", "0")
    print(f"[case] dim={dim} n={n} strain={strain} precision={precision} {opts}", flush=True)
    opts = dict({"method": "coupled"}, **opts)
    P = StokesProblem(dim, n, mesh_seed=2, jitter=0.1, mu=0.05, alpha=100.0, strain=strain,
                      gamma=opts.pop("gamma", 0.0))
    xy = P.mesh()[0]
    f = torch.stack([torch.tensor(inputs.fourier_forcing(xy, 1002 + k % 2)) for k in range(8)]).cuda()
    kw = dict(rtol=1e-11, max_refine=20, precision=precision, **opts)
    both = P.solve(f, **kw)
    assert both[2]["status"] == 0
    for r in (0, 1):
        u, p, info = P.solve(f[r:r + 1].contiguous(), **kw)
        assert info["status"] == 0
        assert float((u[0] - both[0][r]).norm()) <= 1e-9 * float(u.norm())
        assert float((p[0] - both[1][r]).norm()) <= 1e-9 * float(p.norm())
        assert info["inner_iters_u"] <= both[2]["inner_iters_u"] + 4 * info["outer_iters"]
