"""Tolerance-driven velocity CG under a forced number of lanes per row
(STOKES_LANES) that does not divide the width, where the kernels fall back to
the largest compiled number that does: the sums of an iteration are read from
as many workgroups as wrote them.

One context solves eight right-hand sides and then one, two and four, so that
partial sums of a wider batch lie in the scratch array, against a context that
picks its lanes itself.  Widths 2, 3 and 4 form their scalars where they are
used, 6, 8, 12 and 16 in launches of their own; the last 3D mesh is above the
limit of the first form at width 3 (132,651 rows).  Both sides solve to a true
relative residual of 1e-11, so they agree to 1e-9 as in the tests of the
single-launch CG; the host looks at the residual every second iteration, so the
counts may differ by one look in each of the two inner solves of a step."""

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dim,n,precision,lanes,strain", [
    (2, 12, 0, 8, False), (2, 40, 1, 8, False), (2, 40, 1, 4, True), (3, 5, 0, 2, False), (3, 9, 0, 8, False),
    (3, 9, 1, 4, False), (3, 9, 1, 8, True), (3, 24, 1, 8, False), (3, 26, 1, 2, False)])
def test_sums_follow_the_launched_lanes(gpu_lib, monkeypatch, dim, n, precision, lanes, strain):
    from paper_2407_01783_amd import inputs
    from paper_2407_01783_amd.stokes import StokesProblem
    monkeypatch.setenv("STOKES_PCG_SMALL", "0")
    print(f"[case] dim={dim} n={n} precision={precision} lanes={lanes} strain={strain}", flush=True)
    kw = dict(mesh_seed=2, jitter=0.1, mu=0.05, alpha=100.0, strain=strain)
    own = StokesProblem(dim, n, **kw)
    monkeypatch.setenv("STOKES_LANES", str(lanes))
    forced = StokesProblem(dim, n, **kw)
    xy = own.mesh()[0]
    f = torch.stack([torch.tensor(inputs.fourier_forcing(xy, 1002 + k)) for k in range(8)]).cuda()
    for nrhs in (8, 1, 2, 4):
        a, b = (P.solve(f[:nrhs].contiguous(), rtol=1e-11, max_refine=20, precision=precision) for P in (forced, own))
        assert a[2]["status"] == 0 and b[2]["status"] == 0
        for x, y in zip(a[:2], b[:2]):
            assert float((x - y).norm()) <= 1e-9 * float(y.norm()), nrhs
        assert abs(a[2]["inner_iters_u"] - b[2]["inner_iters_u"]) <= 4 * b[2]["outer_iters"], nrhs
