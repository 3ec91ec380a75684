"""What the dense inverse of a coarsest level holds: the hierarchy and the
precision that a solve used, nothing at assembly; and solves without the
memory for it (STOKES_DENSE_MB), which fall back to the polynomial.

2D n = 93 is the largest level that is inverted (8,836 rows: 313 MB in FP32,
625 in FP64); everything else that a context and a solve of that mesh hold is
some tens of MB (76,000 unknowns times 100 vectors, 16 entries of 8 bytes a
row), so 200 MB are allowed for it."""

import gc

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _problem(dim, n):
    from paper_2407_01783_amd import inputs
    from paper_2407_01783_amd.stokes import StokesProblem
    print(f"[case] dim={dim} n={n}", flush=True)
    P = StokesProblem(dim, n, mesh_seed=3, jitter=0.1, mu=0.02, alpha=50.0)
    f = torch.tensor(inputs.fourier_forcing(P.mesh()[0], 1003)[None], device="cuda")
    return P, f


def test_only_what_is_used_is_held(gpu_lib):
    torch.zeros(1, device="cuda")
    _problem(2, 4)  # code objects and per-device scratch
    gc.collect()
    torch.cuda.synchronize()
    start = torch.cuda.mem_get_info()[0]

    def held():
        torch.cuda.synchronize()
        return (start - torch.cuda.mem_get_info()[0]) / 1e6

    P, f = _problem(2, 93)
    seen = [held()]
    for precision in (1, 0):
        info = P.solve(f, rtol=1e-9, max_refine=20, precision=precision, inner_mode=1, coupled_pc=1, cheb_degree=6)[2]
        assert info["status"] == 0
        seen.append(held())
    print("held, MB: assembled %.0f, mixed %.0f, both %.0f" % tuple(seen), flush=True)
    assert seen[0] <= 200 and seen[1] <= 200 + 313 and seen[2] <= 200 + 313 + 625


@pytest.mark.parametrize("dim,n,opts", [(2, 63, {}), (2, 63, {"inner_mode": 1}), (3, 9, {}), (3, 32, {"inner_mode": 1}),
                                        (3, 16, {"vel_pc": 1}), (2, 40, {"precision": 0})])
def test_without_the_memory(gpu_lib, monkeypatch, dim, n, opts):
    kw = dict(dict(rtol=1e-9, max_refine=20, max_outer=500, precision=1), **opts)
    P, f = _problem(dim, n)
    u, p, _ = P.solve(f, **kw)
    monkeypatch.setenv("STOKES_DENSE_MB", "0")
    Q, _ = _problem(dim, n)
    v, q, info = Q.solve(f, **kw)
    assert info["status"] == 0
    # both to a residual of 1e-9 on operators of condition numbers up to 1e4
    assert float((u - v).norm()) <= 1e-5 * float(u.norm())
    assert float((p - q).norm()) <= 1e-5 * float(p.norm())
    x = torch.randn(P.n_p1, dtype=torch.float64, device="cuda")
    assert not torch.equal(P.apply(8, x), Q.apply(8, x))  # the polynomial in place of the inverse
