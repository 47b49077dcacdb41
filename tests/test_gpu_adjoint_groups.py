"""Batched adjoints over more systems than one launch of the reductions takes,
with the summed coefficient gradient on one grid and without it on grids of both
dimensions and different sizes, against each system's own adjoint.

Tolerance 1e-9, the bar of the gradients: both sides solve to 1e-12.
"""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

GRIDS = {"one": [(15, 7)] * 19, "mixed": [(15, 7), (31, 15), (7, 31)] * 6 + [(7, 3, 7), (3, 7, 15), (7, 7)]}


@pytest.mark.parametrize("kind", ["one", "mixed"])
def test_groups(kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_00488_amd as C
    print("adjoint groups", kind, flush=True)
    g = np.random.default_rng(5)
    shapes, n = GRIDS[kind], len(GRIDS[kind])
    cplx = lambda sh: torch.from_numpy(g.standard_normal(sh) + 1j * g.standard_normal(sh)).cuda()
    probs = [C.Problem(torch.from_numpy(g.uniform(0.5, 2.0, sh)).cuda(), 5.0 + k, 40.0 + k)
             for k, sh in enumerate(shapes)]
    zs = [C.minres_solve(p, cplx(sh), tol=1e-12)[0] for p, sh in zip(probs, shapes)]
    gzs = [cplx(sh) for sh in shapes]
    b = C.Batch(probs, timeout_ms=30000)
    if kind == "one":
        out, _ = b.adjoint(zs, gzs, tol=1e-12)
        gf, alpha, beta, ga = out["f"], out["alpha"], out["beta"], out["a"]
    else:
        gf = [torch.empty_like(v) for v in gzs]
        alpha, beta = (torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(2))
        ptrs = lambda vs: (ctypes.c_void_p * n)(*[v.data_ptr() for v in vs])
        o = C._solve_opts(1e-12, 1000, True, 30000)
        st = C.load_library().batch_adjoint(
            b._h, ptrs(zs), ptrs(gzs), ptrs(gf), ctypes.c_void_p(alpha.data_ptr()),
            ctypes.c_void_p(beta.data_ptr()), None, ctypes.byref(o), None, C._stream(b.device))
        torch.cuda.synchronize()
        assert st == 0
    rel = lambda u, v: float((u - v).norm() / v.norm())
    ga_s = torch.zeros(shapes[0], dtype=torch.float64, device="cuda")
    for j, p in enumerate(probs):
        one, _ = C.minres_adjoint(p, zs[j], gzs[j], tol=1e-12, ga=ga_s if kind == "one" else None)
        assert rel(gf[j], one["f"]) <= 1e-9, j
        assert rel(alpha[j], one["alpha"]) <= 1e-9, j
        assert rel(beta[j], one["beta"]) <= 1e-9, j
    if kind == "one":
        assert rel(ga, ga_s) <= 1e-9
    b.close()
    for p in probs:
        p.close()
