"""GPU parity of the 512-thread solver's team phases on 3-D grids with 511 or 1023
points along axis 0 or 1, where a team is a whole wave or two and the lines of
axis 0 are read and written by the workgroup, in both preconditioner precisions,
against the oracle's iterate after the same number of steps.

Tolerances (relative 2-norm): 1e-10 in FP64 (the bar of the iterates); with the
FP32 preconditioner 1e-5, some 1e-7 of rounding in each of six applications
before convergence has damped it.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import csl_oracle as O

pytestmark = pytest.mark.gpu

SHAPES = [(511, 7, 3), (3, 511, 7), (1023, 3, 7), (1023, 15, 3), (3, 1023, 7), (7, 1023, 3)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("fp32", [False, True])
def test_iterate(shape, fp32):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_00488_amd as C
    print("team phases, long lines", shape, fp32, flush=True)
    g = np.random.default_rng(sum(shape))
    a = g.uniform(1.0, 2.0, shape)
    f = g.standard_normal(shape) + 1j * g.standard_normal(shape)
    alpha, beta = 10.0, 400.0
    p = C.Problem(torch.from_numpy(a).cuda(), alpha, beta, pinv_fp32=fp32, dst="fft")
    p.set_schedule(0, 0, 512)
    po = O.Problem(a, alpha, beta)
    ft = torch.from_numpy(f).cuda()
    for k in (1, 6):
        z, info = C.minres_solve(p, ft, maxit=k, tol=1e-30, timeout_ms=20000, raise_on_error=False)
        assert info["iters"] == k, info
        zo, _ = po.solve(f, fixed_iters=k)
        err = np.linalg.norm(z.cpu().numpy() - zo) / np.linalg.norm(zo)
        print("  steps", k, "err", err, flush=True)
        assert err <= (1e-5 if fp32 else 1e-10)
    p.close()
