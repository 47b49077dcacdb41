"""GPU parity of the 512-thread solver's team phases (a line per team of lanes)
where their tiling can go wrong: teams of one lane up to more than a wave,
rounds of one line and of a workgroup's lines, several rounds per tile with a
ragged last one, in both preconditioner precisions, against the oracle's
iterate after the same number of steps.

Tolerances (relative 2-norm): 1e-10 in FP64 (the bar of the iterates); with
the FP32 preconditioner 1e-5, some 1e-7 of rounding in each of six
applications before convergence has damped it.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import csl_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def csl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_00488_amd as C
    C.load_library()
    return C


# (shape, tile_points, tile_elems): tile_points 0 is about one tile per
# workgroup, tile_elems sets the lines of a round
CASES = [((3, 7), 0, 0), ((7, 3), 0, 0), ((7, 7), 0, 0), ((15, 7), 0, 0), ((31, 15), 0, 0),
         ((31, 63), 0, 512), ((63, 31), 1000, 0), ((127, 127), 5000, 0), ((255, 63), 0, 1024),
         ((255, 127), 9000, 0), ((63, 511), 0, 0), ((511, 255), 20000, 0), ((7, 1023), 0, 0),
         ((1023, 15), 12000, 0),
         ((3, 7, 15), 0, 0), ((7, 3, 31), 0, 0), ((15, 31, 7), 600, 0), ((31, 7, 63), 0, 512),
         ((63, 15, 31), 7000, 0), ((7, 127, 15), 3000, 0), ((3, 255, 7), 0, 0), ((127, 7, 3), 0, 0)]


@pytest.mark.parametrize("shape,points,elems", CASES)
@pytest.mark.parametrize("fp32", [False, True])
def test_iterate(csl, shape, points, elems, fp32):
    print("team phases", shape, points, elems, fp32, flush=True)
    g = np.random.default_rng(sum(shape) + points + elems)
    a = g.uniform(1.0, 2.0, shape)
    f = g.standard_normal(shape) + 1j * g.standard_normal(shape)
    lam = 10.0 + 40.0j
    p = csl.Problem(torch.from_numpy(a).cuda(), lam.real, lam.imag, pinv_fp32=fp32, dst="fft")
    p.set_schedule(points, 0, 512, elems)
    po = O.Problem(a, lam.real, lam.imag)
    ft = torch.from_numpy(f).cuda()
    for k in (1, 6):   # one step applies the update alone, six in pairs
        z, info = csl.minres_solve(p, ft, maxit=k, tol=1e-30, raise_on_error=False)
        zo, _ = po.solve(f, fixed_iters=info["iters"])
        err = np.linalg.norm(z.cpu().numpy() - zo) / np.linalg.norm(zo)
        print("  steps", info["iters"], "err", err, flush=True)
        assert err <= (1e-5 if fp32 else 1e-10)
    p.close()
