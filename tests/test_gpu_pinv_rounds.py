"""Stand-alone P^{-1} in FP64 on grids whose passes have more rounds than the GPU
has CUs (about 500 and more; the test asserts it for every pass), so that a
workgroup walks several rounds, loads one while it transforms another and reuses
its lines, with a ragged last round; in place as well.  Against SciPy's
orthonormal DST-I.

Tolerance (relative 2-norm): 4e-15.  An FFT of the odd extension of 1023 points
is off by 4e-16 in rms; two of them along three axes give 1e-15 and as much again
is left for the eigenvalues and the factors, on either side of the comparison.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SHAPES = [(127, 127, 127), (255, 63, 127), (63, 127, 255), (31, 63, 1023), (1023, 31, 63)]


def _rounds(shape):
    """Rounds of the passes along axes 2, 1 and 0: lines of n points are taken
    512 / ((n + 1) / 8) at a time, at most 64; those of axis 0 in groups of
    neighbours along axis 1."""
    n0, n1, n2 = shape
    held = lambda n: min(64, 512 // ((n + 1) // 8))
    return (-(-n0 * n1 // held(n2)), -(-n0 * n2 // held(n1)), n2 * -(-n1 // held(n0)))


@pytest.mark.parametrize("shape", SHAPES)
def test_several_rounds(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from scipy import fft
    import paper_2408_00488_amd as C
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    print("P^-1 rounds", shape, _rounds(shape), "CUs", cus, flush=True)
    assert min(_rounds(shape)) > cus
    g = np.random.default_rng(sum(shape))
    a = g.uniform(1.0, 2.0, shape)
    f = g.standard_normal(shape) + 1j * g.standard_normal(shape)
    alpha, beta = 10.0, 100.0
    p = C.Problem(torch.from_numpy(a).cuda(), alpha, beta, dst="fft")
    x = torch.from_numpy(f).cuda()
    z = C.apply_Pinv(p, x)
    C.apply_Pinv(p, x, x)   # in place
    p.close()

    lam = 0.0
    for ax, n in enumerate(shape):
        mu = (2 * (n + 1) * np.sin(np.pi * np.arange(1, n + 1) / (2 * n + 2))) ** 2
        lam = lam + mu.reshape([-1 if k == ax else 1 for k in range(3)])
    s = 1.0 / np.sqrt((a.mean() * lam + alpha) ** 2 + beta ** 2)
    dst = lambda v: fft.dstn(v, type=1, norm="ortho")
    zo = dst(dst(f.real) * s) + 1j * dst(dst(f.imag) * s)
    for y in (z, x):
        err = float(np.linalg.norm(y.cpu().numpy() - zo) / np.linalg.norm(zo))
        print("  err", err, flush=True)
        assert err <= 4e-15
