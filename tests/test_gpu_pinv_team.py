"""Stand-alone P^{-1} in FP64 through the team passes, where their tiling and
their transforms can go wrong: lines of 3 to 1023 points along each axis,
rounds of eight lines and of a workgroup's, several rounds a workgroup and a
ragged last one, in place as well; against dense sine matrices in extended
precision.

Tolerance (relative 2-norm): 2e-15.  An FFT of the odd extension of 1023 points
is off by 4e-16 in rms; two of them along up to three axes give 1e-15, and as
much again is left for the eigenvalues and the factors.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SHAPES = [(3, 3), (3, 63), (127, 3), (7, 7), (15, 1023), (1023, 15), (63, 511), (511, 127), (255, 255),
          (3, 3, 3), (3, 7, 31), (31, 3, 7), (7, 255, 3), (3, 7, 1023), (511, 3, 15), (15, 127, 31),
          (63, 31, 63)]


@pytest.mark.parametrize("shape", SHAPES)
def test_pinv(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_00488_amd as C
    print("team P^-1", shape, flush=True)
    g = np.random.default_rng(sum(shape))
    a = g.uniform(1.0, 2.0, shape)
    f = g.standard_normal(shape) + 1j * g.standard_normal(shape)
    alpha, beta = 10.0, 100.0
    p = C.Problem(torch.from_numpy(a).cuda(), alpha, beta, dst="fft")
    x = torch.from_numpy(f).cuda()
    z = C.apply_Pinv(p, x)
    C.apply_Pinv(p, x, x)   # in place
    p.close()

    L = np.longdouble
    pi = L("3.14159265358979323846264338327950288")
    v = f.astype(np.clongdouble)
    lam = L(0)
    W = []
    for ax, n in enumerate(shape):
        m = np.arange(1, n + 1)
        W.append(np.sin(pi * (np.outer(m, m) % (2 * n + 2)).astype(L) / (n + 1)) * np.sqrt(L(2) / (n + 1)))
        mu = (2 * (n + 1) * np.sin(pi * m.astype(L) / (2 * n + 2))) ** 2
        lam = lam + mu.reshape([-1 if k == ax else 1 for k in range(len(shape))])

    def transform(u):
        for ax, w in enumerate(W):
            u = np.moveaxis(np.tensordot(w, u, axes=(1, ax)), 0, ax)
        return u

    zo = transform(transform(v) / np.sqrt((L(a.mean()) * lam + alpha) ** 2 + L(beta) ** 2))
    for y in (z, x):
        err = float(np.linalg.norm((y.cpu().numpy() - zo).astype(complex)) / np.linalg.norm(zo.astype(complex)))
        print("  err", err, flush=True)
        assert err <= 2e-15
