"""The 512-thread solver's face coefficients where samples differ widely:
isolated nodes of 1e200 among samples near 1 (every face at one is 2, every
other near 1), in 2-D and 3-D, against the oracle's iterate.

Tolerance 1e-10 (relative 2-norm), the bar of the FP64 iterates.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import csl_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(31, 63), (15, 31, 7)])
def test_samples_far_apart(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_00488_amd as C
    print("team coefficients", shape, flush=True)
    g = np.random.default_rng(sum(shape))
    a = g.uniform(0.9, 1.1, shape)
    # no two next to each other or at the boundary, where a face would be 1e200
    sub = a[tuple(slice(1, n - 1, 2) for n in shape)]
    sub[g.uniform(size=sub.shape) < 0.5] = 1e200
    f = g.standard_normal(shape) + 1j * g.standard_normal(shape)
    p = C.Problem(torch.from_numpy(a).cuda(), 10.0, 40.0, abar_rule="given", abar=1.3, dst="fft")
    p.set_schedule(0, 0, 512)
    z, info = C.minres_solve(p, torch.from_numpy(f).cuda(), maxit=12, tol=1e-30, raise_on_error=False)
    p.close()
    po = O.Problem(a, 10.0, 40.0, abar_rule="given", abar=1.3)
    zo, _ = po.solve(f, fixed_iters=info["iters"])
    err = np.linalg.norm(z.cpu().numpy() - zo) / np.linalg.norm(zo)
    print("  steps", info["iters"], "err", err, flush=True)
    assert info["iters"] == 12 and err <= 1e-10
