"""A batch of one system, which runs in the kernel of a single system but claims
its tiles, against the problem's own solve on the same workgroup size, on every
solver instance; its graph replays to the same bits.

Tolerance 1e-9 (relative 2-norm), the bar of the converged FP64 solutions; 1e-7
with the FP32 preconditioner, whose rounding reaches the iterates of two tilings
through the stopping test at 1e-8.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

CASES = [((63, 127), False, "fft", 512), ((63, 127), True, "fft", 256), ((31, 15, 63), False, "fft", 512),
         ((31, 31, 63), True, "fft", 1024), ((31, 31, 63), False, "fft", 1024), ((40, 63), False, "auto", 256),
         ((40, 63), True, "gemm16", 256)]


@pytest.mark.parametrize("shape,fp32,dst,threads", CASES)
def test_batch_of_one(shape, fp32, dst, threads):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_00488_amd as C
    print("batch of one", shape, fp32, dst, threads, flush=True)
    g = np.random.default_rng(sum(shape))
    a = torch.from_numpy(g.uniform(1.0, 2.0, shape)).cuda()
    f = torch.from_numpy(g.standard_normal(shape) + 1j * g.standard_normal(shape)).cuda()
    p = C.Problem(a, 10.0, 100.0, pinv_fp32=fp32, dst=dst)
    p.set_schedule(0, 0, threads)
    z, info = C.minres_solve(p, f, timeout_ms=20000)
    b = C.Batch([p], timeout_ms=20000, block_threads=threads)
    (z1,), (i1,) = b.solve([f])
    (z2,), (i2,) = b.solve([f])
    b.close()
    p.close()
    assert i1["status"] == 0 and i1 == i2 and torch.equal(z1, z2)
    assert abs(i1["iters"] - info["iters"]) <= 1
    err = float((z1 - z).norm() / z.norm())
    print("  steps", info["iters"], i1["iters"], "err", err, flush=True)
    if i1["iters"] == info["iters"]:
        assert err <= (1e-7 if fp32 else 1e-9)
