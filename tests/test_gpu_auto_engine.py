"""The automatic engine choice: a problem's own solves take the faster of the FFT
and the matrix cores, its batches the FFT unless the matrix cores are faster by
far, and a workgroup size that needs the FFT is accepted and takes it.

15 x 15 x 255 is a grid whose short axes are faster on the matrix cores (by about a
sixth); the automatic solve may take 8% longer than the faster forced one, half
of that.  Iterates: 1e-10 (relative 2-norm) between engines after six steps.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SHAPE = (15, 15, 255)


@pytest.fixture(scope="module")
def csl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_00488_amd as C
    C.load_library()
    return C


def _inputs():
    g = np.random.default_rng(4)
    a = torch.from_numpy(g.uniform(1.0, 2.0, SHAPE)).cuda()
    return a, torch.from_numpy(g.standard_normal(SHAPE) + 1j * g.standard_normal(SHAPE)).cuda()


def _time(csl, p, f):
    """Shortest of ten solves of 30 steps, in ms."""
    best = float("inf")
    z = torch.empty_like(f)
    for _ in range(12):
        e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        e0.record()
        csl.minres_solve(p, f, z, tol=1e-30, maxit=30, timeout_ms=20000, want_info=False)
        e1.record()
        e1.synchronize()
        best = min(best, e0.elapsed_time(e1))
    return best


@pytest.mark.parametrize("fp32", [False, True])
def test_own_solves_take_the_faster(csl, fp32):
    a, f = _inputs()
    ms = {}
    for dst in ("auto", "fft", "gemm"):
        p = csl.Problem(a, 10.0, 100.0, pinv_fp32=fp32, dst=dst)
        ms[dst] = _time(csl, p, f)
        print(dst, p.dst_engines, p.schedule["block_threads"], ms[dst], flush=True)
        p.close()
    assert ms["auto"] <= 1.08 * min(ms["fft"], ms["gemm"])


def test_fft_where_a_workgroup_size_needs_it(csl):
    a, f = _inputs()
    step = lambda p: csl.minres_solve(p, f, tol=1e-30, maxit=6, timeout_ms=20000, raise_on_error=False)[0]
    p = csl.Problem(a, 10.0, 100.0)
    q = csl.Problem(a, 10.0, 100.0, dst="fft")
    own = p.dst_engines
    print("engines", own, flush=True)
    z = step(p)
    for threads in (512, 1024):
        for v in (p, q):
            v.set_schedule(0, 0, threads)
            assert v.dst_engines == ("fft",) * 3 and v.schedule["block_threads"] == threads
        assert torch.equal(step(p), step(q))
    assert float((step(p) - z).norm() / z.norm()) <= 1e-10
    c = p.clone()
    assert c.schedule == p.schedule and torch.equal(step(c), step(p))
    c.close()
    # back to the default schedule: the engines of its own solves again
    p.set_schedule(0, 0, 0)
    assert p.dst_engines == own and torch.equal(step(p), z)
    b = csl.Batch([p, q], tol=1e-30, maxit=6, timeout_ms=20000)
    assert b.schedule["block_threads"] == 512
    zs, _ = b.solve([f, f.clone()], raise_on_error=False)
    assert torch.equal(zs[0], zs[1])
    b.close()
    # the tuner starts from the schedule in force, whatever engines it runs
    p.set_schedule(0, 0, 512)
    t = p.tune(f)
    assert t["ms"] <= t["ms_default"]
    step(p)
    for v in (p, q):
        v.close()
