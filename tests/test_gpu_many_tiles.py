"""Single solves of more than 1024 tiles a phase: flat ones whose workgroups own up
to sixteen tiles each, and one of more, whose tiles are all claimed.  Against a
schedule of few tiles, after the same number of steps; a second solve repeats
the bits (the tiles' sums are added in a fixed order, whoever forms them).

Rows of 127 points at 256 threads: 16 lines of 64 KiB, 1009 chunks; half as many
lines on 32 KiB, 2017.  255 x 255 x 127 at 512 threads: 65025 rows in rounds of 32,
2033.  The plane phase has two tiles for each point of the last axis, 2046.
255 x 255 x 15 in rounds of 8 rows: 8129 tiles on 256 workgroups.

Tolerances (relative 2-norm): 1e-10 in FP64 (the bar of the iterates); with the
FP32 preconditioner 1e-5, some 1e-7 of rounding in each of six applications
before convergence has damped it.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

CASES = [((127, 127, 127), False, (1, 32768, 256), (0, 0, 256)),
         ((127, 127, 127), True, (1, 32768, 256), (0, 0, 256)),
         ((255, 255, 127), False, (1, 0, 512), (0, 0, 512)),
         ((15, 15, 1023), True, (0, 0, 1024), (0, 0, 512)),
         ((15, 7, 1023), False, (0, 0, 1024), (0, 0, 512)),
         ((255, 255, 15), False, (1, 0, 512, 256), (0, 0, 512))]


@pytest.mark.parametrize("shape,fp32,many,few", CASES)
def test_against_few_tiles(shape, fp32, many, few):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_00488_amd as C
    print("many tiles", shape, fp32, many, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(shape))
    a = 1.0 + torch.rand(shape, generator=g, device="cuda", dtype=torch.float64)
    f = torch.view_as_complex(torch.randn(shape + (2,), generator=g, device="cuda", dtype=torch.float64))
    p = C.Problem(a, 10.0, 100.0, pinv_fp32=fp32, dst="fft",
                  tile_elems=many[3] if len(many) > 3 else 0)

    def solve(schedule):
        p.set_schedule(*schedule)
        z, info = C.minres_solve(p, f, maxit=6, tol=1e-30, timeout_ms=20000, raise_on_error=False)
        assert info["iters"] == 6, info
        return z

    z0, z1, z2 = solve(few), solve(many), solve(many)
    p.close()
    err = float((z1 - z0).norm() / z0.norm())
    print("  err", err, flush=True)
    assert torch.equal(z1, z2)
    assert err <= (1e-5 if fp32 else 1e-10)
