"""Batched adjoints whose outputs lie on vectors that earlier systems have used
up.  The results are those of one system after the other, so every gradient
equals, bit for bit, the one computed with buffers of its own.
"""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SHAPE, N = (255, 127), 6
VEC = SHAPE[0] * SHAPE[1]


def _outputs(kind, zs, store):
    """gf[i]: z[i - 1] itself, one buffer for every system, or from the middle of
    z[i - 1] to the middle of z[i - 2] (z[0] lies last in the store)."""
    new = lambda: torch.empty_like(zs[0])
    if kind == "previous":
        return [new()] + zs[:-1]
    if kind == "one":
        return [new()] * N
    flat = store.reshape(-1)
    start = [(N - i) * VEC + VEC // 2 for i in range(N)]
    return [new(), new()] + [flat[start[i]:start[i] + VEC].reshape(SHAPE) for i in range(2, N)]


@pytest.mark.parametrize("summed", [True, False])
@pytest.mark.parametrize("kind", ["previous", "one", "overlap"])
def test_outputs_on_used_vectors(kind, summed):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_00488_amd as C
    print("adjoint outputs", kind, summed, flush=True)
    g = np.random.default_rng(11)
    cplx = lambda: torch.from_numpy(g.standard_normal(SHAPE) + 1j * g.standard_normal(SHAPE)).cuda()
    a = torch.from_numpy(g.uniform(0.5, 2.0, SHAPE)).cuda()
    probs = [C.Problem(a, 5.0 + k, 40.0 + k) for k in range(N)]
    b = C.Batch(probs, timeout_ms=30000)
    store = torch.empty((N,) + SHAPE, dtype=torch.complex128, device="cuda")
    zs = [store[N - 1 - i] for i in range(N)]
    for p, z in zip(probs, zs):
        C.minres_solve(p, cplx(), z)
    gzs = [cplx() for _ in range(N)]
    opts = C._solve_opts(1e-8, 1000, True, 30000)

    def adjoint(gf):
        out = [torch.zeros(N, dtype=torch.float64, device="cuda") for _ in range(2)]
        if summed:
            out.append(torch.zeros(SHAPE, dtype=torch.float64, device="cuda"))
        ptrs = lambda vs: (ctypes.c_void_p * N)(*[v.data_ptr() for v in vs])
        one = [ctypes.c_void_p(v.data_ptr()) for v in out] + [None] * (3 - len(out))
        st = C.load_library().batch_adjoint(b._h, ptrs(zs), ptrs(gzs), ptrs(gf), *one,
                                            ctypes.byref(opts), None, C._stream(b.device))
        torch.cuda.synchronize()
        assert st == 0
        return out

    own = [torch.empty_like(z) for z in zs]
    ref = adjoint(own)
    gf = _outputs(kind, zs, store)
    for u, v in zip(adjoint(gf), ref):
        assert torch.equal(u, v)
    # the last system's gradient stands; where none overlaps another, every one
    assert torch.equal(gf[N - 1], own[N - 1])
    if kind != "one":
        assert all(torch.equal(u, v) for u, v in zip(gf, own))
    b.close()
    for p in probs:
        p.close()
