"""FP64 column kernel (variant 11, fused-step order 6) on shapes that fill the
chip with its workgroups, one of them with an odd z extent and ragged blocks:
bit for bit the blocked kernel's operator, the blocked fused step's samples up
to the grouping of the FP64 sums (1e-13), and the oracle on sampled right-hand
sides (operator 1e-13, samples 1e-10, the parity bounds) (marked gpu).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import estimator as OES  # noqa: E402
from oracle import krylov as OK  # noqa: E402
from oracle.philox import z4_noise, z4_noise_batch  # noqa: E402
from oracle.wilson import WilsonOp, gamma5  # noqa: E402
from paper_2402_00016_amd import inputs, mpmc  # noqa: E402

FP64 = mpmc.FP64


@pytest.mark.parametrize("dims,N", [((8, 8, 8, 4), 128), ((12, 8, 10, 4), 64), ((16, 8, 9, 6), 256)])
def test_column_matches_blocked(dims, N):
    U = inputs.gauge_links(dims, 0.5, seed=8)
    op, ctx = WilsonOp(dims, 0.12, U), mpmc.Context(dims, 0.12, U)
    assert ctx.autotune(N, FP64)[1][11] > 0      # the shape takes the kernel
    ctx.tune_set(N, FP64, -1)
    x = ctx.noise(7, 1, 0, N, FP64)
    X = z4_noise_batch(7, 1, 0, N, op.n)[[0, N - 1]]
    for dagger, theta in ((False, 0), (True, 0), (False, 1)):
        y = ctx.apply_M(x, N, FP64, dagger=dagger, theta=theta)
        ctx.tune_set(N, FP64, 4)
        assert torch.equal(y, ctx.apply_M(x, N, FP64, dagger=dagger, theta=theta)), (dagger, theta)
        ctx.tune_set(N, FP64, -1)
        ref = op.dagger(X) if dagger else op(X)
        ref = gamma5(ref) if theta else ref
        got = ctx.unpack(y, N)[[0, N - 1]].cpu().numpy()
        assert np.linalg.norm(got - ref) < 1e-13 * np.linalg.norm(ref)
    P1, _, _ = OK.gmres_poly(op, z4_noise(1, 0x100, 0, op.n), 9)
    single = ctx.poly_from_roots(P1.roots)
    double = ctx.poly_from_roots(np.array([1.1, 0.9 + 0.1j, 1.0 - 0.1j]), inner=ctx.poly_from_roots(P1.roots[:3]))
    for P in (single, double):       # the double polynomial takes the combining steps
        X1 = ctx.level(P, None, None, 1, 5, 1, 0, N)[0]
        assert np.array_equal(X1, ctx.level(P, None, None, 1, 5, 1, 0, N)[0])
        ctx.tune_set(N, FP64, 4)
        X0 = ctx.level(P, None, None, 1, 5, 1, 0, N)[0]
        ctx.tune_set(N, FP64, -1)
        assert np.linalg.norm(X1 - X0) < 1e-13 * np.linalg.norm(X0)
        if P is single:
            Xr, _ = OES.level_samples(op, P1, None, None, "g5", 5, 1, 0, 2)
            assert np.linalg.norm(X1[:2] - Xr) < 1e-10 * np.linalg.norm(Xr)
    # polynomial application: additive operand and accumulator of the plain form
    y1 = ctx.apply_poly(single, x, N, FP64)
    ctx.tune_set(N, FP64, 4)
    assert torch.equal(y1, ctx.apply_poly(single, x, N, FP64))
