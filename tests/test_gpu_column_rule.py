"""FP32 batches whose default column kernel depends on the number of rounds, on
the block of sites an XCD covers and on the kind of launch (operator, step of a
polynomial): the default against the blocked kernel and both column kernels,
bit for bit (marked gpu).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_00016_amd import inputs, mpmc  # noqa: E402


@pytest.mark.parametrize("dims,N", [
    ((12, 12, 12, 6), 64),       # one round, no larger block: 2x2x2 for both
    ((12, 12, 12, 6), 128),      # second round only: operator 2x2x4, steps 2x2x2
    ((16, 16, 8, 6), 64),        # larger block only: the same
    ((16, 16, 8, 6), 128),       # both: 2x2x4 for both
    ((16, 16, 8, 6), 192)])      # three rounds: 2x2x2 for both
def test_default_matches_every_kernel(dims, N):
    ctx = mpmc.Context(dims, 0.12, inputs.gauge_links(dims, 0.5, seed=8))
    x = ctx.noise(7, 1, 0, N, mpmc.FP32)
    roots = 1.0 + 0.4 * np.exp(2j * np.pi * np.arange(5) / 5 + 0.3j)
    P = [ctx.poly_from_roots(roots[:d]) for d in (2, 5)]
    calls = [lambda: ctx.apply_M(x, N, mpmc.FP32, dagger=True, theta=1)] + \
            [lambda p=p: ctx.apply_poly(p, x, N, mpmc.FP32, out=torch.full_like(x, 255)) for p in P]
    want = [f() for f in calls]
    for v in (5, 10, 12):
        ctx.tune_set(N, mpmc.FP32, v)
        assert all(torch.equal(f(), w) for f, w in zip(calls, want)), v
