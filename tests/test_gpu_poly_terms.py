"""Polynomial application: the sum takes two terms in every other step, the
first step starts it and the last one stores no vector.  Every kernel that
carries the sum, at degrees that end on a paired and on a single term, against
the same recurrence formed from operator applications in complex128 (roundings
of at most six steps: 1e-13 in FP64, 5e-6 in FP32 of the norm), into an output
that holds NaN (marked gpu).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_00016_amd import inputs, mpmc  # noqa: E402

FP64, FP32 = mpmc.FP64, mpmc.FP32
TOL = {FP64: 1e-13, FP32: 5e-6}
CASES = [  # dims, right-hand sides, precision, variant (-1: the default)
    ((4, 6, 4, 8), 1, FP64, -1), ((4, 6, 4, 8), 1, FP32, -1), ((4, 6, 4, 8), 1, FP64, 1), ((4, 6, 4, 8), 1, FP32, 1),
    ((4, 6, 4, 8), 1, FP64, 2), ((4, 6, 4, 8), 1, FP32, 2), ((16, 16, 10, 10), 1, FP64, -1),
    ((3, 5, 4, 7), 5, FP64, -1), ((3, 5, 4, 7), 5, FP32, -1), ((4, 4, 4, 6), 130, FP64, -1),
    ((8, 8, 8, 8), 64, FP64, -1), ((8, 8, 8, 4), 128, FP64, -1), ((3, 5, 4, 7), 64, FP32, -1),
    ((4, 6, 4, 8), 64, FP32, -1), ((4, 6, 3, 8), 64, FP32, 11), ((4, 4, 4, 4), 128, FP32, 12),
    ((4, 4, 4, 4), 64, FP32, 7), ((4, 4, 4, 4), 64, FP64, 9),
]


@pytest.mark.parametrize("dims,N,prec,variant", CASES)
def test_terms(dims, N, prec, variant):
    ctx = mpmc.Context(dims, 0.12, inputs.gauge_links(dims, 0.5, seed=8))
    if variant >= 0:
        ctx.tune_set(N, prec, variant)
    dt = torch.complex128 if prec == FP64 else torch.complex64
    wide = lambda v: v.view(dt).to(torch.complex128)  # noqa: E731
    x = ctx.noise(7, 1, 0, N, prec)
    roots = 1.0 + 0.4 * np.exp(2j * np.pi * np.arange(6) / 6 + 0.3j)
    for d in (1, 2, 3, 4, 5, 6):
        y = torch.full_like(x, 255)      # NaN
        x0 = x.clone()
        ctx.apply_poly(ctx.poly_from_roots(roots[:d]), x, N, prec, out=y)
        assert torch.equal(x, x0)
        w, ref = wide(x), 0
        for k in range(d):
            ref = ref + w / complex(roots[k])
            w = w - wide(ctx.apply_M(w.to(dt).view(x.dtype), N, prec)) / complex(roots[k])
        assert float((wide(y) - ref).norm() / ref.norm()) < TOL[prec], d
