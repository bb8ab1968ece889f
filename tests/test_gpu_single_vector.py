"""Single vectors with eight lanes per site (the default): neighbours computed
from the coordinates on extents 1 and 2, odd ones and a ragged last workgroup,
and above 12^4 sites, against the kernel with a lane per site (whose bits are
the generic kernel's; the two sum the hops in different orders: 1e-14 of the
norm in FP64, 5e-6 in FP32), twice with the same bits (marked gpu).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_00016_amd import inputs, mpmc  # noqa: E402


@pytest.mark.parametrize("prec,tol", [(mpmc.FP64, 1e-14), (mpmc.FP32, 5e-6)])
@pytest.mark.parametrize("dims", [(1, 2, 3, 5), (2, 2, 2, 2), (7, 3, 5, 4), (1, 1, 1, 9), (13, 12, 12, 12)])
def test_eight_lanes_match_site_per_lane(dims, prec, tol):
    ctx = mpmc.Context(dims, 0.12, inputs.gauge_links(dims, 0.5, seed=4))
    dt = torch.complex128 if prec == mpmc.FP64 else torch.complex64
    x = ctx.noise(11, 2, 0, 1, prec)
    P = ctx.poly_from_roots(1.0 + 0.4 * np.exp(2j * np.pi * np.arange(4) / 4 + 0.3j))
    runs = [lambda d=d, t=t: ctx.apply_M(x, 1, prec, dagger=d, theta=t) for d in (False, True) for t in (0, 1)]
    for f in runs + [lambda: ctx.apply_poly(P, x, 1, prec)]:
        got = f().view(dt)
        ctx.tune_set(1, prec, 2)
        want = f().view(dt)
        ctx.tune_set(1, prec, -1)
        assert float((got - want).norm() / want.norm()) < tol
        assert torch.equal(got, f().view(dt))
