"""Deflation terms of the level samples taken from the noise codes, at batch
shapes that take them and at ones that do not, against the FP64 oracle (marked
gpu).  Tolerance: the FP64 level bound of the parity tests, 1e-10 in norm (sums
of n = 2,520 exact products per eigenvector, unit roundoff 1.1e-16).
"""
from types import SimpleNamespace

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import estimator as OES  # noqa: E402
from oracle import krylov as OK  # noqa: E402
from oracle.philox import z4_noise  # noqa: E402
from oracle.wilson import WilsonOp  # noqa: E402
from paper_2402_00016_amd import inputs, mpmc  # noqa: E402

DIMS, KAPPA = (3, 5, 2, 7), 0.12     # 210 sites: not a multiple of a workgroup's four


@pytest.fixture(scope="module")
def field():
    U = inputs.gauge_links(DIMS, 0.5, seed=6)
    op = WilsonOp(DIMS, KAPPA, U)
    b = z4_noise(1, 0x100, 0, op.n)
    return op, mpmc.Context(DIMS, KAPPA, U), [OK.gmres_poly(op, b, d)[0] for d in (5, 3)]


# whole chunks (fused and, at 320, not), a ragged count, and a last batch of 8 after one of 64
@pytest.mark.parametrize("N,batch", [(64, 0), (128, 64), (320, 0), (65, 0), (72, 64)])
@pytest.mark.parametrize("k,theta", [(1, "I"), (4, "g5"), (5, "I"), (9, "g5")])
def test_deflated_samples(field, N, batch, k, theta):
    op, ctx, (P1, P2) = field
    rng = np.random.default_rng(k)
    Z, U = (rng.standard_normal((k, op.n)) + 1j * rng.standard_normal((k, op.n)) for _ in range(2))
    lam = rng.uniform(0.3, 0.6, k) + 0.1j * rng.standard_normal(k)
    D = SimpleNamespace(k=k, lam=lam, Z=Z, U=U)
    dev = ctx.defl_from_arrays(lam, torch.from_numpy(Z).cuda(), torch.from_numpy(U).cuda())
    g1, g2 = ctx.poly_from_roots(P1.roots), ctx.poly_from_roots(P2.roots)
    X, T, _ = ctx.level(g1, g2, dev, int(theta == "g5"), 3, 2, 5, N, max_batch=batch)
    Xr, Tr = OES.level_samples(op, P1, P2, D, theta, 3, 2, 5, N)
    assert np.linalg.norm(X - Xr) < 1e-10 * np.linalg.norm(Xr)
    assert abs(T - Tr) < 1e-10 * abs(Tr)
