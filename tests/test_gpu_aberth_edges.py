"""Aberth-Ehrlich sweeps at the edges of their layout: one to six rows around a
chunk of four, the row counts at which the lanes per root and the columns per
lane change, 256 rows, and workgroups whose spare groups walk along, against
the shifted QR (marked gpu).

Tolerance: 1e-11 of the largest root up to 129 rows, as the two solvers are
compared elsewhere, and in proportion to the rows beyond (rounding of a sum
over a row).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_00016_amd import inputs, mpmc  # noqa: E402


@pytest.mark.parametrize("dims,kappa,seed,rows", [
    ((4, 4, 4, 4), 0.2, 21, (1, 2, 3, 4, 5, 6, 9, 16, 17, 31, 32, 33, 48, 64, 65)),
    ((8, 8, 8, 8), 0.2, 2, (127, 128, 129, 160, 161, 255, 256))])
def test_against_qr(dims, kappa, seed, rows):
    ctx = mpmc.Context(dims, kappa, inputs.gauge_links(dims, 0.5, seed=seed))
    for d in rows:
        P = []
        for method in (mpmc.DENSE_ABERTH, mpmc.DENSE_QR):
            ctx.set_dense_method(method)
            P.append(ctx.gmres_poly(1, 0x100, d))
        ab, qr = (np.asarray(p.roots) for p in P)
        assert P[0].d_eff == P[1].d_eff == d and ab.shape == qr.shape
        gap = np.abs(np.subtract.outer(ab, qr))
        tol = 1e-11 * max(1.0, d / 129) * np.abs(qr).max()
        assert max(gap.min(axis=0).max(), gap.min(axis=1).max()) < tol, d
