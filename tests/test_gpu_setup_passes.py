"""Set-up Arnoldi, delayed form: dot pass at both run lengths with a ragged last
workgroup and odd numbers of vectors, coefficient kernel with more than 64 rows,
against plain CGS2 (GMRES roots and relres; 1e-8 in FP64 and 1e-4 in FP32 of
the largest root, the bounds the two forms are held to) (marked gpu).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_00016_amd import inputs, mpmc  # noqa: E402


@pytest.mark.parametrize("dims,kappa,d,prec,tol", [
    ((15, 13, 16, 15), 0.12, 9, mpmc.FP64, 1e-8), ((15, 13, 16, 15), 0.12, 8, mpmc.FP32, 1e-4),
    ((5, 3, 4, 7), 0.12, 10, mpmc.FP32, 1e-4), ((5, 3, 4, 7), 0.2, 70, mpmc.FP64, 1e-8),
    ((5, 3, 4, 7), 0.2, 64, mpmc.FP64, 1e-8)])
def test_delayed_matches_plain(dims, kappa, d, prec, tol):
    ctx = mpmc.Context(dims, kappa, inputs.gauge_links(dims, 0.5, seed=21))
    ctx.set_setup_precision(prec)
    P = []
    for cgs2 in (1, 0):
        ctx.set_arnoldi_cgs2(cgs2)
        P.append(ctx.gmres_poly(1, 0x100, d))
    r1, r0 = (np.asarray(p.roots) for p in P)
    assert P[0].d_eff == P[1].d_eff == d
    gap = np.abs(np.subtract.outer(r0, r1))
    assert max(gap.min(axis=0).max(), gap.min(axis=1).max()) < tol * np.abs(r1).max()
    assert abs(P[1].relres - P[0].relres) < tol * P[0].relres


def test_more_vectors_than_a_row_holds():
    """260 steps on a lattice whose dot pass runs one row of the grid up to 256
    vectors: the residual (a norm relative to the start vector's) to 1e-10."""
    ctx = mpmc.Context((15, 13, 16, 15), 0.2, inputs.gauge_links((15, 13, 16, 15), 0.5, seed=21))
    P = []
    for cgs2 in (1, 0):
        ctx.set_arnoldi_cgs2(cgs2)
        P.append(ctx.gmres_poly(1, 0x100, 260))
    assert P[0].d_eff == P[1].d_eff == 260
    assert abs(P[0].relres - P[1].relres) < 1e-10
