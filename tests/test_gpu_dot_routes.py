"""Dot products of 64-wide batches on both sides of the lines between the (site,
rhs) tiles and the flat kernels: small lattices (1,200 sites or 150,000 (site,
rhs) pairs) and vectors whose operands grow past what stays cached, so that a
cycle starts flat and ends in tiles.  GMRES iterates against a plain FP64
GMRES(m), with the bounds of the batched solves (marked gpu).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle.wilson import WilsonOp  # noqa: E402
from paper_2402_00016_amd import inputs, mpmc  # noqa: E402
from test_gpu_solve_batches import KAPPA, gmres_iterates  # noqa: E402


@pytest.mark.parametrize("dims,N,prec,m,tol", [
    ((4, 4, 4, 4), 64, mpmc.FP64, 20, 1e-10), ((4, 4, 4, 4), 64, mpmc.FP16S, 9, 2e-2),
    ((5, 4, 6, 5), 192, mpmc.FP32, 20, 1e-4), ((5, 4, 6, 5), 256, mpmc.FP32, 20, 1e-4),
    ((5, 4, 6, 5), 256, mpmc.FP16S, 9, 2e-2), ((6, 6, 6, 6), 64, mpmc.FP64, 20, 1e-10),
    ((7, 8, 9, 8), 128, mpmc.FP32, 16, 1e-4), ((7, 8, 9, 8), 64, mpmc.FP64, 16, 1e-10)])
def test_iterates(dims, N, prec, m, tol):
    U = inputs.gauge_links(dims, 0.5, seed=11)
    op, ctx = WilsonOp(dims, KAPPA, U), mpmc.Context(dims, KAPPA, U)
    rng = np.random.default_rng(N)
    B = rng.standard_normal((N, op.n)) + 1j * rng.standard_normal((N, op.n))
    b, x = ctx.pack(torch.from_numpy(B).cuda()), ctx.vector(N)
    its, _, rc = mpmc.mpmc_solve(ctx.handle, b, x, N, restart=m, tol=1e-15, inner_prec=prec, max_outer=1,
                                 raise_on_noconv=False)
    assert rc == mpmc.ENOCONV and its == m
    pick = [0, 63, N - 1]
    X = ctx.unpack(x, N)[pick].cpu().numpy()
    ref = gmres_iterates(op, B[pick], m)
    assert (np.linalg.norm(X - ref, axis=1) / np.linalg.norm(ref, axis=1)).max() < tol
