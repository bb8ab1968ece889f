"""Solves of one right-hand side: the cycle's correction is added to the FP64
iterate in the flat kernel.  GMRES iterates against a plain FP64 GMRES(m), with
the bounds of the batched solves, at row counts below one workgroup's step,
past it and not a multiple of it (marked gpu).
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


@pytest.mark.parametrize("prec,m,tol", [(mpmc.FP64, 1, 1e-10), (mpmc.FP64, 11, 1e-10), (mpmc.FP32, 1, 1e-4),
                                        (mpmc.FP32, 11, 1e-4), (mpmc.FP16S, 9, 2e-2)])
@pytest.mark.parametrize("dims", [(1, 2, 3, 3), (3, 5, 4, 7), (9, 10, 12, 11)])
def test_iterate(dims, prec, m, tol):
    U = inputs.gauge_links(dims, 0.5, seed=11)
    op, ctx = WilsonOp(dims, KAPPA, U), mpmc.Context(dims, KAPPA, U)
    rng = np.random.default_rng(m)
    B = rng.standard_normal((1, op.n)) + 1j * rng.standard_normal((1, op.n))
    b, x = ctx.pack(torch.from_numpy(B).cuda()), ctx.vector(1)
    its, _, rc = mpmc.mpmc_solve(ctx.handle, b, x, 1, restart=m, tol=1e-15, inner_prec=prec, max_outer=1,
                                 raise_on_noconv=False)
    assert rc == mpmc.ENOCONV and its == m
    ref = gmres_iterates(op, B, m)
    assert np.linalg.norm(ctx.unpack(x, 1).cpu().numpy() - ref) < tol * np.linalg.norm(ref)
