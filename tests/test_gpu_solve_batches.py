"""GMRES iterates of the batched solves at right-hand-side counts around the
edges of the batch kernels' thread layouts, against a plain FP64 GMRES(m) on
the oracle operator (marked gpu).

One outer cycle of m inner steps and no convergence test met: x is then the
minimiser of ||b - M x|| over the m-dimensional Krylov space, so every dot
product and update of every step enters it.  Tolerances: FP64 cycles project
twice and carry only rounding, amplified by the condition of the small
least-squares problem (below 1e3 here): 1e-10.  FP32 vectors: unit roundoff
6e-8, m = 28 steps, one projection, the same condition: 28 x 6e-8 x 60 = 1e-4.
FP16S basis: 2^-11 per stored component and 9 steps: 9 x 5e-4 x 4 = 2e-2.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle.wilson import WilsonOp  # noqa: E402
from paper_2402_00016_amd import inputs, mpmc  # noqa: E402

# 2,520 rows, a multiple of none of the workgroup row counts; vectors below and above the size at
# which the flat kernels take over (10 MB: 43 right-hand sides at 1,210 sites and FP64)
SMALL, LARGE, KAPPA = (3, 5, 2, 7), (11, 5, 2, 11), 0.2


@pytest.fixture(scope="module")
def fields():
    out = {}
    for dims in (SMALL, LARGE):
        U = inputs.gauge_links(dims, 0.5, seed=11)
        out[dims] = WilsonOp(dims, KAPPA, U), mpmc.Context(dims, KAPPA, U)
    return out


def gmres_iterates(op, B, m):
    """x_m of GMRES from x = 0 for every row of B (modified Gram-Schmidt, twice)."""
    N = len(B)
    beta = np.linalg.norm(B, axis=1)
    V, H = [B / beta[:, None]], np.zeros((N, m + 1, m), dtype=complex)
    for j in range(m):
        w = op(V[j])
        for _ in range(2):
            for i, v in enumerate(V):
                h = np.sum(np.conj(v) * w, axis=1)
                H[:, i, j] += h
                w = w - h[:, None] * v
        H[:, j + 1, j] = np.linalg.norm(w, axis=1)
        V.append(w / H[:, j + 1, j][:, None])
    X = np.zeros_like(B)
    for r in range(N):
        rhs = np.zeros(m + 1, dtype=complex)
        rhs[0] = beta[r]
        y = np.linalg.lstsq(H[r], rhs, rcond=None)[0]
        X[r] = sum(y[j] * V[j][r] for j in range(m))
    return X


@pytest.mark.parametrize("prec,m,tol", [(mpmc.FP64, 28, 1e-10), (mpmc.FP32, 28, 1e-4), (mpmc.FP16S, 9, 2e-2)])
@pytest.mark.parametrize("dims,N", [(SMALL, 3), (SMALL, 64), (SMALL, 513), (LARGE, 65), (LARGE, 100), (LARGE, 128),
                                    (LARGE, 130), (LARGE, 257), (LARGE, 511)])
def test_gmres_iterates(fields, dims, N, prec, m, tol):
    op, ctx = fields[dims]
    rng = np.random.default_rng(N)
    B = rng.standard_normal((N, op.n)) + 1j * rng.standard_normal((N, op.n))
    b, x = ctx.pack(torch.from_numpy(B).cuda()), ctx.vector(N)
    its, _, rc = mpmc.mpmc_solve(ctx.handle, b, x, N, restart=m, tol=1e-15, inner_prec=prec, max_outer=1,
                                 raise_on_noconv=False)
    assert rc == mpmc.ENOCONV and its == m
    pick = sorted({0, 1, N // 3, N // 2, N - 2, N - 1})
    X = ctx.unpack(x, N)[pick].cpu().numpy()
    ref = gmres_iterates(op, B[pick], m)
    err = np.linalg.norm(X - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert err.max() < tol


@pytest.mark.parametrize("N", [65, 130])
def test_gmres_iterates_past_the_counted_updates(fields, N):
    """FP32 updates know the number of vectors up to 32: 36 steps, the bound of
    28 scaled by the steps."""
    test_gmres_iterates(fields, LARGE, N, mpmc.FP32, 36, 1.3e-4)
