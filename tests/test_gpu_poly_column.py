"""The column kernels' sum of a polynomial (started without reading the output,
two terms a step, no vector stored by the last step), pinned: the default takes
them on large lattices only.  As test_gpu_poly_terms, into an output that holds
NaN, and against the oracle (marked gpu).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import test_gpu_poly_terms as terms  # noqa: E402
from oracle import poly as OP  # noqa: E402
from oracle.philox import z4_noise_batch  # noqa: E402
from oracle.wilson import WilsonOp  # noqa: E402
from paper_2402_00016_amd import inputs, mpmc  # noqa: E402

FP32 = mpmc.FP32


@pytest.mark.parametrize("dims,N,variant", [
    ((6, 4, 6, 4), 64, 10), ((4, 6, 4, 8), 128, 10), ((8, 8, 4, 5), 64, 10), ((4, 6, 3, 8), 128, 11),
    ((6, 4, 8, 4), 64, 12), ((4, 6, 4, 8), 64, 5)])
def test_terms(dims, N, variant):
    terms.test_terms(dims, N, FP32, variant)


@pytest.mark.parametrize("variant", [5, 10, 11, 12])
def test_garbage_output(variant):
    """Nine roots in FP32: eight steps of a relative rounding below 2e-6 (bound 2e-5)."""
    dims, N = (4, 4, 4, 4), 128
    U = inputs.gauge_links(dims, 0.5, seed=1)
    op, ctx = WilsonOp(dims, 0.115, U), mpmc.Context(dims, 0.115, U)
    ctx.tune_set(N, FP32, variant)
    roots = 1.0 + 0.4 * np.exp(2j * np.pi * np.arange(9) / 9 + 0.3j)
    y = ctx.vector(N, FP32)
    y.view(torch.float32).fill_(float("nan"))
    ctx.apply_poly(ctx.poly_from_roots(roots), ctx.noise(4, 1, 0, N, FP32), N, FP32, out=y)
    got = ctx.unpack(y, N, FP32).cpu().numpy()
    assert np.all(np.isfinite(got))
    want = np.stack([OP.apply_p(op, roots, e) for e in z4_noise_batch(4, 1, 0, N, op.n)[[0, 63, 64, 127]]])
    assert np.linalg.norm(got[[0, 63, 64, 127]] - want) < 2e-5 * np.linalg.norm(want)
