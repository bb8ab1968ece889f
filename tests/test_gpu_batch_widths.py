"""Small batches: the operator in workgroups of one wavefront and of four (the
line lies at 32 wavefronts per compute unit) and the default FP32 kernel on
both sides of the line where column workgroups fill the chip, bit for bit the
blocked kernel's columns; the fused step's samples up to the grouping of FP64
sums (1e-13) (marked gpu).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_00016_amd import inputs, mpmc  # noqa: E402

DT = {mpmc.FP64: torch.complex128, mpmc.FP32: torch.complex64}


@pytest.mark.parametrize("prec", [mpmc.FP64, mpmc.FP32])
@pytest.mark.parametrize("dims,widths", [((8, 8, 8, 16), (63, 64, 65)), ((3, 5, 4, 7), (2, 37, 130))])
def test_columns_do_not_depend_on_the_batch(dims, widths, prec):
    ctx = mpmc.Context(dims, 0.12, inputs.gauge_links(dims, 0.5, seed=8))
    full = 192
    ctx.tune_set(full, prec, 4)
    x = ctx.noise(7, 1, 0, full, prec).view(DT[prec]).view(-1, full)
    ref = ctx.apply_M(x.reshape(-1).view(torch.uint8), full, prec).view(DT[prec]).view(-1, full)
    for n in widths:
        y = ctx.apply_M(x[:, :n].contiguous().reshape(-1).view(torch.uint8), n, prec).view(DT[prec]).view(-1, n)
        assert torch.equal(y, ref[:, :n]), n


@pytest.mark.parametrize("dims,N", [((4, 4, 4, 4), 64), ((8, 8, 8, 8), 128), ((8, 8, 8, 8), 256), ((10, 10, 10, 10), 64),
                                    ((12, 12, 12, 4), 64)])
def test_default_fp32_matches_blocked_and_column(dims, N):
    ctx = mpmc.Context(dims, 0.12, inputs.gauge_links(dims, 0.5, seed=8))
    x = ctx.noise(7, 1, 0, N, mpmc.FP32)
    P = ctx.poly_from_roots(1.0 + 0.4 * np.exp(2j * np.pi * np.arange(5) / 5 + 0.3j))
    y, X = ctx.apply_M(x, N, mpmc.FP32), ctx.level(P, None, None, 1, 5, 1, 0, N, prec=mpmc.FP32)[0]
    for v in (5, 10):
        ctx.tune_set(N, mpmc.FP32, v)
        assert torch.equal(y, ctx.apply_M(x, N, mpmc.FP32))
        X1 = ctx.level(P, None, None, 1, 5, 1, 0, N, prec=mpmc.FP32)[0]
        assert np.linalg.norm(X - X1) < 1e-13 * np.linalg.norm(X1)


@pytest.mark.parametrize("prec,wide", [(mpmc.FP64, 4), (mpmc.FP32, 5)])
@pytest.mark.parametrize("dims,N", [((4, 4, 3, 4), 64), ((7, 8, 9, 8), 64), ((7, 3, 5, 7), 64), ((12, 5, 12, 20), 128)])
def test_default_chunks_match_wide_ones(dims, N, prec, wide):
    """Without a column kernel (odd extents): 32- or 64-wide chunks by the
    operand's size and the number of sites."""
    ctx = mpmc.Context(dims, 0.12, inputs.gauge_links(dims, 0.5, seed=8))
    x = ctx.noise(7, 1, 0, N, prec)
    P = ctx.poly_from_roots(1.0 + 0.4 * np.exp(2j * np.pi * np.arange(5) / 5 + 0.3j))
    y, X = ctx.apply_poly(P, x, N, prec), ctx.level(P, None, None, 1, 5, 1, 0, N, prec=prec)[0]
    ctx.tune_set(N, prec, wide)
    assert torch.equal(y, ctx.apply_poly(P, x, N, prec))
    X1 = ctx.level(P, None, None, 1, 5, 1, 0, N, prec=prec)[0]
    assert np.linalg.norm(X - X1) < 1e-13 * np.linalg.norm(X1)
