"""FP16S operator at batch widths on both sides of the line between workgroups
of one and of four wavefronts: the batch's columns are those of a 64-wide one,
up to half-precision roundings of the result that another order of
contractions can flip (2^-10 of a site's largest component) (marked gpu).
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_00016_amd import inputs, mpmc  # noqa: E402


@pytest.mark.parametrize("dims,widths", [((16, 16, 16, 16), (3, 4, 5)), ((12, 12, 12, 12), (12, 13)),
                                         ((9, 11, 13, 7), (20, 21, 23, 33)), ((3, 5, 4, 7), (7,))])
def test_columns(dims, widths):
    ctx = mpmc.Context(dims, 0.12, inputs.gauge_links(dims, 0.5, seed=8))
    full = 64
    x = ctx.noise(7, 1, 0, full, mpmc.FP16S)
    ref = ctx.unpack(ctx.apply_M(x, full, mpmc.FP16S), full, mpmc.FP16S)
    top = ref.view(full, -1, 12).abs().amax(2, keepdim=True)
    for n in widths:
        y = ctx.unpack(ctx.apply_M(ctx.noise(7, 1, 0, n, mpmc.FP16S), n, mpmc.FP16S), n, mpmc.FP16S)
        assert bool(((y - ref[:n]).view(n, -1, 12).abs() <= top[:n] * 2.0 ** -10).all()), n
