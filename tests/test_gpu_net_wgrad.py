"""Weight gradient of the network at pair counts around the edges of its lane
layout (four right-hand sides a lane, sixteen a wavefront) and with rows that
are not 16-byte aligned, against the FP64 oracle (marked gpu).

Tolerances: BF16 weights and transported inputs (2^-9 each), three layers
forward and the operands of the gradient itself: 2.5e-2 for the loss, 4e-2 in
norm for the gradient and for each layer's block of it.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import net as ON  # noqa: E402
from paper_2402_00016_amd import inputs, mpmc  # noqa: E402

DIMS = (3, 5, 2, 7)


@pytest.fixture(scope="module")
def field():
    U = inputs.gauge_links(DIMS, 0.4, seed=5)
    return mpmc.Context(DIMS, 0.1, U), ON.Transport(DIMS, U)


@pytest.mark.parametrize("P", [1, 2, 4, 5, 12, 16, 18, 20, 33])
@pytest.mark.parametrize("shift", [0, 8])
def test_gradient(field, P, shift):
    ctx, T = field
    n = ctx.n
    rng = np.random.default_rng(P)
    theta = 0.3 * rng.standard_normal(ON.n_params())
    R = rng.standard_normal((P, n)) + 1j * rng.standard_normal((P, n))
    E = rng.standard_normal((P, n)) + 1j * rng.standard_normal((P, n))
    r = ctx.pack(torch.from_numpy(R).cuda(), mpmc.FP32)
    e = ctx.pack(torch.from_numpy(E).cuda(), mpmc.FP32)
    moved = torch.empty(r.numel() + 16, dtype=torch.uint8, device="cuda")[shift:shift + r.numel()]
    moved.copy_(r)
    loss, grad = ctx.net(theta).loss_grad(moved, e, P)
    loss_ref, grad_ref = ON.loss_and_grad(T, theta, R, E)
    assert abs(loss - loss_ref) < 2.5e-2 * abs(loss_ref)
    for a, b in ((0, 576), (576, 1728), (1728, 2304)):
        assert np.linalg.norm(grad[a:b] - grad_ref[a:b]) < 4e-2 * np.linalg.norm(grad_ref[a:b])
