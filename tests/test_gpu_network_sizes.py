"""The network kernels over their grids: fewer entries than the waves of a few blocks (705 entries in
23 steps of 32), four working waves of eight in every block and a few more (9^3: 34,401 entries), and
more steps than waves, so that some waves take a second one (12^3: 87,132)."""
import numpy as np
import pytest

import qh_inputs as qi

from .gpu_setup import gpu_context
from .test_gpu_learned import _bf16, _flat, _unflat, _weights, factor_model
from .test_oracle_learned import edge_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 9, 12])
def test_factor_and_gradient_over_sizes(n):
    """Factor entries within the error model of the BF16 network, gradient per tensor within 2e-2 (the
    BF16 activations' and gradient operands' rounding) of the FP64 oracle fed the same BF16 inputs."""
    from oracle import learned as Lr
    A, rows, cols, f = edge_problem(n)
    ctx = gpu_context(qi.BoxMesh(n), 10 * 7.69e-10 / n)
    w = _weights(2)
    w32 = _unflat(_flat(w).astype(np.float64))
    ctx.precond_set_weights(_flat(w))
    gr, gc, gv = ctx.precond_factor()
    G, bound = factor_model(w32, f, rows, cols, A.diagonal())
    assert np.array_equal(gr, rows) and np.array_equal(gc, cols)
    # the oracle's features are FP64, the kernel's BF16 ones come from FP64 values of its own: an
    # entry on a rounding boundary may fall on the other side (at most 1 in 1000)
    assert (np.abs(gv - G) <= bound).mean() >= 0.999
    V = np.sign(np.random.default_rng(3).standard_normal((A.shape[0], 16))).astype(np.float32)
    loss, grad = ctx.precond_loss_grad(V)
    wb = dict(w32, W1=_bf16(w32["W1"]), W2=_bf16(w32["W2"]))
    loss_b, grad_b, _ = Lr.kaporin_loss_grad(wb, A, _bf16(f), rows, cols, V.astype(np.float64))
    assert abs(loss - loss_b) <= 2e-2 * max(1.0, abs(loss_b))
    for k in ("W1", "W2", "W3", "b1", "b2"):
        a, b = _unflat(grad.astype(np.float64))[k].ravel(), np.asarray(grad_b[k]).ravel()
        assert np.linalg.norm(a - b) <= 2e-2 * np.linalg.norm(b) + 1e-12, k
    ctx.close()
