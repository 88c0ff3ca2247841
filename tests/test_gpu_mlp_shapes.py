"""Training kernels of the committor at their edges: parameters left over in a
row of four, one input and many, batches below, at and above a workgroup's
four samples, a pass of 64 and the 512 samples fetched ahead.  Against the FP64
chain rule: a dot product of n FP32 terms is off by at most n u of the sum of
their magnitudes, so the loss is compared to 1e-5 relative and the gradient to
1e-4 of its norm, far above B u = 6e-5 times the cancellation of these inputs."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_in,B", [(1, 1), (2, 3), (3, 4), (4, 5), (5, 63), (7, 64), (8, 65), (9, 511), (12, 512),
                                    (13, 513), (64, 100), (65, 1025)])
def test_loss_and_gradient(n_in, B):
    print(f"case: training kernels, {n_in} inputs, batch {B}", flush=True)
    from paper_1303_5986_amd import we
    rng = np.random.default_rng(1000 * n_in + B)
    p = rng.normal(0, 0.15, we.n_params(n_in)).astype(np.float32)
    feat = np.concatenate([rng.uniform(0.5, 3.0, n_in), rng.uniform(0.3, 1.5, n_in)]).astype(np.float32)
    x = rng.integers(0, 80, size=(B, n_in)).astype(np.int32)
    y = rng.uniform(0, 1, B).astype(np.float32)
    loss, grad = we.mlp_loss_grad(n_in, p, feat, x, y)
    rl, rg = mlp.loss_grad(p.astype(np.float64), feat.astype(np.float64), x, y.astype(np.float64), n_in)
    assert abs(loss - rl) <= 1e-5 * abs(rl)
    assert np.linalg.norm(grad - rg) <= 1e-4 * np.linalg.norm(rg)
    assert np.all(np.abs(grad - rg) <= 1e-4 * np.abs(rg).max() + 1e-3 * np.abs(rg))
