"""GPU parity of the output layer at the edges of its tiling: hidden widths around what one pass of a workgroup covers for
each wavefront count, batches that end inside a group of 16 samples, one class, sixteen, seventeen and thirty-two."""
import numpy as np
import pytest

from ols_inputs import generate as G
from oracle import ols_oracle as O
from tests.helpers import max_norm_ratio
from tests.test_gpu_gemm_split import one_step
from tests.test_gpu_mlp import small_mlp_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,batch", [
    ((16, 256, 10), 16), ((16, 260, 10), 20),            # four wavefronts and one unit quad more
    ((16, 512, 16), 36), ((16, 516, 16), 12),            # eight wavefronts of four tiles, then of eight
    ((16, 1024, 1), 16), ((16, 1028, 3), 4),             # one pass, then several
    ((16, 2100, 10), 20),
    ((16, 256, 17), 16), ((16, 516, 32), 20), ((1540, 24), 12),   # more than sixteen classes; no hidden layer
])
def test_gradient_and_loss_match_oracle(dims, batch):
    m = 2
    cfg, X, labels, x0 = small_mlp_case(m, dims, batch, 1, seed=511)
    x0 = x0 + G.generic_normal(3, 1, x0.shape, sigma=0.02)
    g, losses = one_step(cfg, dims, batch, X, labels, x0)
    for i in range(m):
        loss, grad = O.mlp_loss_grad(x0, dims, X[i, 0], labels[i, 0])
        assert abs(losses[i] - loss) <= 1e-5 * abs(loss) + 1e-7
        assert max_norm_ratio(g[i], grad) <= 2e-5 or np.abs(grad).max() == 0.0
