"""GPU parity of the normalised block where its reductions run over many short pixel ranges (few workers, small tensors):
range counts that are no multiple of the final pass's stripes, a short last range, channel counts off its 32-channel
workgroups."""
import numpy as np
import pytest

from ols_inputs import generate as G
from oracle import conv_oracle as CO
from tests.helpers import max_norm_ratio
from tests.test_gpu_conv_bn import GRAD_TOL, bn_case, groups_of, one_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,dims,batch,seed", [
    (3, (64, 13, 15, 7), 10, 152),     # 1950 pixels: 31 ranges, the last of 30 pixels
    (1, (48, 32, 33, 4), 4, 154),      # 4224 pixels: 64 ranges of 66, 48 channels
    (2, (16, 8, 9, 3), 1, 151),        # 72 pixels: two ranges of 36
])
def test_gradient_and_loss_match_oracle(m, dims, batch, seed):
    cfg, X, labels, x0 = bn_case(m, dims, batch, 1, seed=seed)
    x0 = x0 + G.generic_normal(7, 6, x0.shape, sigma=0.05)
    g, losses = one_step(cfg, dims, batch, X, labels, x0)
    # seeds whose ReLU inputs keep clear of zero by more than single precision's rounding of them
    assert min(CO.convblock_relu_margin(x0, dims[0], dims[3], X[i, 0], batch_norm=True) for i in range(m)) >= 3e-6
    for i in range(m):
        loss, grad = CO.convblock_bn_loss_grad(x0, dims[0], dims[3], X[i, 0], labels[i, 0])
        assert abs(losses[i] - loss) <= 2e-5 * max(1.0, abs(loss))
        for name, where in groups_of(dims[0], dims[3]).items():
            assert max_norm_ratio(g[i][np.ravel(where)], grad[np.ravel(where)]) <= GRAD_TOL, name
