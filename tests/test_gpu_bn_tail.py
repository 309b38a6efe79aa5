"""GPU parity of the normalised block's tail and of the backward sums formed from what it leaves per sample: images of
exactly 64 pixels (no part of 64 pixels reaches into a second sample), of 65 (every part does), one sample that ends a part
early, and channel counts with 64, 21, 16 and four stripes per workgroup."""
import numpy as np
import pytest

from ols_inputs import generate as G
from oracle import conv_oracle as CO
from tests.helpers import max_norm_ratio
from tests.test_gpu_conv_bn import GRAD_TOL, bn_case, groups_of, one_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,dims,batch,seed", [
    (2, (16, 8, 8, 4), 5, 161),
    (2, (48, 5, 13, 5), 7, 162),
    (1, (208, 7, 10, 3), 2, 163),
    (3, (64, 11, 6, 3), 1, 164),
    (1, (256, 8, 8, 2), 1, 165),
])
def test_gradient_and_loss_match_oracle(m, dims, batch, seed):
    cfg, X, labels, x0 = bn_case(m, dims, batch, 1, seed=seed)
    x0 = x0 + G.generic_normal(7, 6, x0.shape, sigma=0.05)
    # seeds whose ReLU inputs keep clear of zero by more than single precision's rounding of them
    assert min(CO.convblock_relu_margin(x0, dims[0], dims[3], X[i, 0], batch_norm=True) for i in range(m)) >= 3e-6
    g, losses = one_step(cfg, dims, batch, X, labels, x0)
    for i in range(m):
        loss, grad = CO.convblock_bn_loss_grad(x0, dims[0], dims[3], X[i, 0], labels[i, 0])
        assert abs(losses[i] - loss) <= 2e-5 * max(1.0, abs(loss))
        for name, where in groups_of(dims[0], dims[3]).items():
            assert max_norm_ratio(g[i][np.ravel(where)], grad[np.ravel(where)]) <= GRAD_TOL, name
