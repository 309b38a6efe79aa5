"""The kernel gradients of the bf16 blocks where one launch computes both layers' (conv3x3_bf16_dw_pair_splits), and where two
do, against the CPU oracle with the same rounding points.  The bound is that of the blocks' other parity tests: one bf16
rounding that falls the other way moves a value by 0.4 %, and a normalisation spreads it over a channel."""
import numpy as np
import pytest

import ols_inputs as I
from ols_inputs import generate as G
from oracle import conv_oracle as CO
from tests.helpers import l2_ratio, max_norm_ratio

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,dims,batch,batch_norm", [
    (3, (64, 13, 15, 4), 9, True),      # 2295 padded pixels: five ranges, the last shorter
    (3, (64, 13, 15, 4), 9, False),
    (1, (128, 8, 8, 3), 5, True),       # one range of 500; 2 x 2 blocks of the gradient per layer
    (5, (64, 6, 5, 3), 20, False),      # images of 56 padded pixels: a1's signs take the first delta's place, which moves
    (2, (192, 5, 5, 3), 2, True),       # the second layer's sums do not fit the dead tensors: two launches
    (2, (64, 2, 2, 3), 3, False),       # and without a tail
])
def test_both_kernel_gradients(m, dims, batch, batch_norm):
    from paper_2002_09539_amd.session import Session
    cfg = I.get(9 if batch_norm else 8).scaled(m=m, dims=dims, batch=batch, nb=1, seed=901)
    X, labels = G.conv_data(cfg)
    x0 = G.conv_init(cfg)
    C, n_w = dims[0], 9 * dims[0] ** 2
    with Session(m, cfg.d, 2, 0.6, 0.05, 0.0) as s:
        s.attach_convblock(*dims, batch, batch_norm=batch_norm, gemm_dtype="bf16")
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_batch(Xd[:, 0], yd[:, 0])
        s.local_step()
        g = s.gradient()
    loss_grad = CO.convblock_bn_loss_grad if batch_norm else CO.convblock_loss_grad
    second = n_w + (2 * C if batch_norm else C)
    for i in range(m):
        _, want = loss_grad(x0, dims[0], dims[3], X[i, 0], labels[i, 0], bf16_operands=True)
        for at, size in ((0, n_w), (second, n_w)) + (() if batch_norm else ((n_w, C), (second + n_w, C))):   # kernels, biases
            sl = slice(at, at + size)
            assert l2_ratio(g[i][sl], want[sl]) <= 1e-2, (i, at)
            assert max_norm_ratio(g[i][sl], want[sl]) <= 3e-2, (i, at)
    assert np.isfinite(g).all()
