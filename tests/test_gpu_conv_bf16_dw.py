"""Kernel gradient of the bf16 convolutions (input rows in a ring of LDS rows) against the CPU oracle with the same rounding
points, over the lengths of its pixel ranges: 96-pixel slices, odd and even in number, ranges cut inside an image, a last
range that is short or empty, the widest images."""
import pytest

from ols_inputs import generate as G
from oracle import conv_oracle as CO
from tests.helpers import l2_ratio, max_norm_ratio
from tests.test_gpu_conv_bf16 import conv_case, groups_of, make_session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,dims,batch", [
    (1, (64, 4, 14, 3), 1),        # exactly one slice of 96
    (1, (64, 4, 14, 3), 2),        # two
    (1, (64, 9, 9, 3), 2),         # 242: three, the last of 50
    (1, (64, 6, 30, 3), 4),        # 1024: two ranges of 576 and 448
    (3, (64, 9, 11, 4), 9),        # 1287 on three ranges of 480, 480, 327
    (1, (64, 2, 128, 3), 5),       # 2600 pixels at the longest halo: the ring is nearly full
    (1, (64, 5, 61, 3), 6),        # 2646 pixels on six ranges of 480: the last is 246
    (1, (128, 10, 12, 3), 7),      # 2 x 2 blocks, 1176 pixels on three ranges
    (5, (192, 6, 15, 3), 20),      # 45 blocks: five ranges fill one round of the compute units, a sixth would start a second
    (1, (64, 1, 1, 3), 171),       # 1539 pixels of which 171 are image: four ranges of 480, the last of 99
])
def test_kernel_and_bias_gradients(m, dims, batch):
    cfg, X, labels, x0 = conv_case(m, dims, batch, 1, seed=616)
    x0 = x0 + G.generic_normal(7, 6, x0.shape, sigma=0.02)
    with make_session(m, cfg.d, 2, 0.6, 0.05, 0.0) as s:
        s.attach_convblock(*dims, batch, gemm_dtype="bf16")
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_batch(Xd[:, 0], yd[:, 0])
        s.local_step()
        g = s.gradient()
    for i in range(m):
        _, grad = CO.convblock_loss_grad(x0, dims[0], dims[3], X[i, 0], labels[i, 0], bf16_operands=True)
        for name, sl in groups_of(dims[0], dims[3]).items():
            sl = sl.ravel()
            # one bf16 ulp (0.4 %) on the delta of a (sample, channel) where fp32 and double sums round differently
            assert l2_ratio(g[i][sl], grad[sl]) <= 1e-2, "worker %d %s" % (i, name)
            assert max_norm_ratio(g[i][sl], grad[sl]) <= 3e-2, "worker %d %s" % (i, name)
