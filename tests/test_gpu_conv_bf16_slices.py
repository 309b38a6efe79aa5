"""The plain bf16 block in launches of middling size, whose forward and delta take their kernel slices through LDS, against the
small launch's tiles that the oracle tests cover: the same worker alone and as one of many identical ones."""
import pytest

from ols_inputs import generate as G
from tests.helpers import l2_ratio, max_norm_ratio
from tests.test_gpu_conv_bf16 import conv_case, groups_of
from tests.test_gpu_conv_bf16_tiles import one_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,batch,m", [
    ((64, 30, 30, 5), 8, 33),      # 528 tiles of 512 pixels, whole ones
    ((64, 9, 33, 3), 12, 52),      # wider than 32, the longer strip; 4620 padded pixels: a last tile of 12
    ((64, 6, 128, 3), 4, 58),      # the widest image
    ((64, 6, 6, 3), 64, 65),       # images of 64 padded pixels, the smallest with the fused tail
    ((64, 9, 33, 3), 12, 22),      # 220 tiles
    ((128, 13, 15, 7), 20, 11),    # two contraction chunks, two output tiles
    ((192, 14, 14, 5), 16, 12),    # three of each
    ((64, 30, 30, 5), 8, 31),      # 496: the other kernels
])
def test_middling_launch(dims, batch, m):
    cfg, X, labels, x0 = conv_case(1, dims, batch, 1, seed=727)
    x0 = x0 + G.generic_normal(7, 6, x0.shape, sigma=0.02)
    g1, l1 = one_step(cfg, dims, batch, 1, X, labels, x0, False)
    g, losses = one_step(cfg, dims, batch, m, X, labels, x0, False)
    # the pooling's sums of 64 pixels are added over other lanes: 128 additions, 2^-24 of the (non-negative) sum each
    bound = 128 * 2.0 ** -24
    for i in (0, m // 2, m - 1):
        assert abs(losses[i] - l1[0]) <= bound * max(1.0, abs(l1[0]))
        for name, sl in groups_of(dims[0], dims[3]).items():
            sl = sl.ravel()
            if name in ("Wh", "bh"):
                assert max_norm_ratio(g[i][sl], g1[0][sl]) <= 8 * bound, name
            else:   # a last bit of the pooled delta can move it over a bf16 rounding boundary: 0.4 % of one channel of a sample
                assert l2_ratio(g[i][sl], g1[0][sl]) <= 1e-2, name
