"""GPU parity of the bf16 MLP where its forward and delta GEMMs take the kernel of small launches: rows, columns and
contractions that are whole tiles, steps and groups of steps or not, both sides of the rule's lines, and an infinite weight."""
import numpy as np
import pytest

from ols_inputs import generate as G
from oracle import ols_oracle as O
from tests.helpers import l2_ratio
from tests.test_gpu_mlp import make_session, small_mlp_case

from paper_2002_09539_amd import binding as B

pytestmark = pytest.mark.gpu


def one_step(m, dims, batch, cfg, X, labels, x0):
    with make_session(m, cfg.d, 2, 0.6, 0.05, 0.0) as s:
        s.set_option(B.OLS_OPT_FUSE_GEMM_UPDATE, 0)
        s.attach_mlp(dims, batch, "bf16")
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_batch(Xd[:, 0], yd[:, 0])
        s.local_step()
        return s.gradient(), s.losses()


@pytest.mark.parametrize("m,dims,batch", [
    (2, (8, 8, 8, 3), 8),                # a quarter of one step, eight rows and columns
    (3, (128, 40, 24, 5), 40),           # one step per wavefront; eight rows and eight columns more than a tile
    (2, (136, 296, 136, 7), 40),         # a step of eight indices more
    (1, (768, 16, 520, 3), 32),          # a whole group of six steps
    (2, (776, 48, 16, 3), 24),           # seven steps per wavefront: two groups of four
    (2, (2056, 24, 8, 4), 24),           # 17 steps per wavefront: three groups of six
    (25, (320, 1024, 8, 4), 32),         # 8,000 steps of the forward pass, the most that it takes
    (25, (328, 1024, 8, 4), 32),         # 8,800: the 64 x 64 tiles
    (7, (16, 1280, 800, 4), 32),         # 7,000 steps of the delta, the most that it takes
    (8, (1032, 520, 264, 6), 72),        # 13,464 of a long contraction
    (8, (16, 1024, 1032, 4), 32),        # 256 tiles of the delta over a long contraction, the most that it takes
    (8, (16, 1032, 1032, 4), 32),        # 264: the 64 x 64 tiles
    (14, (16, 1112, 80, 4), 32),         # 490 tiles of the delta beside one round of the 64 x 64 ones, the most that it takes
    (38, (16, 568, 160, 4), 64),         # 1368 and two: the 64 x 64 tiles
    (5, (896, 392, 8, 4), 240),          # 520 tiles of the forward pass, 14,560 steps: the 64 x 64 tiles
])
def test_gradient_and_loss_match_oracle(m, dims, batch):
    """2e-2 in L2: a value on a bf16 rounding boundary may fall on either side of it."""
    cfg, X, labels, x0 = small_mlp_case(m, dims, batch, 1, seed=431)
    x0 = x0 + G.generic_normal(3, 1, x0.shape, sigma=0.02)
    g, losses = one_step(m, dims, batch, cfg, X, labels, x0)
    for i in sorted({0, m // 2, m - 1}):
        loss, grad = O.mlp_loss_grad(x0, dims, X[i, 0], labels[i, 0], bf16_operands=True)
        assert abs(losses[i] - loss) <= 1e-3 * abs(loss)
        assert l2_ratio(g[i], grad) <= 2e-2


def test_infinite_weight_stays_in_its_column():
    """Lanes past the contraction's end or past the last row or column hold zeros, and the two columns of a pair stay apart: an
    infinite weight reaches its own units only, forward and back."""
    m, dims, batch = 2, (24, 24, 24, 4), 8
    cfg, X, labels, x0 = small_mlp_case(m, dims, batch, 1, seed=432)
    inf = 24 * 24 + 24                   # second layer's weight [0][0], right behind the first layer's bias
    x0 = x0.copy()
    x0[24 * 24:inf] = -100.0             # first layer: no unit is active ..
    x0[24 * 24 + 1:inf] = 1.0            # .. but those after the first
    x0[inf] = np.inf
    g, losses = one_step(m, dims, batch, cfg, X, labels, x0)
    # 0 * inf is a NaN in the second layer's first unit, which the ReLU takes to 0, and going back in the delta of the first
    # layer's first unit, which is gated to 0; everything else is as with both units inactive
    ref = x0.copy()
    ref[inf] = 0.0
    ref[inf + 24 * 24] = -1e6            # that unit inactive
    for i in range(m):
        loss, grad = O.mlp_loss_grad(ref, dims, X[i, 0], labels[i, 0], bf16_operands=True)
        assert abs(losses[i] - loss) <= 1e-3 * abs(loss)
        assert l2_ratio(g[i], grad) <= 2e-2
