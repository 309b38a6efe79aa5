"""GPU parity of the fp32 MLP where its forward and delta GEMMs take the kernel of small launches: tiles, contraction steps and
groups of steps requested together that are whole or not, both tile widths, and an infinite weight."""
import numpy as np
import pytest

from ols_inputs import generate as G
from oracle import ols_oracle as O
from tests.helpers import l2_ratio, max_norm_ratio
from tests.test_gpu_gemm_split import GRAD_TOL, first_activations, one_step
from tests.test_gpu_mlp import small_mlp_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,dims,batch", [
    (2, (4, 4, 4, 3), 4),                # a quarter of one step, four rows
    (3, (128, 36, 20, 5), 36),           # two steps per wavefront; four rows and four columns more than a tile
    (2, (132, 300, 124, 7), 36),         # one step of four indices more
    (1, (512, 16, 516, 3), 32),          # a whole group of eight steps; contractions of one step and of 33
    (2, (520, 48, 16, 3), 20),           # nine steps per wavefront: two groups of five
    (2, (2060, 24, 8, 4), 20),           # 33 steps per wavefront: five groups of seven
    (32, (360, 444, 8, 4), 24),          # 32 x 32 tiles, the last with 28 columns
    (2, (764, 40, 16, 3), 20),           # twelve steps per wavefront in one sum ..
    (2, (768, 40, 16, 3), 20),           # .. and in two
    (6, (32, 1160, 1376, 4), 80),        # a delta of 1314 tiles, 113,004 steps: one round of 64 x 64 tiles instead
    (6, (760, 384, 92, 6), 164),         # 32 x 32 tiles over two groups of steps, rows no multiple of a tile
])
def test_gradient_and_loss_match_oracle(m, dims, batch):
    cfg, X, labels, x0 = small_mlp_case(m, dims, batch, 1, seed=421)
    x0 = x0 + G.generic_normal(3, 1, x0.shape, sigma=0.02)
    g, losses = one_step(cfg, dims, batch, X, labels, x0)
    for i in sorted({0, m // 2, m - 1}):
        loss, grad = O.mlp_loss_grad(x0, dims, X[i, 0], labels[i, 0])
        assert abs(losses[i] - loss) <= 1e-5 * abs(loss)
        assert max_norm_ratio(g[i], grad) <= GRAD_TOL


def test_infinite_weight_stays_in_its_column():
    """Lanes past the contraction's end (20 indices: a second step of four) and past the last row or column hold zeros, not a
    neighbour's value: an infinite weight reaches its own units only, forward and back."""
    m, dims, batch = 2, (20, 20, 20, 4), 4
    cfg, X, labels, x0 = small_mlp_case(m, dims, batch, 1, seed=422)
    inf = 20 * 20 + 20                   # second layer's weight [0][0], right behind the first layer's bias
    x0 = x0.copy()
    x0[20 * 20:inf] = -100.0             # first layer: no unit is active ..
    x0[20 * 20 + 1:inf] = 1.0            # .. but those after the first
    x0[inf] = np.inf
    g, losses = one_step(cfg, dims, batch, X, labels, x0)
    # 0 * inf is a NaN in the second layer's first unit, which the ReLU takes to 0 as before, and going back in the delta of the
    # first layer's first unit, which is gated to 0; everything else is as with both units inactive
    ref = x0.copy()
    ref[inf] = 0.0
    ref[inf + 20 * 20] = -1e6            # that unit inactive
    for i in range(m):
        loss, grad = O.mlp_loss_grad(ref, dims, X[i, 0], labels[i, 0])
        assert abs(losses[i] - loss) <= 1e-5 * abs(loss)
        assert max_norm_ratio(g[i], grad) <= GRAD_TOL


@pytest.mark.parametrize("m,batch,width,features", [
    (8, 24, 236, 2936),      # 32 x 16 tiles, groups of steps that overlap
    (3, 32, 1200, 912),      # 32 x 16 tiles, groups one behind the other
    (4, 28, 1924, 1872),     # 32 x 32 tiles
])
def test_long_contractions_are_added_in_eight_parts(m, batch, width, features):
    """A sum of n terms of random sign in one chain has an error of 0.3 u sqrt(n) of its own root mean square: each addition rounds a
    partial sum that has grown to sqrt(k) of a term by 0.42 u of it in the root mean square, u = 2^-24.  P chains of K / P terms
    leave 0.3 u sqrt(K / P), the additions that follow less than u.  The 64 x 64 tiles add these contractions in eight ranges;
    the bound lies a fifth above eight chains and a sixth below four."""
    dims = (features, width, 4)
    cfg, X, labels, x0 = small_mlp_case(m, dims, batch, 1, seed=423)
    X = G.generic_normal(11, 2, X.shape)          # (class means would lengthen the sums)
    h = first_activations(cfg, dims, batch, X, labels, x0)
    W = x0[:features * width].reshape(features, width).astype(np.float64)
    ref = np.maximum(X[:, 0].astype(np.float64) @ W + x0[features * width:features * width + width], 0.0)
    bound = 2.0 ** -24 * (1.2 * 0.3 * np.sqrt(features / 8) + 0.42)
    assert l2_ratio(h, ref) <= bound
