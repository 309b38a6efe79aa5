"""The MLP's forward and delta GEMMs that go through LDS tiles, on launches above the work up to which the kernel of small launches
takes them.  That kernel's limits, in steps of a tile (32 x 32 and 32 indices in bf16, 32 x 16 and 16 in fp32):
  bf16 forward 8,000, or 15,000 from 640 indices on; bf16 delta 7,000, or 15,000 from 1024 on;
  fp32 forward 80,000, or 30,000 beyond 2048 indices; fp32 delta 80,000, or 160,000 from 1024 on.
Below, "small tiles" are 64 x 64; a bf16 launch takes them where it has fewer than 256 tiles of 128 x 128, and above that
256 x 128 for batches of more than 128."""
import numpy as np
import pytest

from ols_inputs import generate as G
from oracle import ols_oracle as O
from tests.helpers import l2_ratio, max_norm_ratio
from tests.test_gpu_gemm_split import GRAD_TOL, one_step as f32_step
from tests.test_gpu_gemm_small_bf16 import one_step as bf16_step
from tests.test_gpu_mlp import make_session, small_mlp_case

from paper_2002_09539_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,dims,batch", [
    # fp32, K ranges of 256 indices: forward 1020 -> 508 (98,304 steps; 192 small tiles, four ranges, the last of 252) and its delta
    (24, (68, 1020, 508, 6), 60),
    # forward 1580 -> 824 (108,108 steps): 182 tiles, ranges of 416 indices, the last of 332, which is no whole number of slices
    (7, (1580, 824, 8, 5), 92),
])
def test_fp32_small_tiles(m, dims, batch):
    cfg, X, labels, x0 = small_mlp_case(m, dims, batch, 1, seed=441)
    x0 = x0 + G.generic_normal(3, 1, x0.shape, sigma=0.02)
    g, losses = f32_step(cfg, dims, batch, X, labels, x0)
    for i in (0, m // 2, m - 1):
        loss, grad = O.mlp_loss_grad(x0, dims, X[i, 0], labels[i, 0])
        assert abs(losses[i] - loss) <= 1e-5 * abs(loss)
        assert max_norm_ratio(g[i], grad) <= GRAD_TOL


@pytest.mark.parametrize("m,dims,batch", [
    (4, (1032, 1000, 936, 10), 200),     # small tiles, ragged: forward 29,568 and 26,880 steps, delta 26,880
    (4, (1024, 1024, 1024, 10), 192),    # small tiles, whole: 24,576 steps each
    (255, (264, 128, 8, 4), 128),        # 255 tiles of 128 x 128: the most whose forward takes the small ones (36,720 steps)
    (256, (264, 128, 8, 4), 128),        # 256: 128 x 128
    (64, (136, 520, 504, 10), 120),      # 128 x 128, ragged: 320 and 256 tiles, delta 320
    (64, (128, 512, 512, 10), 128),      # 128 x 128, whole: 256 tiles each
    (16, (136, 1000, 904, 10), 200),     # 256 x 128, ragged: 256 tiles of 128 x 128 each
    (16, (128, 1024, 1024, 10), 256),    # 256 x 128, whole
])
def test_bf16_tiles(m, dims, batch):
    """Against the oracle with the same operand rounding: 2e-2 in L2 where a value may cross a bf16 rounding boundary."""
    cfg, X, labels, x0 = small_mlp_case(m, dims, batch, 1, seed=442)
    x0 = x0 + G.generic_normal(3, 1, x0.shape, sigma=0.02)
    g, losses = bf16_step(m, dims, batch, cfg, X, labels, x0)
    for i in sorted({0, m // 2, m - 1}):
        loss, grad = O.mlp_loss_grad(x0, dims, X[i, 0], labels[i, 0], bf16_operands=True)
        assert abs(losses[i] - loss) <= 1e-3 * abs(loss)
        assert l2_ratio(g[i], grad) <= 2e-2


@pytest.mark.parametrize("dtype,m,dims,batch", [
    ("f32", 24, (64, 1024, 512, 10), 64),         # forward 1024 -> 512 (98,304 steps, four K ranges) and its delta (98,304)
    ("bf16", 4, (1024, 1024, 1024, 10), 192),     # small tiles
    ("bf16", 64, (128, 512, 512, 10), 128),       # 128 x 128
    ("bf16", 16, (128, 1024, 1024, 10), 256),     # 256 x 128
])
def test_full_tile_kernels_match_bounds_checked_kernels_bit_for_bit(dtype, m, dims, batch):
    cfg, X, labels, x0 = small_mlp_case(m, dims, batch, 2, seed=443)
    states = []
    for force in (0, 1):
        with make_session(m, cfg.d, 2, 0.6, 0.05, 0.9) as s:
            s.set_option(B.OLS_OPT_GEMM_FORCE_GENERAL, force)
            s.attach_mlp(dims, batch, dtype)
            Xd, yd = s.upload(X), s.upload(labels)
            s.init_params(x0)
            losses = []
            s.run(3, lambda k: s.set_batch(Xd[:, k % 2], yd[:, k % 2]), losses=losses)
            states.append((s.all_params(), s.params(-1), s.momentum(), np.array(losses)))
    for a, b in zip(*states):
        assert np.array_equal(a, b)
