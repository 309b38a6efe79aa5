"""The forward / delta tiles of the bf16 block that only launches of many tiles take (512 x 64 and 256 x 64), against the small
launch's 256 x 32 that the oracle tests cover: the same worker alone and as one of many identical ones.  A tile's size leaves
the order of a convolution's sum as it is; the pooling's sums of 64 pixels are added over four or eight lanes, and the kernel
gradients over other pixel ranges."""
import numpy as np
import pytest

from ols_inputs import generate as G
from tests.helpers import l2_ratio, max_norm_ratio
from tests.test_gpu_conv_bf16 import conv_case, groups_of, make_session

pytestmark = pytest.mark.gpu


def one_step(cfg, dims, batch, m, X, labels, x0, batch_norm):
    with make_session(m, x0.size, 2, 0.6, 0.05, 0.0) as s:
        s.attach_convblock(*dims, batch, gemm_dtype="bf16", batch_norm=batch_norm)
        Xd = s.upload(np.repeat(X[:1, 0], m, axis=0))
        yd = s.upload(np.repeat(labels[:1, 0], m, axis=0))
        s.init_params(x0)
        s.set_batch(Xd, yd)
        s.local_step()
        return s.gradient(), s.losses()


@pytest.mark.parametrize("dims,batch,m", [
    ((64, 30, 30, 5), 8, 28),      # 16 tiles of 512 pixels per worker, 448 in all
    ((64, 14, 49, 4), 10, 26),     # the widest strip of a 512-pixel tile that two workgroups per compute unit hold
    ((64, 14, 50, 4), 10, 26),     # one column more: 256 x 64
    ((64, 9, 33, 3), 12, 45),      # 4620 padded pixels: a last tile of 12 pixels
    ((128, 13, 15, 7), 20, 21),    # two contraction chunks, two output tiles
    ((256, 14, 14, 5), 16, 8),     # four of each; 256 tiles, where fewer channels would take the kernel slices through LDS
    ((256, 14, 14, 5), 16, 13),    # 416 tiles
])
def test_tile_of_a_large_launch(dims, batch, m):
    cfg, X, labels, x0 = conv_case(1, dims, batch, 1, seed=717)
    x0 = x0 + G.generic_normal(7, 6, x0.shape, sigma=0.02)
    g1, l1 = one_step(cfg, dims, batch, 1, X, labels, x0, False)
    g, losses = one_step(cfg, dims, batch, m, X, labels, x0, False)
    # Pooled features: at most 64 + 63 additions per part and image in another order, 2^-24 of the (non-negative) sum each.  The
    # classifier's gradients are linear in them, with weights that sum to at most B; losses and logits likewise, C terms.
    bound = 128 * 2.0 ** -24
    for i in (0, m // 2, m - 1):
        assert abs(losses[i] - l1[0]) <= bound * max(1.0, abs(l1[0]))
        for name, sl in groups_of(dims[0], dims[3]).items():
            sl = sl.ravel()
            if name in ("Wh", "bh"):
                assert max_norm_ratio(g[i][sl], g1[0][sl]) <= 8 * bound, name
            else:   # a last bit of the pooled delta can move it over a bf16 rounding boundary: 0.4 % of one channel of a sample
                assert l2_ratio(g[i][sl], g1[0][sl]) <= 1e-2, name


@pytest.mark.parametrize("dims,batch,m", [((64, 30, 30, 5), 8, 28), ((64, 14, 50, 4), 10, 26), ((128, 13, 15, 7), 20, 21)])
def test_normalised_block(dims, batch, m):
    """The outputs for a batch normalisation.  Its statistics are merged in chunks whose number depends on the launch, and their
    last bit moves values over a bf16 rounding boundary (0.4 % of the value): the oracle tests' bound for such changes."""
    cfg, X, labels, _ = conv_case(1, dims, batch, 1, seed=718)
    C, classes = dims[0], dims[3]
    rng = np.random.default_rng(5)
    kernels = lambda: (rng.standard_normal(9 * C * C) / np.sqrt(9 * C)).astype(np.float32)   # noqa: E731
    x0 = np.concatenate([kernels(), np.ones(C), 0.02 * rng.standard_normal(C), kernels(), np.ones(C), 0.02 * rng.standard_normal(C),
                         rng.standard_normal(C * classes) / np.sqrt(C), np.zeros(classes)]).astype(np.float32)
    g1, l1 = one_step(cfg, dims, batch, 1, X, labels, x0, True)
    g, losses = one_step(cfg, dims, batch, m, X, labels, x0, True)
    for i in (0, m - 1):
        assert abs(losses[i] - l1[0]) <= 1e-4 * abs(l1[0])
        assert l2_ratio(g[i], g1[0]) <= 1e-2
