"""GPU parity of the fp32 residual block where its convolutions run on the bf16 matrix cores with every operand split into
three bf16 terms: tile and range edges, channel counts off the 64-channel blocks, the widest and the smallest images that
route takes and the first ones it leaves, values at the ends of the fp32 range.  The bars are those of the fp32 route."""
import numpy as np
import pytest

from oracle import conv_oracle as CO
from tests.helpers import max_norm_ratio
from tests.test_gpu_conv_bn import bn_case, groups_of as bn_groups_of, one_step as bn_one_step
from tests.test_gpu_conv_bn import GRAD_TOL as BN_GRAD_TOL
from tests.test_gpu_conv import GRAD_TOL, conv_case, groups_of, make_session

pytestmark = pytest.mark.gpu

SHAPES = [
    (2, (32, 16, 16, 4), 1, 11),     # 256 pixels: exactly two tiles, half an output-channel tile
    (1, (96, 5, 7, 5), 3, 11),       # 105 pixels: a ragged tile; three chunks, one and a half channel blocks
    (3, (64, 2, 2, 3), 40, 12),      # the smallest images: 32 of them in a tile
    (2, (64, 3, 60, 4), 1, 11),      # the widest strips
    (1, (64, 3, 62, 4), 1, 11),      # one column too wide: the fp32 matrix cores
    (1, (32, 1, 30, 3), 3, 11),      # too low for its width: the fp32 matrix cores
    (1, (32, 2, 50, 3), 2, 11),
    (2, (32, 3, 30, 3), 2, 11),      # one row more: a strip of 259 rows
    (1, (64, 1, 1, 3), 4, 11),       # single positions: the fp32 matrix cores
    (1, (32, 31, 33, 4), 9, 11),     # 9207 pixels: thirteen ranges of the kernel gradient, ring wraps, ragged last slice
    (1, (160, 6, 5, 3), 2, 11),      # five chunks, three channel blocks
]


def plain_step(cfg, dims, batch, X, labels, x0):
    with make_session(cfg.m, cfg.d, 2, 0.6, 0.05, 0.0) as s:
        s.attach_convblock(*dims, batch)
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_batch(Xd[:, 0], yd[:, 0])
        s.local_step()
        return s.gradient(), s.losses()


@pytest.mark.parametrize("m,dims,batch,seed", SHAPES)
def test_plain_block(m, dims, batch, seed):
    cfg, X, labels, x0 = conv_case(m, dims, batch, 1, seed=seed)
    x0 = x0 + (0.05 * np.random.default_rng(seed).standard_normal(x0.shape)).astype(np.float32)
    # a ReLU input within single precision's rounding of zero may fall on either side
    assert min(CO.convblock_relu_margin(x0, dims[0], dims[3], X[i, 0]) for i in range(m)) >= 1e-6
    g, losses = plain_step(cfg, dims, batch, X, labels, x0)
    for i in range(m):
        loss, grad = CO.convblock_loss_grad(x0, dims[0], dims[3], X[i, 0], labels[i, 0])
        assert abs(losses[i] - loss) <= 1e-5 * abs(loss)
        for name, sl in groups_of(dims[0], dims[3]).items():
            sl = np.ravel(sl)
            assert max_norm_ratio(g[i][sl], grad[sl]) <= GRAD_TOL, "worker %d %s" % (i, name)


@pytest.mark.parametrize("m,dims,batch,seed", [
    (2, (64, 16, 16, 4), 1, 12),     # whole tiles: statistics of two tiles per worker
    (3, (64, 9, 9, 5), 5, 11),       # 405 pixels: the last tile's statistics over 21 rows
    (1, (128, 13, 11, 4), 4, 12),    # two channel blocks
    (2, (32, 10, 10, 4), 3, 11),     # 32 channels: the statistics read the output
])
def test_normalised_block(m, dims, batch, seed):
    cfg, X, labels, x0 = bn_case(m, dims, batch, 1, seed=seed)
    x0 = x0 + (0.05 * np.random.default_rng(seed).standard_normal(x0.shape)).astype(np.float32)
    assert min(CO.convblock_relu_margin(x0, dims[0], dims[3], X[i, 0], batch_norm=True) for i in range(m)) >= 1e-6
    g, losses = bn_one_step(cfg, dims, batch, X, labels, x0)
    for i in range(m):
        loss, grad = CO.convblock_bn_loss_grad(x0, dims[0], dims[3], X[i, 0], labels[i, 0])
        assert abs(losses[i] - loss) <= 1e-5 * abs(loss)
        for name, sl in bn_groups_of(dims[0], dims[3]).items():
            sl = np.ravel(sl)
            assert max_norm_ratio(g[i][sl], grad[sl]) <= BN_GRAD_TOL, "worker %d %s" % (i, name)


@pytest.mark.parametrize("e", [60, 100])
def test_operands_over_the_exponent_range(e):
    """A batch scaled down and a first kernel scaled up by 2^e: the products stay of order one, the shortcut vanishes, and
    the smallest terms of the split batch are near 2^-(e + 20)."""
    m, dims, batch = 1, (32, 6, 6, 4), 2
    cfg, X, labels, x0 = conv_case(m, dims, batch, 1, seed=13)
    X, x0 = np.ldexp(X, -e).astype(np.float32), x0.copy()
    n_w = 9 * dims[0] * dims[0]
    x0[:n_w] = np.ldexp(x0[:n_w], e)
    g, losses = plain_step(cfg, dims, batch, X, labels, x0)
    loss, grad = CO.convblock_loss_grad(x0, dims[0], dims[3], X[0, 0], labels[0, 0])
    assert abs(losses[0] - loss) <= 1e-5 * abs(loss)
    for name, sl in groups_of(dims[0], dims[3]).items():
        sl = np.ravel(sl)
        assert max_norm_ratio(g[0][sl], grad[sl]) <= GRAD_TOL, name


def test_an_infinity_stays_with_its_worker():
    """inf * finite must stay inf (no inf - inf inside a split): the activations that read the infinity through positive
    weights become inf and reach the second kernel's gradient -- a NaN there would have left the ReLU (fmaxf) as 0 and the
    gradient finite.  The other worker is untouched."""
    m, dims, batch = 2, (32, 6, 6, 4), 3
    cfg, X, labels, x0 = conv_case(m, dims, batch, 1, seed=14)
    X = X.copy()
    X[0, 0, 1, 2, 3, 5] = np.inf
    g, losses = plain_step(cfg, dims, batch, X, labels, x0)
    assert not np.isfinite(g[0][np.ravel(groups_of(dims[0], dims[3])["Wb"])]).all()
    loss, grad = CO.convblock_loss_grad(x0, dims[0], dims[3], X[1, 0], labels[1, 0])
    assert abs(losses[1] - loss) <= 1e-5 * abs(loss)
    assert max_norm_ratio(g[1], grad) <= GRAD_TOL


def tensor_of(s, index, m, dims, batch):
    """Activation-sized tensor [m][batch][H][W][C] number `index` of the workspace: a1, a2, delta at z2, delta at z1."""
    C, H, W, _ = dims
    n = m * batch * H * W * C
    first = index * (-(-4 * n // 256) * 256)
    return s.ws[first:first + 4 * n].cpu().numpy().view(np.float32).reshape(m, batch, H, W, C)


def test_every_activation_that_an_infinity_reaches():
    """Per unit of the first layer: infinite where the weight of its one tap is positive, zero where it is negative, for weights
    that are exact in bf16, that leave positive or negative remainders and that are generic."""
    m, dims, batch = 2, (32, 6, 6, 4), 3
    cfg, X, labels, x0 = conv_case(m, dims, batch, 1, seed=15)
    C = dims[0]
    X, x0 = X.copy(), x0.copy()
    Wa = x0[:9 * C * C].reshape(3, 3, C, C)
    kinds = np.array([1.0, 1.0 + 2.0 ** -9 + 2.0 ** -18, 2.0 - 2.0 ** -10, 1.7, -1.0, -1.3], np.float32)
    Wa[:, :, 5, :] = kinds[np.arange(9 * C).reshape(3, 3, C) % len(kinds)]
    X[0, 0, 1, 2, 3, 5] = np.inf
    with make_session(m, cfg.d, 2, 0.6, 0.05, 0.0) as s:
        s.attach_convblock(*dims, batch)
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_batch(Xd[:, 0], yd[:, 0])
        s.local_step()
        s.sync()
        a1 = tensor_of(s, 0, m, dims, batch)
    for dy in range(3):
        for dx in range(3):       # output (y, x) reads input (y + dy - 1, x + dx - 1)
            want = np.where(Wa[dy, dx, 5] > 0, np.inf, 0.0)
            assert np.array_equal(a1[0, 1, 2 - (dy - 1), 3 - (dx - 1)], want), (dy, dx)
    reached = np.zeros(a1.shape, bool)
    reached[0, 1, 1:4, 2:5] = True
    assert np.isfinite(a1[~reached]).all()


def test_deltas_and_kernel_gradients_past_the_range():
    """A block of positive numbers whose delta at z1 overflows: each of its elements is +inf, and so is the sum of the first
    kernel's gradient that meets no padding (the centre tap)."""
    m, dims, batch = 1, (32, 6, 6, 2), 2
    cfg, X, labels, x0 = conv_case(m, dims, batch, 1, seed=16)
    C, rng = dims[0], np.random.default_rng(16)
    near_one = lambda shape: (1.0 + 0.9 * rng.random(shape)).astype(np.float32)   # noqa: E731
    X = np.ldexp(near_one(X.shape), -36)
    parts = groups_of(C, dims[3])
    x0 = np.zeros_like(x0)
    x0[np.ravel(parts["Wa"])] = near_one(9 * C * C) / (9 * C)
    x0[np.ravel(parts["Wb"])] = np.ldexp(near_one(9 * C * C), 96)
    Wh = np.zeros((C, 2), np.float32)
    Wh[:, 0] = np.ldexp(near_one(C), 48)           # class 0 wins, every label is 1: its delta is 1 / batch
    x0[np.ravel(parts["Wh"])] = Wh.ravel()
    labels = np.ones_like(labels)
    with make_session(m, cfg.d, 2, 0.6, 0.05, 0.0) as s:
        s.attach_convblock(*dims, batch)
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_batch(Xd[:, 0], yd[:, 0])
        s.local_step()
        g = s.gradient()[0]
        dz2, dz1 = (tensor_of(s, k, m, dims, batch) for k in (2, 3))
    assert np.isfinite(dz2).all() and (dz2 > 0).all()
    assert (dz1 == np.inf).all()
    centre = g[np.ravel(parts["Wa"])].reshape(9, C, C)[4]
    assert (centre == np.inf).all()


def test_a_nan_pixel_stays_out_of_the_taps_that_never_read_it():
    """A NaN in an image's corner leaves the ReLU as 0, so the loss is finite; the first kernel's gradient is NaN in the four
    taps that read the corner from inside the image and nowhere else (where there is no pixel the delta counts as zero, and
    NaN times that zero must not be added)."""
    m, dims, batch = 1, (32, 13, 11, 4), 9        # eight pixel ranges
    cfg, X, labels, x0 = conv_case(m, dims, batch, 1, seed=17)
    C, H, W, _ = dims
    X = X.copy()
    X[0, 0, 4, 0, 0, 5] = np.nan
    with make_session(m, cfg.d, 2, 0.6, 0.05, 0.0) as s:
        s.attach_convblock(*dims, batch)
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_batch(Xd[:, 0], yd[:, 0])
        s.local_step()
        g, losses = s.gradient()[0], s.losses()
        dz1 = tensor_of(s, 3, m, dims, batch)[0].astype(np.float64)
    assert np.isfinite(losses[0]) and np.isfinite(dz1).all()
    got = g[np.ravel(groups_of(C, dims[3])["Wa"])].reshape(3, 3, C, C)
    pad = np.zeros((batch, H + 2, W + 2, C))
    pad[:, 1:-1, 1:-1] = X[0, 0]
    for i in range(3):
        for j in range(3):
            want = pad[:, i:i + H, j:j + W].reshape(-1, C).T @ dz1.reshape(-1, C)
            assert np.array_equal(np.isnan(want[5]), np.full(C, i < 2 and j < 2))
            assert np.array_equal(np.isnan(got[i, j]), np.isnan(want)), (i, j)
            rows = ~np.isnan(want[:, 0])
            assert max_norm_ratio(got[i, j][rows], want[rows]) <= GRAD_TOL
