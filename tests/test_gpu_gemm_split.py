"""GPU parity of the fp32 MLP where its forward GEMMs run on the bf16 matrix cores with split operands: ragged rows,
columns and contractions of the launches large enough for that route, K ranges with a short last one, operands at the ends
of the fp32 range, and an infinity that must stay one."""
import numpy as np
import pytest

from ols_inputs import generate as G
from oracle import ols_oracle as O
from tests.helpers import max_norm_ratio
from tests.test_gpu_mlp import make_session, small_mlp_case

from paper_2002_09539_amd import binding as B

pytestmark = pytest.mark.gpu

GRAD_TOL = 2e-5      # fp32 accumulation against the fp64 oracle, max-norm relative


def one_step(cfg, dims, batch, X, labels, x0):
    with make_session(cfg.m, cfg.d, 2, 0.6, 0.05, 0.0) as s:
        s.set_option(B.OLS_OPT_FUSE_GEMM_UPDATE, 0)     # keep the gradients in g so they can be read
        s.attach_mlp(dims, batch, "f32")
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_batch(Xd[:, 0], yd[:, 0])
        s.local_step()
        return s.gradient(), s.losses()


@pytest.mark.parametrize("m,dims,batch", [
    (16, (2048, 512, 10), 124),         # 128 tiles over four K ranges; ragged rows
    (22, (2060, 260, 5), 68),           # 132 tiles, the last K range short and no whole number of slices; ragged columns
    (32, (1060, 516, 5), 68),           # 320 tiles over one range
    (64, (36, 1028, 516, 3), 8),        # contractions of 36 (two slices, the second of four indices) and 1028
    (43, (128, 772, 7), 128),           # exactly one group of four slices; a last column tile of four
])
def test_gradient_and_loss_match_oracle(m, dims, batch):
    cfg, X, labels, x0 = small_mlp_case(m, dims, batch, 1, seed=411)
    x0 = x0 + G.generic_normal(3, 1, x0.shape, sigma=0.02)
    g, losses = one_step(cfg, dims, batch, X, labels, x0)
    for i in (0, m // 2, m - 1):
        loss, grad = O.mlp_loss_grad(x0, dims, X[i, 0], labels[i, 0])
        assert abs(losses[i] - loss) <= 1e-5 * abs(loss)
        assert max_norm_ratio(g[i], grad) <= GRAD_TOL


@pytest.mark.parametrize("e", [60, 100])
def test_operands_over_the_exponent_range(e):
    """A batch scaled down and first-layer weights scaled up by 2^e: the products stay of order one."""
    m, dims, batch = 64, (64, 1024, 10), 16
    cfg, X, labels, x0 = small_mlp_case(m, dims, batch, 1, seed=412)
    X, x0 = np.ldexp(X, -e).astype(np.float32), x0.copy()
    n_w = dims[0] * dims[1]
    x0[:n_w] = np.ldexp(x0[:n_w], e)
    g, losses = one_step(cfg, dims, batch, X, labels, x0)
    for i in (0, m - 1):
        loss, grad = O.mlp_loss_grad(x0, dims, X[i, 0], labels[i, 0])
        assert abs(losses[i] - loss) <= 1e-5 * abs(loss)
        for sl in (slice(0, n_w), slice(n_w, None)):
            assert max_norm_ratio(g[i][sl], grad[sl]) <= GRAD_TOL


def test_an_infinity_stays_one():
    """A feature that is infinite makes the units it reaches through positive weights infinite (a NaN from inf - inf inside
    a split would leave the ReLU as 0 and the loss finite); the other workers are untouched.  Values next to the largest
    finite one, which round to a bf16 infinity, must stay finite."""
    m, dims, batch = 64, (64, 1024, 10), 16
    cfg, X, labels, x0 = small_mlp_case(m, dims, batch, 1, seed=413)
    big = np.float32(3.4e38)
    X = X.copy()
    X[0, 0, 3, 5] = np.inf
    X[1, 0, 2, 7] = big
    x0 = x0.copy()
    x0[7 * dims[1]:8 * dims[1]] *= np.float32(2.0 ** -100)     # feature 7's weights (not below 2^-109: their last term must be a normal bf16)
    g, losses = one_step(cfg, dims, batch, X, labels, x0)
    assert not np.isfinite(losses[0])
    for i in (1, 2, m - 1):
        loss, grad = O.mlp_loss_grad(x0, dims, X[i, 0], labels[i, 0])
        assert abs(losses[i] - loss) <= 1e-5 * abs(loss)
        assert max_norm_ratio(g[i], grad) <= GRAD_TOL


def first_activations(cfg, dims, batch, X, labels, x0):
    """The first hidden layer's activations [m][batch][dims[1]] of one step: they come first in the workspace."""
    with make_session(cfg.m, cfg.d, 2, 0.6, 0.05, 0.0) as s:
        s.attach_mlp(dims, batch, "f32")
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_batch(Xd[:, 0], yd[:, 0])
        s.local_step()
        s.sync()
        n = cfg.m * batch * dims[1]
        return s.ws[:4 * n].cpu().numpy().view(np.float32).reshape(cfg.m, batch, dims[1])


@pytest.mark.parametrize("m,dims,batch", [(64, (64, 1024, 10), 16), (16, (2048, 512, 10), 124)])   # one K range, and four
def test_every_unit_that_an_infinity_reaches(m, dims, batch):
    """Per unit: infinite where the weight is positive, zero (ReLU of the negative infinity) where it is negative, for weights
    that are exact in bf16, that leave positive or negative remainders and that are generic; likewise finite operands whose
    product overflows.  Every other sample is as near to 64 bits as without."""
    cfg, X, labels, x0 = small_mlp_case(m, dims, batch, 1, seed=414)
    X, x0 = X.copy(), x0.copy()
    W = x0[:dims[0] * dims[1]].reshape(dims[0], dims[1])
    kinds = np.array([1.0, 1.0 + 2.0 ** -9 + 2.0 ** -18, 2.0 - 2.0 ** -10, 1.7, -1.0, -1.3], np.float32)
    w = kinds[np.arange(dims[1]) % len(kinds)]
    W[5], W[7] = w, np.ldexp(w, 40)
    X[:, 0, :, 7] = 0.0
    X[0, 0, 3, 5] = np.inf
    X[1, 0, 2, 7] = 3e38
    h = first_activations(cfg, dims, batch, X, labels, x0)
    want = np.where(w > 0, np.inf, 0.0)
    assert np.array_equal(h[0, 3], want) and np.array_equal(h[1, 2], want)
    bias = x0[dims[0] * dims[1]:dims[0] * dims[1] + dims[1]].astype(np.float64)
    for i in (0, 1, m - 1):
        rows = [r for r in range(batch) if (i, r) not in ((0, 3), (1, 2))]
        ref = np.maximum(X[i, 0, rows].astype(np.float64) @ W.astype(np.float64) + bias, 0.0)
        assert max_norm_ratio(h[i, rows], ref) <= GRAD_TOL


def test_order_of_the_products():
    """A first layer that goes by column strips adds the indices 4 .. 7 and 8 .. 11 of every sixteen in each other's place; any other layer
    adds them as they come.  So the strips' product of the first samples is, to the bit, the plain one with those places exchanged."""
    m, dims, few, many = 64, (512, 512, 3), 64, 256       # strips take up to 128 samples
    cfg, X, labels, x0 = small_mlp_case(m, dims, many, 1, seed=415)
    n_w = dims[0] * dims[1]
    place = np.arange(dims[0]).reshape(-1, 4, 4)[:, [0, 2, 1, 3]].reshape(-1)
    moved = x0.copy()
    moved[:n_w] = x0[:n_w].reshape(dims[0], dims[1])[place].reshape(-1)
    strips = first_activations(cfg, dims, few, X[:, :, :few], labels[:, :, :few], x0)
    plain = first_activations(cfg, dims, many, X, labels, x0)[:, :few]
    exchanged = first_activations(cfg, dims, many, X[..., place], labels, moved)[:, :few]
    assert np.array_equal(strips, exchanged)
    assert not np.array_equal(strips, plain) and max_norm_ratio(strips, plain) <= GRAD_TOL
