"""The fp32 MLP's first hidden layer by column strips: the gradients against the oracle, and the loop inside the library, whose
launches form the next step's product from the weights that they have just updated, against one call per step -- to the bit, over
ragged rows, columns and batches, one range of rows and several, and every rule of synchronisation."""
import numpy as np
import pytest

from ols_inputs import generate as G
from oracle import ols_oracle as O
from tests.helpers import max_norm_ratio
from tests.test_gpu_mlp import GRAD_TOL, make_session, small_mlp_case

from paper_2002_09539_amd import binding as B

pytestmark = pytest.mark.gpu

SHAPES = [
    (64, (324, 388, 10), 36),           # one range; six tiles, the last of four rows; a last strip of four columns
    (60, (520, 260, 36, 7), 64),        # whole batch blocks; another hidden layer; a last tile of eight rows
    (48, (840, 516, 5), 100),           # by halves of the samples; the last block of the batch is four samples
    (10, (2060, 388, 10), 72),          # several ranges, the last one short
    (12, (1856, 380, 24), 128),         # several ranges, whole batch; more than 16 classes
    (32, (1028, 640, 9), 4),            # the smallest batch
    (64, (520, 380, 36, 12, 7), 64),    # whole batch blocks and other hidden layers again
    (32, (1028, 896, 9), 4),            # the smallest batch again, on state beyond the memory-side cache in whole lines
    (60, (324, 1024, 10), 36),          # several rounds of strips, the same state
    (28, (616, 1024, 9), 128),          # by halves of a whole batch, the same state
    (108, (2000, 100, 10), 20),         # fewer columns than a strip; two ranges
]
# over how many ranges of the weights' rows they go by column strips (0: by other kernels), which test_mlp_strip_plan_cpu.py checks
RANGES = [1, 0, 1, 6, 6, 0, 1, 1, 1, 1, 2]


def case(m, dims, batch, nb, seed):
    cfg, X, labels, x0 = small_mlp_case(m, dims, batch, nb, seed)
    return cfg, X, labels, x0 + G.generic_normal(3, 1, x0.shape, sigma=0.02)


@pytest.mark.parametrize("m,dims,batch", SHAPES)
def test_gradient_and_loss_match_oracle(m, dims, batch):
    cfg, X, labels, x0 = case(m, dims, batch, 1, 511)
    with make_session(m, cfg.d, 2, 0.6, 0.05, 0.0) as s:
        s.set_option(B.OLS_OPT_FUSE_GEMM_UPDATE, 0)     # keep the gradients in g so they can be read
        s.attach_mlp(dims, batch, "f32")
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_batch(Xd[:, 0], yd[:, 0])
        s.local_step()
        g, losses = s.gradient(), s.losses()
    for i in (0, m // 2, m - 1):
        loss, grad = O.mlp_loss_grad(x0, dims, X[i, 0], labels[i, 0])
        assert abs(losses[i] - loss) <= 1e-5 * abs(loss)
        assert max_norm_ratio(g[i], grad) <= GRAD_TOL


def run(m, dims, batch, X, labels, x0, tau, K, library, mu=0.9, setup=lambda s: None, rule=None, beta_z=0.0, second=True):
    with make_session(m, x0.size, tau, 0.6, 0.05, mu, overlap_buffer=second) as s:
        if beta_z:
            s.set_anchor_momentum(beta_z)
        s.attach_mlp(dims, batch, "f32")
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        if rule == "stale":
            s.set_stale_average()
        elif rule == "mixing":
            w = np.zeros((m + 1, m + 1))
            w[:m, :m] = 0.5 * np.eye(m) + 0.5 / m
            w[:m, m] = 1.0 / m
            s.set_mixing(w)
        elif rule == "one_pass":
            s.set_option(B.OLS_OPT_FUSE_MEAN, 1)
        setup(s)
        if library:
            s.run_resident(K - 2, Xd, yd)
            s.run_resident(2, Xd, yd)
        else:
            s.run(K, lambda k: s.set_batch(Xd[:, k % X.shape[1]], yd[:, k % X.shape[1]]))
        out = [s.all_params(), s.params(-1), s.losses()]
        return out + ([s.momentum()] if mu else [])


def same(a, b):
    return all(np.array_equal(p, q, equal_nan=True) for p, q in zip(a, b))


@pytest.mark.parametrize("m,dims,batch", SHAPES)
@pytest.mark.parametrize("tau,mu", [(2, 0.9), (1, 0.0)])
def test_library_loop_equals_one_call_per_step(m, dims, batch, tau, mu):
    cfg, X, labels, x0 = case(m, dims, batch, 3, 512)
    a = run(m, dims, batch, X, labels, x0, tau, 7, True, mu)
    b = run(m, dims, batch, X, labels, x0, tau, 7, False, mu)
    assert same(a, b) and np.isfinite(a[0]).all() and not np.array_equal(a[0][0], x0)


@pytest.mark.parametrize("rule,kw", [
    ("stale", {}), ("mixing", {}), ("one_pass", {}), (None, dict(beta_z=0.7)), (None, dict(second=False)),
    (None, dict(setup=lambda s: s.set_option(B.OLS_OPT_NESTEROV, 0))),
    (None, dict(setup=lambda s: s.set_option(B.OLS_OPT_SERIALIZE, 0))),
    (None, dict(setup=lambda s: s.set_option(B.OLS_OPT_HEAD_DW_GUEST, 0))),
    (None, dict(setup=lambda s: s.set_option(B.OLS_OPT_FUSE_GEMM_UPDATE, 0))),
    (None, dict(setup=lambda s: s.set_option(B.OLS_OPT_KERNEL_TIMING, 1))),
])
@pytest.mark.parametrize("shape", [0, 3])
def test_every_rule_and_schedule(rule, kw, shape):
    m, dims, batch = SHAPES[shape]
    cfg, X, labels, x0 = case(m, dims, batch, 3, 513)
    a = run(m, dims, batch, X, labels, x0, 3, 8, True, rule=rule, **kw)
    b = run(m, dims, batch, X, labels, x0, 3, 8, False, rule=rule, **kw)
    assert same(a, b)


@pytest.mark.parametrize("shape", [0, 2])
def test_infinite_and_huge_values(shape):
    """Inputs and weights that round to a bf16 infinity, and infinities: the same bits, finite where they do not reach."""
    m, dims, batch = SHAPES[shape]
    cfg, X, labels, x0 = case(m, dims, batch, 2, 514)
    X = X.copy()
    X[0, 1, 1, 3] = 3.4e38
    X[1, 1, 2, dims[0] - 1] = np.inf
    X[2, 0, 0, 0] = -np.inf
    a = run(m, dims, batch, X, labels, x0, 2, 4, True)
    b = run(m, dims, batch, X, labels, x0, 2, 4, False)
    assert same(a, b)
    assert np.isnan(a[0][2]).any()
    solo = run(m, dims, batch, X, labels, x0, 4, 2, True)     # before any synchronisation the other workers are untouched
    assert np.isfinite(solo[0][3]).all() and np.isfinite(solo[0][m - 1]).all()


@pytest.mark.parametrize("e", [60, 100])
@pytest.mark.parametrize("small", ["batch", "delta"])
def test_gradients_over_the_exponent_range(small, e):
    """A batch scaled down and first-layer weights scaled up by 2^e, or the output layer's weights, and with them the delta, scaled
    down by 2^e: the split operands keep their bits while their last term is a normal bf16."""
    m, dims, batch = SHAPES[0]
    cfg, X, labels, x0 = case(m, dims, batch, 1, 518)
    X, x0, n_w = X.copy(), x0.copy(), dims[0] * dims[1]
    if small == "batch":
        X, x0[:n_w] = np.ldexp(X, -e).astype(np.float32), np.ldexp(x0[:n_w], e)
    else:
        w2 = slice(n_w + dims[1], n_w + dims[1] + dims[1] * dims[2])
        x0[w2] = np.ldexp(x0[w2], -e)
    with make_session(m, cfg.d, 2, 0.6, 0.05, 0.0) as s:
        s.set_option(B.OLS_OPT_FUSE_GEMM_UPDATE, 0)
        s.attach_mlp(dims, batch, "f32")
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_batch(Xd[:, 0], yd[:, 0])
        s.local_step()
        g, losses = s.gradient(), s.losses()
    for i in (0, m - 1):
        loss, grad = O.mlp_loss_grad(x0, dims, X[i, 0], labels[i, 0])
        assert abs(losses[i] - loss) <= 1e-5 * abs(loss)
        for sl in (slice(0, n_w), slice(n_w, n_w + dims[1]), slice(n_w + dims[1], None)):
            assert np.abs(grad[sl]).max() > 0.0 and max_norm_ratio(g[i][sl], grad[sl]) <= GRAD_TOL


@pytest.mark.parametrize("m,dims,batch", [(64, (324, 388, 36, 10), 36), (10, (2060, 388, 36, 10), 72)])   # last tiles of 4 and 12 rows
def test_infinite_delta(m, dims, batch):
    """A delta that overflows to an infinity: the updated weights are infinite and so is the next step's first activation.  The
    rows that the last tile does not have would be NaN (zero times the infinity) and must not reach it."""
    cfg, X, labels, _ = case(m, dims, batch, 2, 515)
    X, labels = np.abs(X) + np.float32(0.5), np.zeros_like(labels)
    big = np.float32(1e20)
    x0 = np.concatenate([np.concatenate([np.full(a * b, w, np.float32), np.full(b, v, np.float32)]) for a, b, w, v in
                         zip(dims, dims[1:], (0.0, -big, 0.0), (1e-30, 1e3, 0.0))])
    w3 = x0[-(dims[2] * dims[3] + dims[3]):-dims[3]].reshape(dims[2], dims[3])
    w3[:, 0] = -big                      # class 0 is never predicted and always right: the delta is 1e20 times -1e20
    a = run(m, dims, batch, X, labels, x0, 4, 2, True)
    b = run(m, dims, batch, X, labels, x0, 4, 2, False)
    assert np.isposinf(b[0][:, :dims[0] * dims[1]]).all()    # the weights that the infinite activations come from
    assert same(a, b)


def test_forced_ranges_of_the_forward_gemm():
    """OLS_OPT_GEMM_SPLITK holds for a layer whose strips are one range and whose plan has scratch for several."""
    m, dims, batch = 64, (520, 380, 36, 12, 7), 64
    cfg, X, labels, x0 = case(m, dims, batch, 1, 516)
    h = []
    for count in (1, 2, 4):
        with make_session(m, cfg.d, 2, 0.6, 0.05, 0.0) as s:
            s.set_option(B.OLS_OPT_GEMM_SPLITK, count)
            s.attach_mlp(dims, batch, "f32")
            Xd, yd = s.upload(X), s.upload(labels)
            s.init_params(x0)
            s.set_batch(Xd[:, 0], yd[:, 0])
            s.local_step()
            s.sync()
            h.append(s.ws[:4 * m * batch * dims[1]].cpu().numpy().view(np.float32).reshape(m, batch, dims[1]))
    W = x0[:dims[0] * dims[1]].reshape(dims[0], dims[1]).astype(np.float64)
    bias = x0[dims[0] * dims[1]:(dims[0] + 1) * dims[1]].astype(np.float64)
    for a in h:
        assert max_norm_ratio(a[3], np.maximum(X[3, 0].astype(np.float64) @ W + bias, 0.0)) <= GRAD_TOL
    assert not np.array_equal(h[0], h[1]) and not np.array_equal(h[1], h[2])    # sums over other ranges


@pytest.mark.parametrize("shape", [0, 3])
def test_timing_times_the_launches_of_the_loop(shape):
    """Per-kernel timing leaves the library's loop as it is: the first product of every step but a call's first comes with the
    weight gradient of the step before."""
    m, dims, batch = SHAPES[shape]
    cfg, X, labels, x0 = case(m, dims, batch, 2, 517)
    with make_session(m, cfg.d, 4, 0.6, 0.05, 0.9) as s:
        s.attach_mlp(dims, batch, "f32")
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_option(B.OLS_OPT_KERNEL_TIMING, 1)
        s.run_resident(3, Xd, yd)
        s.run_resident(2, Xd, yd)
        stats = s.kernel_stats()
        assert stats["gemm_fwd"][0] == 2 and stats["gemm_dw"][0] == 5 and stats["head_fwd"][0] == 5


@pytest.mark.parametrize("tau,delay,serialize,products", [
    (1, 50, 0, 4),     # nothing else of a round to hide behind: every step's forward GEMM beside the refresh
    (1, 50, 1, 1),     # blocking: nothing to hide
    (2, 200, 0, 2),    # longer than the round's other step (64 x 130,000 element-replicas, 67 us at the rule's rate): the first step of each round
    (2, 10, 0, 1),     # shorter
    (1, 0, 0, 1),
])
def test_forward_gemms_that_an_emulated_latency_hides_behind(tau, delay, serialize, products):
    m, dims, batch = SHAPES[0]
    cfg, X, labels, x0 = case(m, dims, batch, 2, 519)
    options = [(B.OLS_OPT_SERIALIZE, serialize), (B.OLS_OPT_ANCHOR_DELAY_US, delay)]
    with make_session(m, cfg.d, tau, 0.6, 0.05, 0.9) as s:
        for key, value in options:
            s.set_option(key, value)
        s.attach_mlp(dims, batch, "f32")
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_option(B.OLS_OPT_KERNEL_TIMING, 1)
        s.run_resident(4, Xd, yd)
        assert s.kernel_stats()["gemm_fwd"][0] == products
    setup = lambda s: [s.set_option(key, value) for key, value in options]   # noqa: E731
    a = run(m, dims, batch, X, labels, x0, tau, 6, True, setup=setup)
    assert same(a, run(m, dims, batch, X, labels, x0, tau, 6, False, setup=setup)) and same(a, run(m, dims, batch, X, labels, x0, tau, 6, True))
