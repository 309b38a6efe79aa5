"""GPU parity of the convolutional workload (3 x 3 implicit-GEMM convolutions on the fp32 matrix cores, pooling,
classifier) against the CPU oracle (oracle/conv_oracle.py), through the C boundary: gradients and loss of one step at
ragged and tile-sized shapes, whole Overlap Local-SGD runs, and the schedule variants."""
import numpy as np
import pytest

import ols_inputs as I
from ols_inputs import generate as G
from oracle import conv_oracle as CO
from oracle import workloads as OW
from tests.helpers import l2_ratio, max_norm_ratio

from paper_2002_09539_amd import binding as B

pytestmark = pytest.mark.gpu

GRAD_TOL = 2e-5     # fp32 MFMA accumulation against the fp64 oracle, max-norm relative per parameter group
E2E_TOL = 1e-3      # the benchmark specification's bar for fp32 end-to-end parameters


def make_session(*a, **kw):
    from paper_2002_09539_amd.session import Session
    return Session(*a, **kw)


def conv_case(m, dims, batch, nb, seed, **kw):
    cfg = I.get(6).scaled(m=m, dims=tuple(dims), batch=batch, nb=nb, seed=seed, **kw)
    X, labels = G.conv_data(cfg)
    return cfg, X, labels, G.conv_init(cfg)


def groups_of(C, classes):
    idx = np.arange(CO.convblock_param_count(C, classes))
    return dict(zip(("Wa", "ba", "Wb", "bb", "Wh", "bh"), CO.convblock_unpack(idx, C, classes)))


@pytest.mark.parametrize("m,dims,batch", [
    (2, (16, 5, 6, 4), 3),        # ragged everywhere: 90 pixels, one 16-channel slice per tap
    (3, (32, 8, 8, 10), 5),       # 320 pixels: several row tiles with a tail, 32-channel slices
    (2, (48, 7, 9, 10), 4),       # 48 channels: 16-wide slices, column tile with a tail
    (2, (80, 6, 6, 7), 3),        # more than 64 channels: two column tiles, 2 x 2 blocks of the kernel gradient
    (2, (64, 32, 32, 10), 6),     # the benchmark's per-image shape (64 channels, 32 x 32), several pixel ranges
    (14, (80, 5, 10, 4), 12),     # 168 blocks over two ranges of the kernel gradient: two workgroups on some units, one on others
    (1, (16, 1, 1, 3), 2),        # a single position: every tap but the centre falls outside
    (2, (16, 40, 3, 5), 2),       # narrow images: rows shorter than a K slice of the weight-gradient contraction
])
def test_gradient_and_loss_match_oracle(m, dims, batch):
    cfg, X, labels, x0 = conv_case(m, dims, batch, 1, seed=111)
    x0 = x0 + G.generic_normal(7, 3, x0.shape, sigma=0.02)      # non-zero biases as well
    with make_session(m, cfg.d, 2, 0.6, 0.05, 0.0) as s:
        s.attach_convblock(*dims, batch)
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_batch(Xd[:, 0], yd[:, 0])
        s.local_step()
        g, losses = s.gradient(), s.losses()
    for i in range(m):
        loss, grad = CO.convblock_loss_grad(x0, dims[0], dims[3], X[i, 0], labels[i, 0])
        assert abs(losses[i] - loss) <= 1e-5 * abs(loss)
        for name, sl in groups_of(dims[0], dims[3]).items():
            sl = sl.ravel()
            assert max_norm_ratio(g[i][sl], grad[sl]) <= GRAD_TOL, "worker %d %s" % (i, name)


@pytest.mark.parametrize("m,dims,batch,tau,K", [(3, (16, 6, 5, 4), 4, 2, 7), (2, (32, 8, 8, 10), 8, 3, 6)])
def test_small_runs_match_oracle(m, dims, batch, tau, K):
    cfg, X, labels, x0 = conv_case(m, dims, batch, 2, seed=222, tau=tau)
    st = OW.run_config(cfg, x0, OW.conv_grad_fn(cfg.dims, X, labels), K=K)
    with make_session(m, cfg.d, tau, cfg.alpha, cfg.gamma, cfg.mu) as s:
        s.attach_convblock(*dims, batch)
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        losses = []
        s.run(K, lambda k: s.set_batch(Xd[:, k % 2], yd[:, k % 2]), losses=losses)
        x, z, buf = s.all_params(), s.params(-1), s.momentum()
    assert max(l2_ratio(x[i], st["x"][i]) for i in range(m)) <= E2E_TOL
    assert max(l2_ratio(buf[i], st["buf"][i]) for i in range(m)) <= E2E_TOL
    assert l2_ratio(z, st["z"]) <= E2E_TOL
    np.testing.assert_allclose(np.array(losses), st["losses"], rtol=1e-3)


def test_full_shape_short_run_matches_oracle():
    """The benchmark's per-worker shape (64 channels, 32 x 32, batch 128) on 2 of the 16 workers for one round, in the
    launch configuration the benchmark times (ols_run_steps over the resident data)."""
    cfg = I.get(6).scaled(m=2, nb=2, K=2)
    X, labels = G.conv_data(cfg)
    x0 = G.conv_init(cfg)
    st = OW.run_config(cfg, x0, OW.conv_grad_fn(cfg.dims, X, labels))
    with make_session(cfg.m, cfg.d, cfg.tau, cfg.alpha, cfg.gamma, cfg.mu) as s:
        s.attach_convblock(*cfg.dims, cfg.batch)
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.run_resident(cfg.K, Xd, yd)
        x, z, losses = s.all_params(), s.params(-1), s.losses()
    assert max(l2_ratio(x[i], st["x"][i]) for i in range(cfg.m)) <= E2E_TOL
    assert l2_ratio(z, st["z"]) <= E2E_TOL
    np.testing.assert_allclose(losses, st["losses"][-1], rtol=1e-3)


def test_schedule_variants_and_library_loop_are_bit_identical():
    m, dims, batch, tau, K = 3, (32, 6, 6, 5), 4, 2, 7
    cfg, X, labels, x0 = conv_case(m, dims, batch, 2, seed=333)
    outs = []
    for opts, library in (((), True), ((), False), (((B.OLS_OPT_SERIALIZE, 1),), True),
                          (((B.OLS_OPT_ANCHOR_DELAY_US, 2000),), True), (((B.OLS_OPT_FUSE_PULL, 0),), True)):
        with make_session(m, cfg.d, tau, cfg.alpha, cfg.gamma, cfg.mu) as s:
            for key, val in opts:
                s.set_option(key, val)
            s.attach_convblock(*dims, batch)
            Xd, yd = s.upload(X), s.upload(labels)
            s.init_params(x0)
            if library:
                s.run_resident(K, Xd, yd)
            else:
                s.run(K, lambda k: s.set_batch(Xd[:, k % 2], yd[:, k % 2]))
            outs.append((s.all_params(), s.params(-1), s.momentum(), s.losses()))
    for other in outs[1:]:
        for a, b in zip(outs[0], other):
            assert np.array_equal(a, b)
