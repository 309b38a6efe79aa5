"""The blocks' merged launches: the classifier's gradients inside the last kernel gradient's launch, and the statistics of a
convolution's output merged in one level or in two."""
import numpy as np
import pytest

import ols_inputs as I
from ols_inputs import generate as G
from oracle import conv_oracle as CO
from tests.helpers import l2_ratio

from paper_2002_09539_amd import binding as B

pytestmark = pytest.mark.gpu


def gradient(cfg, dims, batch, batch_norm, dtype, X, labels, x0, options=()):
    from paper_2002_09539_amd.session import Session
    with Session(cfg.m, cfg.d, 2, 0.6, 0.05, 0.0) as s:
        for key, value in options:
            s.set_option(key, value)
        s.attach_convblock(*dims, batch, batch_norm=batch_norm, gemm_dtype=dtype)
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_batch(Xd[:, 0], yd[:, 0])
        s.local_step()
        return s.gradient(), s.losses()


@pytest.mark.parametrize("m,dims,batch,batch_norm,dtype", [
    (3, (64, 8, 9, 10), 5, True, "bf16"),     # both kernels' gradients in one launch
    (2, (192, 5, 5, 16), 33, False, "bf16"),  # more samples than the guest stages at a time, all classes of the narrow form
    (1, (64, 5, 6, 17), 3, True, "bf16"),     # the wide form
    (2, (48, 6, 5, 32), 65, False, "f32"),    # a half-empty workgroup of units
    (2, (16, 4, 4, 2), 3, False, "f32"),
    (2, (64, 9, 8, 7), 4, True, "f32"),
])
def test_classifier_gradients_ride_along(m, dims, batch, batch_norm, dtype):
    cfg = I.get((9 if dtype == "bf16" else 7) if batch_norm else (8 if dtype == "bf16" else 6)).scaled(m=m, dims=dims, batch=batch, nb=1, seed=77)
    X, labels = G.conv_data(cfg)
    x0 = G.conv_init(cfg)
    g, losses = gradient(cfg, dims, batch, batch_norm, dtype, X, labels, x0)
    own, own_losses = gradient(cfg, dims, batch, batch_norm, dtype, X, labels, x0, [(B.OLS_OPT_HEAD_DW_GUEST, 0)])
    assert np.array_equal(g, own) and np.array_equal(losses, own_losses)
    assert np.abs(g[:, -dims[3]:]).max() > 0.0


@pytest.mark.parametrize("dims,batch", [((64, 2, 2, 3), 2),       # four parts, one with image pixels
                                        ((128, 9, 11, 3), 90),    # 204: a second round of twelve per stripe, partly empty
                                        ((64, 32, 32, 3), 21),    # 380 and 400 parts: about the last in one level and the first in two
                                        ((64, 32, 32, 3), 22)])
def test_statistics_levels(dims, batch):
    cfg = I.get(9).scaled(m=1, dims=dims, batch=batch, nb=1, seed=78)
    X, labels = G.conv_data(cfg)
    X = X + np.float32(3.0)    # a mean well off zero
    x0 = G.conv_init(cfg)
    g, losses = gradient(cfg, dims, batch, True, "bf16", X, labels, x0)
    loss, want = CO.convblock_bn_loss_grad(x0, dims[0], dims[3], X[0, 0], labels[0, 0], bf16_operands=True)
    # the statistics enter the loss and the classifier's gradients through values that no later rounding to bf16 follows
    # but that of a1: the bounds of the blocks' other parity tests
    assert abs(losses[0] - loss) <= 1e-4 * abs(loss)
    head = slice(-(dims[0] * dims[3] + dims[3]), None)
    assert l2_ratio(g[0][head], want[head]) <= 1e-3
    assert l2_ratio(g[0], want) <= 1e-2


def counted(attach, d, m, X, labels, x0, options=()):
    """Launches per kind of one timed local step."""
    from paper_2002_09539_amd.session import Session
    with Session(m, d, 2, 0.6, 0.05, 0.0) as s:
        for key, value in options:
            s.set_option(key, value)
        attach(s)
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_option(B.OLS_OPT_KERNEL_TIMING, 1)
        s.set_batch(Xd[:, 0], yd[:, 0])
        s.local_step()
        s.sync()
        return {kind: n for kind, (n, _) in s.kernel_stats().items()}


@pytest.mark.parametrize("dims,batch,batch_norm,dtype,options,want", [
    ((64, 8, 9, 10), 5, True, "bf16", (), dict(pool=0, head_bwd=0, conv_dw=1)),                        # a tail, one launch for both kernels
    ((64, 8, 9, 10), 5, False, "bf16", [(B.OLS_OPT_HEAD_DW_GUEST, 0)], dict(pool=0, head_bwd=1, conv_dw=1)),
    ((192, 5, 5, 3), 2, True, "bf16", (), dict(pool=1, head_bwd=0, conv_dw=2)),                        # no tail, two launches
    ((48, 6, 5, 10), 9, False, "f32", (), dict(pool=1, head_bwd=0, conv_dw=2)),
    ((64, 9, 8, 7), 4, True, "f32", (), dict(pool=0, head_bwd=0, conv_dw=2)),
])
def test_blocks_count_what_they_launch(dims, batch, batch_norm, dtype, options, want):
    cfg = I.get((9 if dtype == "bf16" else 7) if batch_norm else (8 if dtype == "bf16" else 6)).scaled(m=2, dims=dims, batch=batch, nb=1, seed=79)
    X, labels = G.conv_data(cfg)
    got = counted(lambda s: s.attach_convblock(*dims, batch, batch_norm=batch_norm, gemm_dtype=dtype), cfg.d, 2, X, labels, G.conv_init(cfg), options)
    assert {k: got.get(k, 0) for k in want} == want
    assert got["conv_fwd"] == 2 and got["conv_dx"] == 1 and got["head_fwd"] == 1


@pytest.mark.parametrize("m,casts", [(3, 0), (200, 1)])    # a small first forward GEMM, and one that takes the converted batch
def test_mlps_count_the_conversion_that_they_launch(m, casts):
    dims, batch = (264, 280, 7), 104
    cfg = I.get(3).scaled(m=m, dims=dims, batch=batch, nb=1, seed=80)
    X, labels = G.mlp_data(cfg)
    got = counted(lambda s: s.attach_mlp(dims, batch, "bf16"), cfg.d, m, X, labels % 7, G.mlp_init(cfg))
    assert got.get("cast_bf16", 0) == casts and got["gemm_fwd"] == 1
