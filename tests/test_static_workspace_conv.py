"""fp32 convolutional blocks near the size of the library's static workspace: where the kernels that ols_run_steps takes
need more scratch than the array holds, ols_run_steps_static takes the ones that need the least."""
import numpy as np
import pytest

import ols_inputs as I
from ols_inputs import generate as G
from tests.helpers import l2_ratio
from tests.test_boundary_cpu import FAKE, code_of, dry, kinds

from paper_2002_09539_amd import binding as B


def params(C, classes, bn):
    return 2 * (9 * C * C + (2 if bn else 1) * C) + C * classes + classes


def attach(h, C, S, batch, bn):
    (B.ols_attach_convblock_bn if bn else B.ols_attach_convblock)(h, C, S, S, 10, batch)


# scratch that holds: four or six activation-sized tensors, pooled values, the gradients' partial sums
@pytest.mark.parametrize("m,C,S,batch,bn", [(1, 128, 32, 16, False), (2, 128, 16, 32, False), (1, 256, 8, 128, False),
                                           (1, 64, 16, 128, True), (1, 256, 16, 16, True), (1, 48, 32, 60, False)])
def test_blocks_that_fit_with_the_least_scratch_run(m, C, S, batch, bn):
    h = dry(m=m, d=params(C, 10, bn), mu=0.9, tau=2)
    attach(h, C, S, batch, bn)
    full = B.ols_workspace_bytes(h)
    B.ols_bind_workspace(h, FAKE, full)
    B.ols_init_params(h, FAKE)
    B.ols_set_option(h, B.OLS_OPT_TRACE, 1)
    B.ols_run_steps(h, 2, FAKE, FAKE, 1)
    whole = kinds(B.ols_trace(h))
    B.ols_run_steps_static(h, 2, FAKE, FAKE, 1)
    assert kinds(B.ols_trace(h))[len(whole):] == whole
    assert B.ols_workspace_bytes(h) <= min(full, B.ols_static_workspace_bytes())
    B.ols_destroy(h)


def test_a_block_that_does_not_fit_either_way_is_refused_and_keeps_its_plan():
    h = dry(m=4, d=params(128, 10, False), mu=0.9, tau=2)
    attach(h, 128, 32, 16, False)
    need = B.ols_workspace_bytes(h)
    B.ols_init_params(h, FAKE)
    assert need > B.ols_static_workspace_bytes()
    assert code_of(B.ols_run_steps_static, h, 1, FAKE, FAKE, 1) == B.OLS_ENOMEM
    assert B.ols_workspace_bytes(h) == need
    B.ols_destroy(h)


@pytest.mark.parametrize("bn", [False, True])
def test_a_full_workspace_brings_the_other_kernels_back(bn):
    h = dry(m=1, d=params(128, 10, bn), mu=0.9, tau=2)
    attach(h, 128, 32, 10 if bn else 16, bn)
    full = B.ols_workspace_bytes(h)
    assert full > B.ols_static_workspace_bytes()
    B.ols_init_params(h, FAKE)
    for _ in range(2):
        B.ols_run_steps_static(h, 2, FAKE, FAKE, 1)
        lean = B.ols_workspace_bytes(h)
        assert lean < full
        assert code_of(B.ols_bind_workspace, h, FAKE, lean - 1) == B.OLS_ENOMEM
        B.ols_bind_workspace(h, FAKE, full - 1)          # too little for the others: still accepted
        assert B.ols_workspace_bytes(h) == lean
        B.ols_bind_workspace(h, FAKE, full)
        assert B.ols_workspace_bytes(h) == full
        B.ols_run_steps(h, 2, FAKE, FAKE, 1)
    B.ols_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("dims,batch,bn", [((128, 32, 32, 10), 16, False), ((64, 16, 16, 10), 128, True)])
def test_same_trajectory_as_with_the_full_workspace(dims, batch, bn):
    from paper_2002_09539_amd.session import Session
    cfg = I.get(7 if bn else 6).scaled(m=1, dims=dims, batch=batch, nb=1, seed=77)
    X, labels = G.conv_data(cfg)
    x0, out = G.conv_init(cfg), []
    for static in (False, True):
        with Session(1, cfg.d, 2, 0.6, 0.05, 0.0) as s:
            s.attach_convblock(*dims, batch, batch_norm=bn)
            Xd, yd = s.upload(X), s.upload(labels)
            s.init_params(x0)
            full = B.ols_workspace_bytes(s.h)
            (s.run_resident_static if static else s.run_resident)(2, Xd, yd)
            s.sync()
            assert not static or B.ols_workspace_bytes(s.h) < full
            out.append(s.params(0) - np.asarray(x0, np.float32)[: s.d])
    # two steps of gradients that differ by the rounding of fp32 sums; a ReLU may flip where a sum is next to zero
    assert l2_ratio(out[1], out[0]) <= 1e-3
