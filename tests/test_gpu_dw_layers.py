"""The weight gradients of several layers share launches where nobody times them: the bits of one launch per layer (which the
library takes while OLS_OPT_KERNEL_TIMING is on)."""
import numpy as np
import pytest

from ols_inputs import generate as G
from tests.test_gpu_mlp import make_session, small_mlp_case

from paper_2002_09539_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,m,dims,batch,guest", [
    ("f32", 3, (100, 72, 44, 10), 36, 1),
    ("f32", 2, (132, 64, 68, 36, 40, 96, 72, 7), 20, 1),      # six hidden layers: four, then two
    ("f32", 3, (260, 128, 192, 64, 10), 128, 1),              # the persistent kernel between layers that share
    ("f32", 20, (516, 1024, 1024, 10), 16, 0),                # above the memory-side cache; one layer's rows are whole lines
    ("f32", 64, (520, 380, 36, 12, 7), 64, 1),                # the first layer by column strips
    ("bf16", 3, (104, 72, 48, 10), 24, 1),
    ("bf16", 2, (136, 64, 72, 40, 48, 96, 80, 7), 40, 0),
    ("bf16", 12, (1032, 1024, 136, 1024, 10), 72, 1),         # 64 x 64 and 64 x 128 tiles
])
@pytest.mark.parametrize("tau", [1, 2])
def test_shared_launches_leave_the_bits_of_separate_ones(dtype, m, dims, batch, guest, tau):
    cfg, X, labels, x0 = small_mlp_case(m, dims, batch, 2, seed=611)
    x0 = x0 + G.generic_normal(3, 1, x0.shape, sigma=0.02)
    states = []
    for timed in (0, 1):
        with make_session(m, cfg.d, tau, 0.6, 0.05, 0.9) as s:
            s.set_option(B.OLS_OPT_KERNEL_TIMING, timed)
            s.set_option(B.OLS_OPT_HEAD_DW_GUEST, guest)
            s.attach_mlp(dims, batch, dtype)
            Xd, yd = s.upload(X), s.upload(labels)
            s.init_params(x0)
            s.run_resident(5, Xd, yd)
            states.append((s.all_params(), s.params(-1), s.momentum(), s.losses()))
    assert not np.array_equal(states[0][0][0], x0)
    for a, b in zip(*states):
        assert np.array_equal(a, b)
