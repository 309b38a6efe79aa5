"""The bf16 MLP's GEMMs on small launches: parity on either side of the line between the weight gradient's tiles, and of forward and
delta GEMMs by the kernel of small launches, which takes all of these (test_gpu_gemm_tiles.py has those above its limits)."""
import numpy as np
import pytest

from ols_inputs import generate as G
from oracle import ols_oracle as O
from tests.helpers import l2_ratio
from tests.test_gpu_mlp import make_session, small_mlp_case

from paper_2002_09539_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,dims,batch", [
    (3, (72, 136, 72, 10), 72),        # ragged in every dimension of a tile
    (1, (64, 64, 64, 10), 64),         # one tile of the weight gradient
    (255, (64, 128, 8, 4), 16),        # many workers: 2,040 steps of the forward GEMM
    (256, (64, 128, 8, 4), 16),        # 2,048
    (8, (1024, 1024, 16, 4), 24),      # 1024 tiles of the weight gradient: the most that take the small ones
    (8, (1032, 1024, 16, 4), 24),      # one tile row more
])
def test_bf16_gradient_and_loss(m, dims, batch):
    """Against the oracle with the same operand rounding: 2e-2 in L2 where a value may cross a bf16 rounding boundary."""
    cfg, X, labels, x0 = small_mlp_case(m, dims, batch, 1, seed=611)
    x0 = x0 + G.generic_normal(5, 2, x0.shape, sigma=0.02)
    with make_session(m, cfg.d, 2, 0.6, 0.05, 0.0) as s:
        s.set_option(B.OLS_OPT_FUSE_GEMM_UPDATE, 0)
        s.attach_mlp(dims, batch, "bf16")
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_batch(Xd[:, 0], yd[:, 0])
        s.local_step()
        g, losses = s.gradient(), s.losses()
    for i in sorted({0, m // 2, m - 1}):
        loss, grad = O.mlp_loss_grad(x0, dims, X[i, 0], labels[i, 0], bf16_operands=True)
        assert abs(losses[i] - loss) <= 1e-3 * abs(loss)
        assert l2_ratio(g[i], grad) <= 2e-2
