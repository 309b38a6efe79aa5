"""The first forward GEMM of small bf16 MLPs, which rounds the fp32 batch itself and leaves it for the weight gradient, at the
edges of its tiles of 32 samples x 32 units and steps of 32 inputs, against the CPU oracle with the same rounding points."""
import numpy as np
import pytest

import ols_inputs as I
from ols_inputs import generate as G
from oracle import ols_oracle as O
from tests.helpers import l2_ratio

from paper_2002_09539_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,dims,batch", [
    (1, (8, 8, 2), 8),            # a quarter of a step and of a tile
    (3, (40, 40, 5), 32),         # one index group past a step; a second, partly empty column tile; samples fill a tile
    (2, (264, 32, 72, 3), 40),    # one column tile; a second row tile of eight samples
    (2, (1032, 104, 10), 104),    # two trips of requests per wavefront
    (64, (24, 16, 3), 64),        # many workers
])
def test_rounded_batch(m, dims, batch):
    cfg = I.get(3).scaled(m=m, dims=dims, batch=batch, nb=2, seed=505)
    X, labels = G.mlp_data(cfg)
    labels = (labels % dims[-1]).astype(labels.dtype)
    x0 = G.mlp_init(cfg)
    from paper_2002_09539_amd.session import Session
    with Session(m, cfg.d, 4, 0.6, 0.05, 0.0) as s:
        s.set_option(B.OLS_OPT_FUSE_GEMM_UPDATE, 0)
        s.attach_mlp(dims, batch, "bf16")
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_batch(Xd[:, 1], yd[:, 1])      # batches of a worker lie apart in memory
        s.local_step()
        g, losses = s.gradient(), s.losses()
    for i in range(0, m, 21):
        loss, want = O.mlp_loss_grad(x0, dims, X[i, 1], labels[i, 1], bf16_operands=True)
        assert abs(losses[i] - loss) <= 1e-3 * abs(loss)
        first = slice(0, dims[0] * dims[1])
        # the bound of the other bf16 parity tests: a stored activation may cross a rounding boundary (0.4 % of it)
        assert l2_ratio(g[i][first], want[first]) <= 5e-3
        assert l2_ratio(g[i], want) <= 5e-3
    assert np.isfinite(g).all()
