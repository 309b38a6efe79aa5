"""Refreshes of a few MiB with tau = 1 inside ols_run_steps, which stay on the main stream where another step follows: the same
models, anchor and replica buffer as with the overlapped schedule, also across calls and beside the other rules."""
import numpy as np
import pytest
import torch

import ols_inputs as I
from ols_inputs import generate as G

from paper_2002_09539_amd import binding as B

pytestmark = pytest.mark.gpu


def outcome(m, dims, tau, calls, options, setup):
    from paper_2002_09539_amd.session import Session
    cfg = I.get(2).scaled(m=m, dims=dims, batch=20, nb=3, tau=tau, seed=611)
    X, labels = G.mlp_data(cfg)
    labels = (labels % dims[-1]).astype(labels.dtype)
    with Session(m, cfg.d, tau, 0.6, 0.05, 0.9) as s:
        for key, value in options:
            s.set_option(key, value)
        s.attach_mlp(dims, 20, "f32")
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(G.mlp_init(cfg))
        setup(s)
        for steps in calls:
            s.run_resident(steps, Xd, yd)
        torch.cuda.synchronize()
        return s.x.clone(), s.x_alt.clone(), s.all_params(), s.params(-1), s.momentum()


@pytest.mark.parametrize("m,dims,tau,calls,setup", [
    (5, (788, 300, 124, 7), 1, (4, 3, 1, 4), lambda s: None),   # 6.6 MB; a call's last refresh runs beside the next call
    (5, (788, 300, 124, 7), 1, (6,), lambda s: s.set_anchor_momentum(0.7)),
    (5, (788, 300, 124, 7), 1, (6,), lambda s: s.set_stale_average()),
    (2, (400, 240, 10), 1, (7,), lambda s: None),               # 1.2 MB: just past the refreshes that always run in line
    (7, (1200, 436, 10), 1, (6,), lambda s: None),              # 16.9 MB: past the limit
    (5, (788, 300, 124, 7), 2, (8,), lambda s: None),           # two steps to hide behind
])
def test_same_as_overlapped(m, dims, tau, calls, setup):
    default = outcome(m, dims, tau, calls, (), setup)
    overlapped = outcome(m, dims, tau, calls, [(B.OLS_OPT_SERIALIZE, 0)], setup)
    for a, b in zip(default, overlapped):
        assert torch.equal(a, b) if torch.is_tensor(a) else np.array_equal(a, b)
