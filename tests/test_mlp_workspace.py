"""fp32 MLPs with a forward GEMM that is a little faster over K ranges, whose partial sums need scratch: a workspace without that
scratch is taken too, and so is the static one."""
import pytest

from ols_inputs import generate as G
from oracle import ols_oracle as O
from tests.helpers import max_norm_ratio
from tests.test_boundary_cpu import FAKE, code_of, dry

from tests.test_gpu_gemm_split import GRAD_TOL
from tests.test_gpu_mlp import make_session, small_mlp_case

from paper_2002_09539_amd import binding as B

M, BATCH, DIMS = 20, 52, (1984, 236, 4)
SCRATCH = 8 * M * BATCH * 236 * 4        # eight ranges; a multiple of 256


def attached(dims=DIMS):
    h = dry(m=M, d=sum(a * b + b for a, b in zip(dims, dims[1:])), mu=0.9, tau=2)
    B.ols_attach_mlp(h, dims, BATCH, 0)
    return h


def test_a_workspace_without_the_scratch_is_taken():
    h = attached()
    full = B.ols_workspace_bytes(h)
    little = full - SCRATCH
    assert little > 0
    for size in (full, little, full - 1, full):
        B.ols_bind_workspace(h, FAKE, size)
        assert B.ols_workspace_bytes(h) == (full if size >= full else little)
        before = B.ols_workspace_bytes(h)
        assert code_of(B.ols_bind_workspace, h, FAKE, little - 1) == B.OLS_ENOMEM
        assert B.ols_workspace_bytes(h) == before      # the bound workspace's plan
    B.ols_init_params(h, FAKE)
    B.ols_run_steps(h, 2, FAKE, FAKE, 1)
    B.ols_destroy(h)


def test_the_static_workspace_holds_what_fits_without_the_scratch():
    h = attached((1984, 236, 6900, 4))
    full = B.ols_workspace_bytes(h)
    assert full > B.ols_static_workspace_bytes() >= full - SCRATCH
    B.ols_bind_workspace(h, FAKE, full)
    B.ols_init_params(h, FAKE)
    B.ols_run_steps(h, 2, FAKE, FAKE, 1)
    B.ols_run_steps_static(h, 2, FAKE, FAKE, 1)
    assert B.ols_workspace_bytes(h) == full - SCRATCH
    B.ols_bind_workspace(h, FAKE, full)
    assert B.ols_workspace_bytes(h) == full
    B.ols_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("spare", [0, SCRATCH])
def test_either_route_matches_the_oracle(spare):
    cfg, X, labels, x0 = small_mlp_case(M, DIMS, BATCH, 1, seed=451)
    x0 = x0 + G.generic_normal(3, 1, x0.shape, sigma=0.02)
    with make_session(M, cfg.d, 2, 0.6, 0.05, 0.0) as s:
        s.set_option(B.OLS_OPT_FUSE_GEMM_UPDATE, 0)
        s.attach_mlp(DIMS, BATCH, "f32")
        full = B.ols_workspace_bytes(s.h)
        B.ols_bind_workspace(s.h, s.ws.data_ptr(), full - spare)
        assert B.ols_workspace_bytes(s.h) == full - spare
        Xd, yd = s.upload(X), s.upload(labels)
        s.init_params(x0)
        s.set_batch(Xd[:, 0], yd[:, 0])
        s.local_step()
        g, losses = s.gradient(), s.losses()
    for i in (0, M // 2, M - 1):
        loss, grad = O.mlp_loss_grad(x0, DIMS, X[i, 0], labels[i, 0])
        assert abs(losses[i] - loss) <= 1e-5 * abs(loss)
        assert max_norm_ratio(g[i], grad) <= GRAD_TOL
