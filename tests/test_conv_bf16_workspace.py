"""A workspace that once was enough for a bf16 convolutional block stays enough: the sizes are what ols_workspace_bytes asked for
while the convolutions read their kernels as they are and the delta was gated by the activations themselves."""
import numpy as np
import pytest

from tests.helpers import l2_ratio
from tests.test_boundary_cpu import FAKE, code_of, dry
from tests.test_gpu_conv_bf16 import conv_case, make_session
from tests.test_static_workspace_conv import params

from paper_2002_09539_amd import binding as B


@pytest.mark.parametrize("m,dims,batch,bn,size", [
    (16, (64, 32, 32, 10), 128, False, 1897449472),
    (16, (64, 32, 32, 10), 128, True, 3430201344),
    (3, (128, 13, 15, 7), 20, False, 43540992),
    (3, (128, 13, 15, 7), 20, True, 59839744),
    (15, (64, 23, 24, 10), 59, False, 491392000),     # kernel slices through LDS: neither images nor sign bytes
    (2, (64, 5, 5, 4), 300, False, 32233216),         # images of fewer than 64 padded pixels
    (2, (64, 5, 5, 4), 300, True, 40054528),
    (600, (64, 4, 4, 4), 256, False, 4594560000),
    (1, (64, 1, 1, 3), 1, False, 304640),
    (1, (64, 1, 1, 3), 1, True, 308736),
    (4, (192, 8, 8, 10), 16, False, 41727232),
])
def test_earlier_sizes_are_accepted(m, dims, batch, bn, size):
    h = dry(m=m, d=params(dims[0], dims[3], bn), mu=0.9, tau=2)
    (B.ols_attach_convblock_bn_bf16 if bn else B.ols_attach_convblock_bf16)(h, *dims, batch)
    need = B.ols_workspace_bytes(h)
    assert code_of(B.ols_bind_workspace, h, FAKE, need - 1) == B.OLS_ENOMEM
    B.ols_bind_workspace(h, FAKE, size)
    B.ols_init_params(h, FAKE)
    B.ols_run_steps(h, 2, FAKE, FAKE, 1)
    B.ols_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("m,dims,batch,bn", [
    (2, (64, 5, 5, 4), 190, False),     # images of fewer than 64 padded pixels: the sign bytes lie in the partial sums' place
    (520, (64, 5, 5, 4), 190, False),   # 9310 padded pixels: one range of the kernel gradient, whose place holds 9232
    (2, (64, 7, 7, 4), 190, True),      # the same with images of fewer than 64 pixels
    (520, (64, 7, 7, 4), 190, True),
])
def test_places_of_the_sign_bytes(m, dims, batch, bn):
    """The same worker alone and as one of many identical ones, whose sign bytes lie elsewhere."""
    cfg, X, labels, _ = conv_case(1, dims, batch, 1, seed=733)
    C, classes = dims[0], dims[3]
    rng = np.random.default_rng(6)
    kernels = lambda: (rng.standard_normal(9 * C * C) / np.sqrt(9 * C)).astype(np.float32)   # noqa: E731
    per_conv = lambda: [np.ones(C)] * bn + [0.02 * rng.standard_normal(C)]                   # noqa: E731
    x0 = np.concatenate([kernels(), *per_conv(), kernels(), *per_conv(), rng.standard_normal(C * classes) / np.sqrt(C),
                         np.zeros(classes)]).astype(np.float32)

    def step(workers):
        with make_session(workers, x0.size, 2, 0.6, 0.05, 0.0) as s:
            s.attach_convblock(*dims, batch, gemm_dtype="bf16", batch_norm=bn)
            s.init_params(x0)
            s.set_batch(s.upload(X[:, 0]).expand(workers, *X.shape[2:]), s.upload(labels[:, 0]).expand(workers, batch))
            s.local_step()
            s.sync()
            return s.g[[0, workers // 2, workers - 1], :x0.size].cpu().numpy(), s.losses()
    one, l1 = step(1)
    many, losses = step(m)
    for k, i in enumerate((0, m // 2, m - 1)):
        # another number of pixel ranges, and of chunks in the statistics: last bits, and the bf16 roundings that they move
        assert abs(losses[i] - l1[0]) <= 1e-4 * abs(l1[0])
        assert l2_ratio(many[k], one[0]) <= 1e-2
