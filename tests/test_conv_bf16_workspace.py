"""A workspace that once was enough for a bf16 convolutional block stays enough: the sizes are what ols_workspace_bytes asked for
while the convolutions read their kernels as they are and the delta was gated by the activations themselves."""
import pytest

from tests.test_boundary_cpu import FAKE, code_of, dry
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
