"""State that fits the memory-side cache is updated with plain accesses, larger state with non-temporal ones: the same worker
on either side of that line keeps the same bits, through a local step and one with the pull-back."""
import numpy as np
import pytest

from ols_inputs import generate as G
from tests.test_gpu_mlp import make_session, small_mlp_case

pytestmark = pytest.mark.gpu


def two_steps(m, dims, batch, dtype, X, labels, x0):
    with make_session(m, x0.size, 2, 0.6, 0.05, 0.9) as s:
        s.attach_mlp(dims, batch, dtype)
        Xd, yd = s.upload(np.repeat(X, m, axis=0)), s.upload(np.repeat(labels, m, axis=0))
        s.init_params(x0)
        s.run_resident(2, Xd, yd)
        return s.all_params()


@pytest.mark.parametrize("dtype,dims,batch,below,above", [
    ("f32", (1024, 1024, 10), 64, 16, 17),      # 204 and 216 MB of replica buffers and momenta; 64 x 64 tiles
    ("f32", (1024, 512, 10), 128, 32, 33),      # 202 and 209 MB; the persistent kernel
    ("bf16", (1024, 1024, 10), 128, 13, 14),    # 193 and 208 MB; fewer than 1024 tiles of 64 x 128
])
def test_either_side_of_the_line(dtype, dims, batch, below, above):
    cfg, X, labels, x0 = small_mlp_case(1, dims, batch, 2, seed=431)
    x0 = x0 + G.generic_normal(3, 1, x0.shape, sigma=0.02)
    a = two_steps(below, dims, batch, dtype, X, labels, x0)
    b = two_steps(above, dims, batch, dtype, X, labels, x0)
    assert not np.array_equal(a[0], x0)
    for i in (0, below - 1):
        assert np.array_equal(a[i], b[i])


@pytest.mark.parametrize("dtype,dims,batch,m", [
    ("f32", (1024, 1028, 10), 64, 17),          # 216 MB; rows of 32 lines and 16 bytes
    ("f32", (68, 100, 128, 192, 10), 128, 3),   # the third layer's rows are whole lines that start inside one
    ("bf16", (1024, 1048, 10), 64, 20),
    ("f32", (1024, 1040, 10), 160, 17),         # halves of a line, streamed
    ("f32", (72, 80, 1024, 1032, 10), 128, 20),    # a streamed layer whose first row starts in the middle of a line, and a plain one
])
def test_rows_that_are_no_whole_lines(dtype, dims, batch, m):
    """Their state is accessed plainly at any size unless rows are whole half lines or the operands bf16: worker by worker the same
    bits either way."""
    cfg, X, labels, x0 = small_mlp_case(1, dims, batch, 2, seed=433)
    x0 = x0 + G.generic_normal(3, 1, x0.shape, sigma=0.02)
    a = two_steps(m, dims, batch, dtype, X, labels, x0)
    assert not np.array_equal(a[0], x0)
    for i in range(1, m):
        assert np.array_equal(a[0], a[i])
    b = two_steps(m + 1, dims, batch, dtype, X, labels, x0)
    assert np.array_equal(a[m - 1], b[0])
