"""The streaming kernels use plain accesses up to 25 million elements of state and non-temporal ones beyond: the same columns
on either side of that line keep the same bits, under every synchronisation rule that has such a kernel."""
import pytest
import torch

from tests.test_gpu_update import make_session

from paper_2002_09539_amd import binding as B

pytestmark = pytest.mark.gpu

M, BELOW = 16, 1_562_496       # 24,999,936 elements; one more row stride of 64 is over the line


def rounds(d, rule, mu, nesterov, cols):
    """Two rounds of two steps on the columns' gradients, zeros behind them."""
    gen = torch.Generator(device="cuda").manual_seed(5)
    with make_session(M, d, 2, 0.6, 0.1, mu, own_gradient=False) as s:
        assert s.ld == d
        g = torch.zeros(2, M, d, device="cuda")
        g[:, :, :cols] = 0.1 * torch.randn(2, M, cols, generator=gen, device="cuda")
        x0 = torch.zeros(d, device="cuda")
        x0[:cols] = torch.randn(cols, generator=gen, device="cuda")
        s.bind(g[0])
        s.set_option(B.OLS_OPT_NESTEROV, 1 if nesterov else 0)
        s.init_params(x0)
        if rule == "one_pass":
            s.set_option(B.OLS_OPT_FUSE_MEAN, 1)
        elif rule == "stale":
            s.set_stale_average()
        s.run(4, lambda k: s.set_gradient(g[k % 2]))
        s.sync()
        out = [torch.from_numpy(s.all_params()[:, :cols]), torch.from_numpy(s.params(-1)[:cols])]
        return out + ([s.buf[:, :cols].cpu()] if mu else [])


@pytest.mark.parametrize("rule,mu,nesterov", [("paper", 0.9, True), ("paper", 0.9, False), ("paper", 0.0, True),
                                              ("one_pass", 0.9, True), ("one_pass", 0.0, True), ("stale", 0.9, True)])
def test_either_side_of_the_line(rule, mu, nesterov):
    cols = 4099
    below, above = (rounds(d, rule, mu, nesterov, cols) for d in (BELOW, BELOW + 64))
    assert float(below[0].abs().max()) > 0.0
    for a, b in zip(below, above):
        assert torch.equal(a, b)
