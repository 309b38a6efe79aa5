"""The library-driven loop over a small least-squares problem runs the local steps of a round (and, for few parameters, the
anchor average) in one launch: bits of the step-by-step calls at the edges of that kernel's paths, whatever the workspace
holds, and when the launches are replayed from a captured graph."""
import numpy as np
import pytest

import ols_inputs as I
from ols_inputs import generate as G

pytestmark = pytest.mark.gpu


def make_session(*a, **kw):
    from paper_2002_09539_amd.session import Session
    return Session(*a, **kw)


def state_of(s):
    return s.all_params(), s.params(-1), s.losses()


@pytest.mark.parametrize("m,d,batch,tau,mu,pieces", [
    (4, 1024, 32, 2, 0.0, (4, 3)),     # whole wavefronts, one pass; the second piece ends in mid-round
    (3, 1000, 31, 3, 0.9, (7, 5)),     # ragged rows and columns, pieces that start in mid-round
    (2, 8, 4, 1, 0.9, (5,)),           # a synchronisation after every step
    (5, 1028, 12, 2, 0.9, (6,)),       # one column past a single pass
    (2, 4096, 8, 2, 0.0, (4,)),        # the widest, mini-batch just fits the LDS copy
    (2, 4096, 64, 2, 0.9, (4,)),       # ... and does not
    (3, 512, 64, 2, 0.9, (4,)),        # four rows per wavefront
    (16, 1024, 16, 2, 0.9, (4,)),      # 16384 parameters over the workers: the largest in-launch average
    (17, 1024, 8, 2, 0.9, (4,)),       # one worker more: the mean kernel
    (1, 64, 8, 2, 0.9, (4,)),
    (40, 64, 4, 2, 0.9, (4,)),         # many replicas of few parameters: the average split sixteen ways
    (2, 128, 8, 70, 0.9, (141,)),      # a round longer than a launch takes
    (32, 64, 33, 2, 0.9, (5, 3)),      # the most replicas that the last workgroup averages; a second pass over one sample
    (33, 64, 4, 2, 0.9, (4,)),         # one more: the mean kernel
    (3, 201, 12, 3, 0.9, (5, 4)),      # ragged rows of few columns: rounds by the wide kernel
    (2, 1001, 40, 1, 0.0, (3,)),
    (5, 1028, 32, 2, 0.9, (3, 4)),     # just half of the wide kernel's passes; pieces of one step take the step kernel
    (5, 1028, 31, 2, 0.9, (4, 3)),     # ... and just less: rounds of two with their average
    (20, 1028, 31, 2, 0.9, (4,)),      # ... too many replicas for it: a launch per step
    (20, 1028, 12, 3, 0.9, (6,)),      # rounds of three
    (4, 1540, 12, 4, 0.9, (4,)),       # wider than those: a launch per step
    (4, 2048, 32, 2, 0.9, (4,)),       # the most columns of an in-launch average
    (2, 2052, 32, 2, 0.9, (4,)),
    (3, 1600, 32, 1, 0.9, (3,)),       # a single step filled well enough for the wide kernel
])
def test_rounds_in_one_launch_leave_the_bits_of_single_steps(m, d, batch, tau, mu, pieces):
    cfg = I.get(1).scaled(m=m, d_flat=d, batch=batch, tau=tau, mu=mu, nb=5)
    A, y, _, _ = G.lsq_data(cfg)
    x0 = G.generic_normal(21, 0, (d,), sigma=0.05)
    gamma = 0.01 if d >= 512 else 0.002
    outs = []
    for library in (True, False):
        with make_session(m, d, tau, cfg.alpha, gamma, mu) as s:
            s.attach_lsq(batch)
            s.ws.fill_(0xA5)           # nothing in the workspace needs clearing
            Ad, yd = s.upload(A), s.upload(y)
            s.init_params(x0)
            if library:
                for n in pieces:
                    s.run_resident(n, Ad, yd)
            else:
                s.run(sum(pieces), lambda k: s.set_batch(Ad[:, k % cfg.nb], yd[:, k % cfg.nb]))
            outs.append(state_of(s) + ((s.momentum(),) if mu else ()))
    for a, b in zip(*outs):
        assert np.isfinite(a).all() and np.array_equal(a, b)


def test_replayed_rounds():
    import torch
    m, d, batch, tau = 4, 256, 16, 2
    cfg = I.get(1).scaled(m=m, d_flat=d, batch=batch, tau=tau, mu=0.9, nb=2 * tau)
    A, y, _, _ = G.lsq_data(cfg)
    x0 = G.generic_normal(22, 0, (d,), sigma=0.05)
    with make_session(m, d, tau, cfg.alpha, 0.005, 0.9) as s, make_session(m, d, tau, cfg.alpha, 0.005, 0.9) as ref:
        for q in (s, ref):
            q.attach_lsq(batch)
            q.init_params(x0)
        Ad, yd = s.upload(A), s.upload(y)
        for q in (s, ref):
            q.run_resident(2 * tau, Ad, yd)      # kernels loaded before the capture
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s.main):
            s.run_resident(2 * tau, Ad, yd)
        for _ in range(4):
            with torch.cuda.stream(s.main):
                graph.replay()
            torch.cuda.synchronize()
            ref.run_resident(2 * tau, Ad, yd)
            for a, b in zip(state_of(s), state_of(ref)):
                assert np.array_equal(a, b)
