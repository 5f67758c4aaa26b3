"""The reverse sweep's two forms: a reverse and a recomputed step per launch on
small lattices, a stream for each kind above 256 blocks of 256 cells. A segment's
states are recomputed bit for bit, so the gradients do not depend on the
checkpoint distance; with one segment nothing runs beside the reverse steps."""

import numpy as np
import pytest
import torch

import workloads as wl
from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("shape,bc", [((60, 50, 1), (0, 1, 0)), ((250, 255, 1), (0, 0, 0)),
                                      ((270, 250, 1), (1, 0, 0)), ((41, 40, 43), (0, 1, 1))],
                         ids=["pairs", "pairs-256", "streams-315", "streams-3d"])
def test_gradient_is_that_of_one_segment(shape, bc, prec):
    import paper_1211_3286_amd as rlb
    prob = wl.random_modes(*shape, seed=9, umax=0.1, amp=0.05, bc=bc)
    T, nc = 11, int(np.prod(shape))
    gen = torch.Generator().manual_seed(4)
    du = torch.randn(3, nc, generator=gen, dtype=torch.float64).cuda()
    de = torch.randn(nc, generator=gen, dtype=torch.float64).cuda()
    ref = None
    for every in (T, 4, 3, 1, 2):
        say("sweep", shape, "prec", prec, "checkpoint every", every)
        sim = rlb.from_problems(prob, precision=prec, ckpt_every=every, tape_steps=T)
        sim.step(T)
        for again in range(2):
            dtau, deps0, du0 = sim.grad(du, de)
            got = [np.asarray(dtau), deps0.cpu().numpy(), du0.cpu().numpy()]
            assert all(np.isfinite(x).all() for x in got)
            if ref is None:
                ref = got
            for x, y in zip(got, ref):
                assert np.array_equal(x, y), (every, again)
        sim.close()
