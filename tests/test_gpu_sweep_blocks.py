"""The reverse sweep on two streams on both sides of the block count up to which a
recomputed step keeps to four waves a SIMD (3584 blocks of 64 x 4 cells). The states
are recomputed bit for bit, so the gradients are those of one segment."""

import numpy as np
import pytest
import torch

import workloads as wl
from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(896, 1024, 1), (893, 1027, 1)], ids=["3584", "3598"])
def test_gradient_is_that_of_one_segment_around_the_line(shape, prec):
    import paper_1211_3286_amd as rlb
    prob = wl.random_modes(*shape, seed=9, umax=0.1, amp=0.05, bc=(0, 1, 0))
    T, nc = 5, int(np.prod(shape))
    gen = torch.Generator().manual_seed(4)
    du = torch.randn(3, nc, generator=gen, dtype=torch.float64).cuda()
    de = torch.randn(nc, generator=gen, dtype=torch.float64).cuda()
    ref = None
    for every in (T, 2):
        say("sweep", shape, "prec", prec, "checkpoint every", every)
        sim = rlb.from_problems(prob, precision=prec, ckpt_every=every, tape_steps=T)
        sim.step(T)
        for again in range(2):
            dtau, deps0, du0 = sim.grad(du, de)
            got = [torch.as_tensor(np.asarray(dtau)), deps0.clone(), du0.clone()]
            assert all(bool(torch.isfinite(x).all()) for x in got)
            ref = ref or got
            for x, y in zip(got, ref):
                assert torch.equal(x, y), (every, again)
        sim.close()
