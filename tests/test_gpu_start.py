"""The start of a handle: rlb_init reads the caller's fields only during the call,
with a tape (which keeps them) as without."""

import numpy as np
import pytest
import torch

import workloads as wl
from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
def test_taped_start_has_read_the_fields_when_it_returns(prec):
    """Fields overwritten from another stream as soon as rlb_init is back change
    nothing in the gradients (dL/deps0 and dL/du0 are taken at the taped fields)."""
    import paper_1211_3286_amd as rlb
    prob = wl.random_modes(128, 96, 80, seed=5, umax=0.1, amp=0.05)
    nc = prob.params.ncells
    gen = torch.Generator().manual_seed(7)
    du = torch.randn(3, nc, generator=gen, dtype=torch.float64).cuda()
    de = torch.randn(nc, generator=gen, dtype=torch.float64).cuda()
    fields = [torch.from_numpy(np.ascontiguousarray(a)) for a in rlb.problem_fields([prob])]
    mine, other = torch.cuda.Stream(), torch.cuda.Stream()
    got = []
    for overwrite in (False, True):
        n, e, u = [t.cuda() for t in fields]
        torch.cuda.synchronize()
        say("taped start, fields overwritten:", overwrite)
        sim = rlb.Simulation([prob.params], n, e, u, precision=prec, ckpt_every=2, tape_steps=4,
                             stream=mine)
        if overwrite:
            with torch.cuda.stream(other):
                for t in (u, e, n):
                    t.fill_(0.5)
        sim.step(4)
        got.append(sim.grad(du, de))
        torch.cuda.synchronize()
        sim.close()
    for a, b in zip(got[0], got[1]):
        assert np.array_equal(np.asarray(torch.as_tensor(a).cpu()),
                              np.asarray(torch.as_tensor(b).cpu()))
