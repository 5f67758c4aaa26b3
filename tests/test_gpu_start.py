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


def test_a_stream_of_its_own_waits_for_the_current_one():
    """Fields that the current stream is still computing, and gradients' inputs
    likewise, reach a handle on another stream as if on the same one; so they do
    the allocation-free run."""
    import paper_1211_3286_amd as rlb
    prob = wl.random_modes(64, 48, 40, seed=6, umax=0.1, amp=0.05)
    nc = prob.params.ncells
    n0, e0, u0 = [torch.from_numpy(np.ascontiguousarray(a)).cuda()
                  for a in rlb.problem_fields([prob])]
    w = torch.rand(4096, 4096, device="cuda")
    torch.cuda.synchronize()

    def late(t):
        """t, but only after some milliseconds of the current stream's work."""
        out, v = torch.full_like(t, 0.25), w
        for _ in range(12):
            v = (v @ w) * 1e-4
        return out.copy_(t + 0.0 * v.flatten()[0].clamp(0, 1))

    class Raw:  # anything with a stream's address
        def __init__(self, s):
            self.keep, self.cuda_stream = s, s.cuda_stream

    got = []
    for stream in (None, torch.cuda.Stream(), Raw(torch.cuda.Stream())):
        say("handle on", "the current stream" if stream is None else type(stream).__name__)
        sim = rlb.Simulation([prob.params], late(n0), late(e0), late(u0), precision=0,
                             ckpt_every=2, tape_steps=4, stream=stream)
        sim.step(4)
        m = sim.moments()
        dtau, de0, du0 = sim.grad(late(m["u"]), late(m["eps"]))
        r = rlb.run_noalloc(prob.params, late(n0), late(e0), late(u0), 3, precision=1,
                            stream=stream)
        torch.cuda.synchronize()
        got.append([m["u"], m["eps"], torch.as_tensor(dtau), de0, du0, r["u"], r["eps"]])
        sim.close()
    assert nc == got[0][1].numel()
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert bool((a == b).all())
