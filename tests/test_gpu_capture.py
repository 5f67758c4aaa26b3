"""rlb_step only enqueues: the first step of a fresh handle, in its default variant,
can be captured into a HIP graph. A replay repeats the captured launches on the
handle's two buffers: the calls here make an even number of them, so that it goes
on from the replay before (whole members take one launch from the one buffer to the
other, and repeat it). Eager work runs between the replays."""

import pytest
import torch

import workloads as wl
from gpu_helpers import say

pytestmark = pytest.mark.gpu

FP64, FP32 = 0, 1


def _modes(shape, lattice="d3q19", corr=0):
    p = wl.random_modes(*shape, seed=4, umax=0.2, amp=0.1, bc=(0, 1, 0))
    p.params.lattice, p.params.correction = lattice, corr
    return p


CASES = {
    "tubes": (lambda: wl.tube_batch(n_tubes=6, lmin=300, lmax=900, seed=5), "k_step_tubes", 64),
    "whole_tubes": (lambda: wl.tube_batch(n_tubes=3, lmin=90, lmax=120, seed=5), "k_step_tubes", 7),
    "strips": (lambda: [_modes((4, 400, 1), "d2q9"), _modes((6, 300, 1), "d2q9")], "k_d2q9_strips", 32),
    "strips_c7": (lambda: [_modes((5, 300, 1), "d2q9", 1)], "k_d2q9_strips", 24),
    "cells": (lambda: [_modes((16, 15, 14))], "k_step_cells", 12),
    "members": (lambda: [_modes((9, 8, 7))], "k_step_members", 12),
    "lattice": (lambda: [_modes((40, 30, 20))], "k_step_lattice", 12),
    "tiles": (lambda: [_modes((300, 200, 1), "d2q9")], "k_d2q9_tiles", 6),
    "march": (lambda: [_modes((128, 96, 64))], "k_step_march", 12),
    "d2q9_march": (lambda: [_modes((1500, 900, 1), "d2q9")], "k_d2q9_march", 8),
}


@pytest.mark.parametrize("prec", [FP64, FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("case", list(CASES))
def test_first_step_can_be_captured(case, prec):
    import paper_1211_3286_amd as rlb
    make, kernel, n = CASES[case]
    probs = make()
    ref = rlb.from_problems(probs, precision=prec)
    after = []
    for _ in range(3):
        ref.step(n)
        after.append([t.clone() for t in ref.populations()])
    stream = torch.cuda.Stream()
    sim = rlb.from_problems(probs, precision=prec, stream=stream)
    assert sim.kernel_name == ref.kernel_name and kernel in sim.kernel_name
    say("capture", case, sim.kernel_name)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        sim.step(n)
    for k in range(3):
        with torch.cuda.stream(stream):
            graph.replay()
        torch.cuda.synchronize()
        f, g = sim.populations()
        want = after[0 if case == "whole_tubes" else k]
        assert bool((f == want[0]).all() and (g == want[1]).all()), k
        ref.step(1)  # eager work in between
        ref.moments()
    sim.close()
    ref.close()
