"""Names of the variants, the tuner's choices and its cache."""

import json
import math

import pytest

import workloads as wl
from gpu_helpers import say

pytestmark = pytest.mark.gpu

FP64, FP32 = 0, 1


def _modes(shape, lattice="d3q19", corr=0, bc=(0, 0, 0)):
    p = wl.random_modes(*shape, seed=4, umax=0.2, amp=0.1, bc=bc)
    p.params.lattice, p.params.correction = lattice, corr
    return p


@pytest.mark.parametrize("make,kw,steps", [
    (lambda: _modes((40, 30, 20)), {}, "k_step_lattice<float,64,4,1>"),
    (lambda: _modes((200, 150, 30)), {"ckpt_every": 4, "tape_steps": 8},
     "k_step_lattice<float,64,4,1>"),
    (lambda: _modes((3000, 7, 1), "d2q9"), {}, "k_d2q9_lattice<float,256,1,1>"),
    (lambda: _modes((60, 400, 1), "d2q9", 1, bc=(1, 1, 0)), {}, "k_d2q9_lattice<float,64,4,1>+c7"),
], ids=["planes", "tape", "few-rows", "few-columns"])
def test_marching_variants_that_cannot_march(make, kw, steps):
    """They bear the name of the kernel that runs, and the tuner neither times nor
    picks them."""
    import paper_1211_3286_amd as rlb
    sim = rlb.from_problems(make(), precision=FP32, **kw)
    names = sim.variants()
    idle = [v for v, n in enumerate(names) if "march" in n]
    say(sim.kernel_name, [names[v] for v in idle])
    assert idle and all(names[v] == f"{steps} (no march)" for v in idle)
    sim.variant = idle[0]
    assert sim.kernel_name == f"{steps} (no march)"
    res = sim.tune(trial_steps=2)
    assert res["variant"] not in idle and "march" not in res["name"]
    assert res["ms_per_step"][names[idle[0]]] == math.inf
    sim.close()
