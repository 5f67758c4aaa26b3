"""Marching launches in forms that need a lattice of some size: D3Q19 in FP32, whose
populations are stored in blocks only from 128 MiB of double-buffered state on,
with tiles (32 x 13 cells) cut by the lattice's end, planes of no whole number of
blocks, single rows, columns and planes; both lattices with the general equation of
state; rounds cut to the load of the CUs. Populations equal the one-step (or
one-block) kernel's bit for bit, and those are the oracle's within the bound of
every step form (FP64 1e-12, FP32 1e-5 of the largest population)."""

import numpy as np
import pytest

import oracle
import workloads as wl
from gpu_helpers import gpu_state, relmax, say

pytestmark = pytest.mark.gpu

FP64, FP32 = 0, 1
TOL = {FP64: 1e-12, FP32: 1e-5}

# more than 441,506 cells each: stored in blocks in FP32
SHAPES = [
    ((64, 52, 140), (0, 0, 0)),     # whole tiles
    ((33, 53, 257), (1, 1, 1)),     # one cell past a tile along x and y
    ((95, 64, 75), (0, 1, 0)),      # one cell short
    ((1, 1031, 430), (0, 0, 1)),    # a single column of cells
    ((1025, 1, 435), (1, 0, 0)),    # a single row
    ((700, 641, 1), (0, 1, 1)),     # a single plane
    ((417, 531, 2), (1, 0, 0)),     # two planes
]


def _problem(shape, bc, eta=0.0):
    prob = wl.random_modes(*shape, seed=17, umax=0.2, amp=0.1, bc=bc)
    if eta:
        prob.n *= 1.7e-7 / 0.0314
        prob.eps *= 5.1e-7
        p = prob.params
        p.eta_s, p.tau_v, p.tau_e, p.tau_eps, p.a_e, p.a_eps = eta, 0.8, 0.8, 0.8, 1.0, 1.0
    return prob


def _gas(shape, bc, lattice):
    """P = (Gamma - 1)(eps - m n), where the model is linearly stable."""
    p = wl.random_modes(*shape, seed=23, umax=0.25, amp=0.1, tau_v=0.8, tau_e=0.6, tau_eps=0.7,
                        tau_f=0.7, bc=bc)
    p.params.lattice, p.params.eos_gamma, p.params.mass = lattice, 1.5, 0.6
    return p


def _march_and_one_step(prob, prec, calls, variant=None):
    """A handle that marches (asserted) and one of one-step kernels, both run."""
    import paper_1211_3286_amd as rlb
    a, b = (rlb.from_problems(prob, precision=prec) for _ in range(2))
    marches = [v for v, n in enumerate(a.variants()) if "march" in n]
    a.variant = marches[0] if variant is None else variant
    assert "march" in a.kernel_name and "no march" not in a.kernel_name
    b.variant = 0
    for n in calls:
        a.step(n)
    b.step(sum(calls))
    for x, y in zip(a.populations(), b.populations()):
        assert bool((x == y).all()), a.kernel_name
    b.close()
    return a


def _check(sim, prob, steps, prec):
    st = oracle.run(prob, steps)
    gs, _, bad = gpu_state(sim, prob)
    assert bad == st.bad == 0
    assert relmax(gs[0]["f"], st.f) < TOL[prec] and relmax(gs[0]["g"], st.g) < TOL[prec]


@pytest.mark.parametrize("shape,bc", SHAPES, ids=["x".join(map(str, s)) for s, _ in SHAPES])
def test_fp32_march_equals_the_one_step_kernel(shape, bc):
    cells = int(np.prod(shape))
    assert 2 * 38 * cells * 4 >= 128 << 20 and shape[0] * shape[1] >= 1024
    prob = _problem(shape, bc)
    say("FP32 march", shape, bc)
    sim = _march_and_one_step(prob, FP32, (5, 2))
    _check(sim, prob, 7, FP32)
    sim.close()


def test_fp32_march_with_per_cell_taus():
    prob = _problem((70, 61, 107), (1, 0, 1), eta=0.1)
    sim = _march_and_one_step(prob, FP32, (4, 3))
    _check(sim, prob, 7, FP32)
    sim.close()


@pytest.mark.parametrize("prec", [FP64, FP32], ids=["fp64", "fp32"])
def test_march_with_the_general_eos(prec):
    prob = _gas((70, 61, 107), (0, 1, 0), "d3q19")
    say("march, general equation of state, prec", prec)
    sim = _march_and_one_step(prob, prec, (4, 3))
    _check(sim, prob, 7, prec)
    sim.close()


@pytest.mark.parametrize("prec", [FP64, FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("shape,bc", [((187, 151, 1), (0, 1, 0)), ((122, 140, 1), (1, 0, 0))],
                         ids=["187x151", "122x140"])
def test_d2q9_march_with_the_general_eos(shape, bc, prec):
    import paper_1211_3286_amd as rlb
    prob = _gas(shape, bc, "d2q9")
    sim = rlb.from_problems(prob, precision=prec)
    marches = [v for v, n in enumerate(sim.variants()) if "march" in n]
    sim.close()
    assert len(marches) == 2
    for v in marches:
        say("d2q9 march", v, "general equation of state, prec", prec)
        sim = _march_and_one_step(prob, prec, (9, 2), variant=v)
        _check(sim, prob, 11, prec)
        sim.close()


@pytest.mark.parametrize("prec", [FP64, FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("corr", [0, 1], ids=["plain", "c7"])
def test_strip_rounds_cut_to_the_load(corr, prec):
    """12 members of 4 x 800: more segments than CUs, so that rounds of 8 steps
    lengthen to no more than keeps the fullest CU at as many of them (12 steps)."""
    import paper_1211_3286_amd as rlb
    probs = []
    for k in range(12):
        p = wl.random_modes(4, 800 - k, 1, seed=k, umax=0.2, amp=0.1, bc=(k % 2, k % 3 == 0, 0))
        p.params.lattice, p.params.correction = "d2q9", corr
        probs.append(p)
    ref = rlb.from_problems(probs, precision=prec)
    ref.variant = 0
    calls = (29, 1, 13)
    ref.step(sum(calls))
    want = ref.populations()
    for v, name in enumerate(ref.variants()):
        if "strips" not in name:
            continue
        say("strip rounds", name, "prec", prec)
        sim = rlb.from_problems(probs, precision=prec)
        sim.variant = v
        for n in calls:
            sim.step(n)
        for x, y in zip(sim.populations(), want):
            assert bool((x == y).all()), name
        sim.close()
    states, _, bad = gpu_state(ref, probs)
    assert bad == 0
    st = oracle.run(probs[3], sum(calls))
    assert relmax(states[3]["f"], st.f) < TOL[prec] and relmax(states[3]["g"], st.g) < TOL[prec]
    ref.close()


@pytest.mark.parametrize("prec", [FP64, FP32], ids=["fp64", "fp32"])
def test_tube_rounds_cut_to_the_load(prec):
    """The 64 ragged tubes: rounds of fewer steps than the variant's name tells."""
    import paper_1211_3286_amd as rlb
    tubes = wl.tube_batch()
    ref = rlb.from_problems(tubes, precision=prec)
    ref.variant = 0
    ref.step(45)
    want = ref.populations()
    for v, name in enumerate(ref.variants()):
        if "tubes" not in name:
            continue
        say("tube rounds", name, "prec", prec)
        sim = rlb.from_problems(tubes, precision=prec)
        sim.variant = v
        sim.step(33)
        sim.step(12)
        for x, y in zip(sim.populations(), want):
            assert bool((x == y).all()), name
        sim.close()
    ref.close()
