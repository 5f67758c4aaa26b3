"""Two steps per launch (k_step_march) on lattices stored in blocks of 32 cells:
tiles cut by the lattice's end, planes that are no whole number of blocks, z
ranges of a few planes, odd step counts and diagnostics steps in between. A
marching run gives the populations of the one-step kernel bit for bit, and
those are the oracle's within the bound every step form is held to (FP64
1e-12, FP32 1e-5 of the largest population)."""

import numpy as np
import pytest

import oracle
import workloads as wl
from gpu_helpers import gpu_state, relmax, say

pytestmark = pytest.mark.gpu

FP64, FP32 = 0, 1
TOL = {FP64: 1e-12, FP32: 1e-5}
MARCH, ONE = 10, 2

# at least 128 MiB of double-buffered state, so that the lattice is blocked;
# tiles own 32 x 13 (FP32) or 16 x 12 (FP64) cells
SHAPES = [
    ((64, 52, 130), (0, 0, 0)),     # whole FP32 tiles
    ((33, 53, 245), (1, 1, 1)),     # one cell past a tile along x and y
    ((95, 64, 71), (0, 1, 0)),      # one cell short
    ((1, 1031, 410), (0, 0, 1)),    # a single column of cells
    ((1025, 1, 415), (1, 0, 0)),    # a single row
    ((700, 601, 1), (0, 1, 1)),     # a single plane
    ((417, 511, 2), (1, 0, 0)),     # two planes
]


def _problem(shape, bc, eta=0.0):
    prob = wl.random_modes(*shape, seed=17, umax=0.2, amp=0.1, bc=bc)
    if eta:
        prob.n *= 1.7e-7 / 0.0314
        prob.eps *= 5.1e-7
        p = prob.params
        p.eta_s, p.tau_v, p.tau_e, p.tau_eps, p.a_e, p.a_eps = eta, 0.8, 0.8, 0.8, 1.0, 1.0
    return prob


def _plane(nx, ny, bc, eta=0.0):
    prob = _problem((nx, ny, 1), bc + (0,), eta)
    prob.params.lattice, prob.params.kappa = "d2q9", 4 / 3
    return prob


def _run(prob, prec, variant, calls, **kw):
    import paper_1211_3286_amd as rlb
    sim = rlb.from_problems(prob, precision=prec, **kw)
    sim.variant = variant
    assert ("march" in sim.kernel_name) == (variant >= (17 if sim.q == 9 else MARCH))
    for n in calls:
        sim.step(n)
    return sim


@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("shape,bc", SHAPES, ids=["x".join(map(str, s)) for s, _ in SHAPES])
def test_march_equals_the_one_step_kernel(shape, bc, prec):
    prob = _problem(shape, bc)
    say("march", shape, bc, "prec", prec)
    a = _run(prob, prec, MARCH, (5, 2))
    b = _run(prob, prec, ONE, (7,))
    for x, y in zip(a.populations(), b.populations()):
        assert bool((x == y).all())
    st = oracle.run(prob, 7)
    gs, _, bad = gpu_state(a, prob)
    assert bad == st.bad == 0
    assert relmax(gs[0]["f"], st.f) < TOL[prec] and relmax(gs[0]["g"], st.g) < TOL[prec]
    a.close()
    b.close()


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_march_with_per_cell_taus(prec):
    prob = _problem((70, 61, 101), (1, 0, 1), eta=0.1)
    a, b = _run(prob, prec, MARCH, (6,)), _run(prob, prec, ONE, (6,))
    for x, y in zip(a.populations(), b.populations()):
        assert bool((x == y).all())


def test_march_counts_inadmissible_cells_once():
    """The halo cells of a tile are computed by several tiles; each counts once."""
    prob = wl.blast(80)
    a, b = _run(prob, FP64, MARCH, (4,)), _run(prob, FP64, ONE, (4,))
    st = oracle.run(prob, 4)
    bad = [s.moments(allow_unphysical=True)["bad"] for s in (a, b)]
    say("inadmissible", bad, st.bad)
    assert bad == [st.bad, st.bad] and st.bad > 50


def test_march_keeps_the_diagnostics_steps():
    """Diagnostics steps run one by one between marching launches: the same
    partial sums at the same steps as the one-step kernel's."""
    prob = _problem((96, 80, 64), (0, 0, 0))
    a, b = (_run(prob, FP32, v, (), diag_every=5) for v in (MARCH, ONE))
    for n in (9, 1, 14):
        a.step(n)
        b.step(n)
        (sa, ta, _), (sb, tb, _) = a.diagnostics(), b.diagnostics()
        assert ta == tb == a.steps and np.array_equal(sa, sb)
    for x, y in zip(a.populations(), b.populations()):
        assert bool((x == y).all())


# D2Q9: strips own 58 (H = 4) or 60 columns of 64; ranges of a few rows
PLANES = [
    ((58, 300), (0, 0)), ((59, 290), (0, 1)), ((64, 257), (1, 1)), ((65, 260), (1, 0)),
    ((122, 140), (1, 1)), ((3, 6000), (0, 1)), ((2049, 8), (1, 0)), ((2100, 9), (0, 1)),
    ((187, 151), (1, 1)), ((63, 300), (1, 1)), ((2400, 7), (0, 0)),
]


@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("eta", [0.0, 0.1], ids=["fixed", "eta_s"])
@pytest.mark.parametrize("shape,bc", PLANES, ids=["x".join(map(str, s)) for s, _ in PLANES])
def test_d2q9_march_equals_the_one_step_kernel(shape, bc, eta, prec):
    """Every marching variant against the first one-step kernel, bit for bit, and
    that one against the oracle; lattices too small to march run step by step."""
    prob = _plane(*shape, bc, eta)
    say("d2q9 march", shape, bc, eta, "prec", prec)
    ref = _run(prob, prec, 0, (11,))
    st = oracle.run(prob, 11)
    gs, _, bad = gpu_state(ref, prob)
    assert bad == st.bad == 0
    assert relmax(gs[0]["f"], st.f) < TOL[prec] and relmax(gs[0]["g"], st.g) < TOL[prec]
    for v in (17, 18):
        sim = _run(prob, prec, v, (9, 2))
        for x, y in zip(sim.populations(), ref.populations()):
            assert bool((x == y).all()), sim.kernel_name
        sim.close()


def test_d2q9_march_counts_and_diagnostics():
    prob = wl.blast_disk(136)
    st = oracle.run(prob, 4)
    for v in (17, 18):
        sim = _run(prob, FP64, v, (4,))
        assert sim.moments(allow_unphysical=True)["bad"] == st.bad > 50
    prob = _plane(200, 150, (0, 0))
    a, b = (_run(prob, FP32, v, (), diag_every=7) for v in (17, 3))
    for n in (13, 1, 9):
        a.step(n)
        b.step(n)
        (sa, ta, _), (sb, tb, _) = a.diagnostics(), b.diagnostics()
        assert ta == tb == a.steps and np.array_equal(sa, sb)
    for x, y in zip(a.populations(), b.populations()):
        assert bool((x == y).all())


@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("eta", [0.0, 0.1], ids=["fixed", "eta_s"])
@pytest.mark.parametrize("shape,bc", PLANES, ids=["x".join(map(str, s)) for s, _ in PLANES])
def test_d2q9_march_with_the_correction(shape, bc, eta, prec):
    """The corrected marching kernel (a stage holds a row until the next one's
    fields are known) against the one-step kernel that recovers both neighbours,
    bit for bit, and that one against the oracle."""
    prob = _plane(*shape, bc, eta)
    prob.params.correction = 1
    say("d2q9 march +c7", shape, bc, eta, "prec", prec)
    ref = _run(prob, prec, 0, (7,))
    st = oracle.run(prob, 7)
    gs, _, bad = gpu_state(ref, prob)
    assert bad == st.bad == 0
    assert relmax(gs[0]["f"], st.f) < TOL[prec] and relmax(gs[0]["g"], st.g) < TOL[prec]
    sim = _run(prob, prec, 17, (5, 2))
    for x, y in zip(sim.populations(), ref.populations()):
        assert bool((x == y).all())


def test_d2q9_corrected_march_counts_inadmissible_cells():
    prob = wl.blast_disk(136, correction=1)
    st = oracle.run(prob, 4)
    sim = _run(prob, FP64, 17, (4,))
    assert sim.moments(allow_unphysical=True)["bad"] == st.bad > 50


@pytest.mark.parametrize("eta", [0.0, 0.1], ids=["fixed", "eta_s"])
@pytest.mark.parametrize("variant", [17, 18])
def test_d2q9_march_mixes_its_launches(variant, eta):
    """Calls of 1 to 13 steps, as launches of 4 and 3 and single ones, leave the
    populations of single steps; so do runs with diagnostics every 6th step."""
    import paper_1211_3286_amd as rlb
    prob = _plane(300, 290, (1, 0), eta)
    for every in (0, 6):
        sim, ref = (rlb.from_problems([prob], precision=FP64, diag_every=every) for _ in range(2))
        sim.variant, ref.variant = variant, 0
        for n in (1, 2, 3, 4, 5, 6, 7, 9, 10, 13):
            sim.step(n)
            ref.step(n)
            for x, y in zip(sim.populations(), ref.populations()):
                assert bool((x == y).all()), (n, every)
        if every:
            a, b = sim.diagnostics(), ref.diagnostics()
            assert a[1] == b[1] and relmax(a[0], b[0]) < 1e-13
