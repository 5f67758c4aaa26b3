"""Small lattices and batches: one launch per step over all members (k_step_cells,
k_d2q9_cells), rounds that take whole members through all steps in one launch,
and the default variants. All give the one-block member kernel's populations
bit for bit; that kernel is checked against the oracle elsewhere, and here once
per batch (FP64 1e-12, FP32 1e-5, the bounds of every step form)."""

import numpy as np
import pytest

import oracle
import workloads as wl
from gpu_helpers import gpu_state, relmax, say

pytestmark = pytest.mark.gpu

FP64, FP32 = 0, 1
TOL = {FP64: 1e-12, FP32: 1e-5}


def _tube(L, bc, seed):
    t = wl.tube_batch(n_tubes=1, seed=seed, lmin=L, lmax=L)[0]
    t.params.bc = (0, 0, bc)
    return t


def _plane(nx, ny, bc, corr=0):
    p = wl.random_modes(nx, ny, 1, seed=5, umax=0.2, amp=0.1, bc=bc)
    p.params.lattice, p.params.correction = "d2q9", corr
    return p


BATCHES = {
    # every member fits a block whole: one launch for all steps
    "whole_tubes": lambda: [_tube(L, bc, L) for L, bc in ((1, 1), (127, 1), (128, 0), (64, 0))],
    "whole_strips": lambda: [_plane(4, 16, (0, 1, 0)), _plane(3, 21, (0, 0, 0))],
    # blocks of 64 and 256 cells: members one cell short of, at and past them
    "cells": lambda: [wl.random_modes(*s, seed=3, umax=0.2, amp=0.1, bc=bc) for s, bc in (
        ((7, 9, 1), (0, 0, 0)), ((8, 8, 1), (1, 0, 1)), ((5, 13, 1), (0, 1, 0)),
        ((15, 17, 1), (0, 0, 0)), ((16, 16, 1), (1, 1, 1)), ((257, 1, 1), (0, 0, 0)),
        ((11, 12, 13), (1, 0, 1)))],
    "d2q9_cells": lambda: [_plane(*s, bc) for s, bc in (
        ((7, 9), (0, 0, 0)), ((8, 8), (1, 0, 0)), ((257, 1), (0, 1, 0)), ((31, 45), (1, 1, 0)))],
    "d2q9_cells_c7": lambda: [_plane(33, 47, (1, 1, 0), 1), _plane(20, 13, (0, 0, 0), 1)],
}


@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("batch", list(BATCHES))
def test_every_variant_equals_the_member_kernel(batch, prec):
    import paper_1211_3286_amd as rlb
    probs = BATCHES[batch]()
    calls = (19, 1, 4)  # more than a round, a single step, an even count
    ref = None
    names = rlb.from_problems(probs, precision=prec).variants()
    assert sum("cells" in n for n in names) == 2
    for v, name in enumerate(names):
        sim = rlb.from_problems(probs, precision=prec, diag_every=3)
        sim.variant = v
        try:
            for n in calls:
                sim.step(n)
        except rlb.RLBError as e:
            assert e.code == -7 and any(k in name for k in ("tubes", "strips", "segments"))
            sim.close()
            continue
        say(batch, name, "prec", prec)
        f, g = [t.cpu().numpy() for t in sim.populations()]
        sums, step, bad = sim.diagnostics()
        assert step == sum(calls) and bad == 0
        if ref is None:
            ref = f, g, sums
            states, _, _ = gpu_state(sim, probs)
            for p, gs in zip(probs, states):
                st = oracle.run(p, sum(calls))
                assert relmax(gs["f"], st.f) < TOL[prec] and relmax(gs["g"], st.g) < TOL[prec]
        assert np.array_equal(f, ref[0]) and np.array_equal(g, ref[1]), name
        assert relmax(sums, ref[2]) < 1e-13, name
        sim.close()


def test_default_variants():
    """Members of up to 1024 cells stay on the one-block kernel, tubes and narrow
    D2Q9 members take rounds, the rest one launch per step."""
    import paper_1211_3286_amd as rlb
    for probs, want in (
            ([wl.random_modes(8, 8, 16, seed=1)], "k_step_members<double,512,1>"),
            ([wl.random_modes(5, 5, 41, seed=1)], "k_step_cells<double,64>"),
            ([_tube(300, 1, 1), _tube(50, 0, 2)], "k_step_tubes<double,128>/h32"),
            ([_plane(15, 100, (0, 1, 0))], "k_d2q9_strips<double,256>/h8"),
            ([_plane(16, 100, (0, 1, 0))], "k_d2q9_cells<double,64>"),
            ([_plane(7, 100, (0, 1, 0), 1)], "k_d2q9_strips<double,256>/h8+c7"),
            ([_plane(8, 200, (0, 1, 0), 1)], "k_d2q9_cells<double,64>+c7")):
        sim = rlb.from_problems(probs, precision=FP64)
        assert sim.kernel_name == want
        sim.step(2)
        sim.close()


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_lattice_defaults_equal_the_first_variant(prec):
    """Lattices too small to march take 64 x 4 or 128 x 2 blocks, D2Q9 ones rounds
    of three steps (with eta/s or the correction while each window finds a CU):
    names, and populations of variant 0 bit for bit after 7 and after 1 more."""
    import paper_1211_3286_amd as rlb
    t = "double" if prec == FP64 else "float"
    corr = _plane(145, 130, (1, 1, 0), 1)
    wide = _plane(300, 260, (0, 1, 0), 1)
    for prob, want in (
            (wl.random_modes(27, 25, 26, seed=3), f"k_step_lattice<{t},64,4,1>"),
            (wl.random_modes(65, 20, 14, seed=3), f"k_step_lattice<{t},128,2,1>"),
            (_plane(300, 260, (0, 1, 0)), f"k_d2q9_tiles<{t},32,16>/h3"),
            (corr, f"k_d2q9_tiles<{t},32,16>/h3+c7"), (wide, f"k_d2q9_lattice<{t},64,4,1>+c7")):
        sim, ref = (rlb.from_problems([prob], precision=prec) for _ in range(2))
        assert sim.kernel_name == want
        ref.variant = 0
        for n in (7, 1):
            sim.step(n)
            ref.step(n)
            for x, y in zip(sim.populations(), ref.populations()):
                assert bool((x == y).all()), (prob.name, n)
