"""Calls of few steps, and runs with diagnostics, on handles whose kernels make
several steps a launch: the steps left over run one by one. Populations are the
first one-step kernel's bit for bit, lattice sums the same up to rounding."""

import time

import pytest
import torch

import workloads as wl
from gpu_helpers import relmax, say

pytestmark = pytest.mark.gpu

FP64, FP32 = 0, 1


def _plane(nx, ny, corr=0, bc=(0, 1, 0)):
    p = wl.random_modes(nx, ny, 1, seed=5, umax=0.2, amp=0.1, bc=bc)
    p.params.lattice, p.params.correction = "d2q9", corr
    return p


def _us(sim, calls, n=1, reps=9):
    best = 1e30
    for _ in range(reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(calls):
            sim.step(n)
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t0) / (calls * n) * 1e6)
    return best


@pytest.mark.parametrize("every", [0, 1, 4])
@pytest.mark.parametrize("shape,corr,prec", [
    ((300, 260), 0, FP32), ((300, 260), 0, FP64), ((560, 540), 0, FP32), ((145, 130), 1, FP64),
], ids=["fp32", "fp64", "two-singles", "c7"])
def test_tile_rounds_with_steps_left_over(shape, corr, prec, every):
    import paper_1211_3286_amd as rlb
    sim, ref = (rlb.from_problems([_plane(*shape, corr)], precision=prec, diag_every=every)
                for _ in range(2))
    sim.variant = next(i for i, n in enumerate(sim.variants()) if "tiles" in n and ",32,16>/h3" in n)
    ref.variant = 0
    say("tiles", shape, "prec", prec, "diagnostics every", every)
    for n in (1, 2, 3, 4, 5, 6, 1, 8):
        sim.step(n)
        ref.step(n)
        for x, y in zip(sim.populations(), ref.populations()):
            assert bool((x == y).all()), n
        if every:
            a, b = sim.diagnostics(), ref.diagnostics()
            assert a[1] == b[1] == sim.steps and relmax(a[0], b[0]) < 1e-13
    sim.close()
    ref.close()


def test_single_steps_of_a_tile_default_cost_a_one_step_kernel():
    """A loop of step(1), as a program that looks at each step runs it: the tile
    default made a round of each, 1.5 to 1.8 times the time at these sizes."""
    import paper_1211_3286_amd as rlb
    sim, one = (rlb.from_problems([_plane(500, 460)], precision=FP32) for _ in range(2))
    assert "tiles" in sim.kernel_name
    one.variant = 2
    a, b = _us(sim, 40), _us(one, 40)
    say("step(1) us", f"{a:.2f}", "one-step kernel", f"{b:.2f}")
    assert a < 1.3 * b  # between 1 and the 1.5 and more of a round
    sim.close()
    one.close()


@pytest.mark.parametrize("shape,lattice,prec,blocks", [
    ((96, 80, 64), "d3q19", FP32, 2), ((160, 72, 64), "d3q19", FP32, 1),
    ((45, 60, 140), "d3q19", FP64, 1), ((300, 290, 1), "d2q9", FP64, 3),
    ((700, 400, 1), "d2q9", FP64, 2), ((1000, 300, 1), "d2q9", FP32, 2),
    ((219, 800, 1), "d2q9", FP64, 2),
], ids=["d3q19-96", "d3q19-160", "d3q19-45", "d2q9-300", "d2q9-700", "d2q9-1000", "d2q9-219"])
def test_steps_between_marching_launches_by_row_length(shape, lattice, prec, blocks):
    """Single and diagnostics steps of a marching handle take the block shape that
    suits the rows: the sums are added in its order."""
    import numpy as np
    import paper_1211_3286_amd as rlb
    prob = wl.random_modes(*shape, seed=8, umax=0.2, amp=0.1, bc=(0, 1, 0))
    prob.params.lattice = lattice
    sim, ref = (rlb.from_problems(prob, precision=prec, diag_every=1) for _ in range(2))
    sim.variant = next(i for i, n in enumerate(sim.variants()) if "march" in n)
    ref.variant = blocks
    say(shape, sim.kernel_name, ref.kernel_name)
    for n in (1, 3):
        sim.step(n)
        ref.step(n)
        assert np.array_equal(sim.diagnostics()[0], ref.diagnostics()[0])
    for x, y in zip(sim.populations(), ref.populations()):
        assert bool((x == y).all())
    sim.close()
    ref.close()


@pytest.mark.parametrize("shape,blocks", [((1501, 200), "64,4,1"), ((2000, 1252), "64,4,1"),
                                          ((1998, 1253), "128,2,1")])
def test_blocks_of_corrected_lattices_by_rows_and_size(shape, blocks):
    """One-step default of a corrected lattice in FP32 with eta/s, and the steps
    between the marching launches of one without, which add the same sums."""
    import numpy as np
    import paper_1211_3286_amd as rlb
    prob = _plane(*shape, corr=1)
    sim, ref = (rlb.from_problems(prob, precision=FP64, diag_every=1) for _ in range(2))
    sim.variant = next(i for i, n in enumerate(sim.variants()) if "march" in n)
    ref.variant = next(i for i, n in enumerate(ref.variants()) if f",{blocks}>+c7" in n)
    say(shape, sim.kernel_name, ref.kernel_name)
    for n in (1, 2):
        sim.step(n)
        ref.step(n)
        assert np.array_equal(sim.diagnostics()[0], ref.diagnostics()[0])
    for x, y in zip(sim.populations(), ref.populations()):
        assert bool((x == y).all())
    sim.close()
    ref.close()
    prob.n *= 1.7e-7 / 0.0314
    prob.eps *= 5.1e-7
    prob.params.eta_s, prob.params.a_e, prob.params.a_eps = 0.1, 1.0, 1.0
    sim = rlb.from_problems(prob, precision=FP32)
    assert f",{blocks}>+c7" in sim.kernel_name
    sim.close()
