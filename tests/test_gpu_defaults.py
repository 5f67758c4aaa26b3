"""Default variants of batches: which kernel a handle starts with, by the work that
its forms would do for the batch, and its populations, which are the one-block
member kernel's (variant 0) bit for bit."""

import pytest

import workloads as wl
from gpu_helpers import say

pytestmark = pytest.mark.gpu

FP64, FP32 = 0, 1


def _plane(nx, ny, corr=0, eta=0.0):
    p = wl.random_modes(nx, ny, 1, seed=5, umax=0.2, amp=0.1, bc=(0, 1, 0))
    p.params.lattice, p.params.correction = "d2q9", corr
    if eta:
        p.n *= 1.7e-7 / 0.0314
        p.eps *= 5.1e-7
        q = p.params
        q.eta_s, q.tau_v, q.tau_e, q.tau_eps, q.a_e, q.a_eps = eta, 0.8, 0.8, 0.8, 1.0, 1.0
    return p


def _default_is(prob, members, prec, want, steps=(9, 1)):
    import paper_1211_3286_amd as rlb
    a, b = (rlb.from_problems([prob] * members, precision=prec) for _ in range(2))
    say(members, "of", prob.params.shape, "prec", prec, a.kernel_name)
    assert a.kernel_name == want
    b.variant = 0
    for n in steps:
        a.step(n)
        b.step(n)
        for x, y in zip(a.populations(), b.populations()):
            assert bool((x == y).all())
    a.close()
    b.close()


@pytest.mark.parametrize("nx,ny,members,corr,eta,window", [
    (4, 800, 4, 0, 0.0, 256),     # every segment has a CU
    (15, 100, 2, 0, 0.0, 256),    # 200 segments, a row each
    (15, 100, 64, 0, 0.0, 512),   # 6400 of them compute 17 times the cells
    (12, 500, 64, 0, 0.0, 512),
    (4, 800, 64, 0, 0.0, 256),    # the smaller windows lose little
    (4, 100, 256, 0, 0.0, 512),   # whole members in the larger windows
    (7, 500, 64, 1, 0.0, 512),
    (4, 800, 64, 1, 0.0, 256),
    (15, 500, 64, 0, 0.1, 512),
    (7, 500, 64, 0, 0.1, 256),
])
def test_strip_windows_by_the_cells_they_compute(nx, ny, members, corr, eta, window):
    for prec, t in ((FP64, "double"), (FP32, "float")):
        form = f"{window}>/h8"
        if prec == FP32 and eta and window == 512:  # shorter rounds instead
            form = "256>/h4"
        _default_is(_plane(nx, ny, corr, eta), members, prec,
                    f"k_d2q9_strips<{t},{form}" + ("+c7" if corr else ""))


def _box(nx, ny, nz, eta=0.0):
    p = wl.random_modes(nx, ny, nz, seed=5, umax=0.2, amp=0.1, bc=(0, 1, 0))
    if eta:
        p.n *= 1.7e-7 / 0.0314
        p.eps *= 5.1e-7
        q = p.params
        q.eta_s, q.tau_v, q.tau_e, q.tau_eps, q.a_e, q.a_eps = eta, 0.8, 0.8, 0.8, 1.0, 1.0
    return p


MEMBERS, LAUNCHES = "members", "cells"


@pytest.mark.parametrize("make,members,want", [
    (lambda: _box(11, 11, 11), 64, {FP32: LAUNCHES, FP64: LAUNCHES}),
    (lambda: _box(11, 11, 11), 128, {FP32: LAUNCHES, FP64: MEMBERS}),
    (lambda: _box(11, 11, 11), 256, {FP32: MEMBERS, FP64: MEMBERS}),
    (lambda: _box(16, 16, 16), 256, {FP32: LAUNCHES, FP64: MEMBERS}),
    (lambda: _box(24, 24, 24), 96, {FP32: LAUNCHES, FP64: LAUNCHES}),
    (lambda: _box(11, 11, 11, 0.1), 256, {FP32: LAUNCHES, FP64: MEMBERS}),
    (lambda: _plane(40, 40), 16, {FP32: LAUNCHES, FP64: LAUNCHES}),
    (lambda: _plane(40, 40), 64, {FP32: MEMBERS, FP64: MEMBERS}),
    (lambda: _plane(33, 32), 1, {FP32: MEMBERS, FP64: LAUNCHES}),
    (lambda: _plane(64, 64), 256, {FP32: MEMBERS, FP64: MEMBERS}),
    (lambda: _plane(40, 40, 1), 128, {FP32: MEMBERS, FP64: MEMBERS}),
    (lambda: _plane(40, 40, 0, 0.1), 128, {FP32: LAUNCHES, FP64: MEMBERS}),
    (lambda: _plane(40, 40, 0, 0.1), 256, {FP32: MEMBERS, FP64: MEMBERS}),
    (lambda: _plane(33, 32, 0, 0.1), 512, {FP32: MEMBERS, FP64: MEMBERS}),
    (lambda: _box(11, 11, 11, 0.1), 800, {FP32: MEMBERS, FP64: MEMBERS}),
])
def test_batches_that_fill_the_chip_take_the_member_kernel(make, members, want):
    prob = make()
    for prec, t in ((FP64, "double"), (FP32, "float")):
        name = "k_d2q9_" if prob.params.lattice == "d2q9" else "k_step_"
        if want[prec] == MEMBERS:
            name += f"members<{t},512,1>"
        else:
            small = 4096 if prob.params.lattice == "d2q9" else 1000
            name += f"cells<{t},{64 if members * -(-prob.params.ncells // 64) <= small else 256}>"
        _default_is(prob, members, prec, name + ("+c7" if prob.params.correction else ""),
                    steps=(3, 1))


def test_a_large_member_among_small_ones_spreads_over_the_chip():
    """The member kernel would wait for one block; the small members fill no CU."""
    import paper_1211_3286_amd as rlb
    probs = [_box(20, 15, 8)] + [_box(3, 3, 3)] * 300
    sim = rlb.from_problems(probs, precision=FP64)
    assert sim.kernel_name == "k_step_cells<double,64>"
    sim.close()


def test_tiles_by_default_where_their_windows_are_full():
    """Thin lattices, and diagnostics at every step over many windows, keep the
    one-step kernel; so do FP32 lattices of more than 5 windows a CU."""
    import paper_1211_3286_amd as rlb
    for shape, prec, every, want in (
            ((9000, 4), FP32, 0, "lattice"), ((9000, 7), FP64, 0, "lattice"),
            ((20000, 1), FP32, 0, "lattice"), ((2500, 8), FP32, 0, "tiles"),
            ((550, 540), FP32, 0, "tiles"), ((550, 540), FP32, 1, "lattice"),
            ((550, 540), FP32, 2, "lattice"), ((550, 540), FP32, 3, "tiles"),
            ((300, 260), FP32, 1, "tiles"), ((450, 430), FP64, 1, "tiles"),
            ((700, 500), FP32, 0, "lattice"), ((20000, 1, 1), FP32, 0, "lattice<float,256,1,1>+c7"),
            ((10000, 2, 1), FP64, 0, "lattice<double,64,4,1>+c7")):
        prob = _plane(*shape)
        sim, ref = (rlb.from_problems([prob], precision=prec, diag_every=every) for _ in range(2))
        say(shape, prec, every, sim.kernel_name)
        assert want in sim.kernel_name, (shape, prec, every)
        ref.variant = 0
        sim.step(7)
        ref.step(7)
        for x, y in zip(sim.populations(), ref.populations()):
            assert bool((x == y).all())
        sim.close()
        ref.close()
