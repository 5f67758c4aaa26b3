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
    (lambda: _modes((3000, 7, 1), "d2q9"), {}, "k_d2q9_lattice<float,64,4,1>"),
    (lambda: _modes((10000, 7, 1), "d2q9"), {}, "k_d2q9_lattice<float,256,1,1>"),
    (lambda: _modes((60, 400, 1), "d2q9", 1, bc=(1, 1, 0)), {}, "k_d2q9_lattice<float,64,4,1>+c7"),
], ids=["planes", "tape", "few-rows", "few-long-rows", "few-columns"])
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


def test_tuning_cache_tells_handles_apart(tmp_path):
    """Handles that dispatch to other kernels have other keys, and a stored choice
    is taken only where its number and name still are a variant."""
    import paper_1211_3286_amd as rlb
    box = _modes((64, 48, 40))
    eta = _modes((64, 48, 40))
    eta.params.eta_s = 0.1
    eos = _modes((64, 48, 40))
    eos.params.eos_gamma = 1.5
    clamped = _modes((64, 48, 40), bc=(1, 0, 0))
    tubes = [wl.tube_batch(n_tubes=1, seed=s, lmin=L, lmax=L)[0] for s, L in ((1, 300), (2, 500))]
    others = [wl.tube_batch(n_tubes=1, seed=s, lmin=L, lmax=L)[0] for s, L in ((1, 350), (2, 450))]
    sims = [rlb.from_problems(p, precision=FP32, **kw) for p, kw in (
        (box, {}), (box, {"ckpt_every": 2, "tape_steps": 4}), (eta, {}), (eos, {}), (clamped, {}),
        (tubes, {}), (others, {}))]
    keys = [s.tune_key() for s in sims]
    say(*keys)
    assert len(set(keys)) == len(keys)
    again = rlb.from_problems(tubes, precision=FP32)
    assert again.tune_key() == keys[5]
    cache = tmp_path / "tune.json"
    first = sims[0].tune(trial_steps=2, cache=str(cache))
    assert sims[0].tune(trial_steps=2, cache=str(cache)) == first
    db = json.loads(cache.read_text())
    # a choice under this key that the handle does not have: timed anew
    for variant, name in ((500, first["name"]), (first["variant"], "k_gone<float>")):
        db[keys[0]] = dict(first, variant=variant, name=name)
        cache.write_text(json.dumps(db))
        res = sims[0].tune(trial_steps=2, cache=str(cache))
        assert res["name"] == sims[0].variants()[res["variant"]] == sims[0].kernel_name
    for s in sims + [again]:
        s.close()


@pytest.mark.parametrize("prec", [FP64, FP32], ids=["fp64", "fp32"])
def test_segmented_variants_in_any_order(prec):
    """A table of many segments after one of few: the flags beyond the few had
    stayed behind, and the launch gave up its waits with RLB_E_DEVICE. The tuner,
    which goes through the tables, can be called again."""
    import paper_1211_3286_amd as rlb
    probs = [_modes((13, 11, 21)), _modes((9, 7, 16), bc=(1, 1, 1))]
    probs += wl.tube_batch(n_tubes=2, lmin=1500, lmax=2500, seed=5)
    sim, ref = (rlb.from_problems(probs, precision=prec) for _ in range(2))
    seg = [v for v, n in enumerate(sim.variants()) if "segments" in n]
    ref.variant = 0
    for v in (seg[-1], seg[0], seg[1], seg[0], seg[-1], seg[0]):
        say("segments", sim.variants()[v])
        sim.variant = v
        sim.step(3)
        ref.step(3)
        for x, y in zip(sim.populations(), ref.populations()):
            assert bool((x == y).all())
    for _ in range(3):
        sim.tune(trial_steps=2)
        sim.step(2)
        ref.step(2)
    for x, y in zip(sim.populations(), ref.populations()):
        assert bool((x == y).all())
    sim.close()
    ref.close()


@pytest.mark.parametrize("make,prec,variant,steps", [
    (lambda: _modes((2048, 2048, 1), "d2q9"), FP64, "k_d2q9_march<double>/h4", 80),
    (lambda: wl.shock_tube(800), FP64, "k_step_tubes<double,128>/h32", 640),
    (lambda: _modes((4, 800, 1), "d2q9"), FP64, "k_d2q9_strips<double,256>/h8", 320),
], ids=["march", "tubes", "strips"])
def test_the_tuner_prices_whole_launches(make, prec, variant, steps):
    """Five trial steps of a kernel that makes 4, 16 or 32 a launch cost what long
    runs cost a step: timed as one launch and single steps, or as a part of a
    round, they read 1.4 times that and more."""
    import time
    import torch
    import paper_1211_3286_amd as rlb
    sim = rlb.from_problems(make(), precision=prec)
    ratios = []
    for _ in range(5):
        priced = sim.tune(trial_steps=5)["ms_per_step"][variant] * 1e3
        sim.variant = sim.variants().index(variant)
        sim.step(steps)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        sim.step(steps)
        torch.cuda.synchronize()
        run = (time.perf_counter() - t0) / steps * 1e6
        say(variant, f"priced {priced:.2f} us, run {run:.2f} us a step")
        ratios.append(priced / run)
    assert sorted(ratios)[2] < 1.25
    sim.close()
