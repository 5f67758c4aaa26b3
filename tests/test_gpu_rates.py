"""Relaxation times from eta/s at densities far below and above equilibrium:
where lambda = n / n_eq underflows (tau_v is infinite, nothing relaxes), where
tau_v is 1/2 to the last bit, and where s turns negative. Tolerances as for
ordinary densities: FP64 1e-12, FP32 1e-5 of the largest population, 3 steps.
"""

import pytest

import oracle
import workloads as wl
from gpu_helpers import gpu_run, gpu_state, say

pytestmark = pytest.mark.gpu

FP64, FP32 = 0, 1
TOL = {FP64: 1e-12, FP32: 1e-5}


def relmax(a, b):
    return abs(a - b).max() / abs(b).max()


@pytest.mark.parametrize("prec,scale", [(FP64, 1e-120), (FP64, 1e-60), (FP64, 1e-20),
                                        (FP64, 0.0), (FP64, 1e30), (FP32, 1e-20), (FP32, 1e20)])
@pytest.mark.parametrize("shape,lattice", [((16, 12, 6), "d3q19"), ((40, 24, 1), "d2q9")],
                         ids=["d3q19", "d2q9"])
def test_extreme_densities(shape, lattice, prec, scale):
    p = wl.random_modes(*shape, seed=5, umax=0.2, amp=0.1, tau_v=0.8, tau_e=0.6, tau_eps=0.7,
                        tau_f=0.7, bc=(0, 1, 0))
    p.params.lattice = lattice
    p.params.eta_s, p.params.kappa = 0.1, 4 / 3
    p.params.a_e, p.params.a_f, p.params.a_eps = 0.4, 0.8, 1.0
    p.n = p.n * scale
    say("rates", shape, "prec", prec, "n x", scale)
    sim = gpu_run(p, 3, prec)
    (gs,), _, bad = gpu_state(sim, p)
    st = oracle.run(p, 3)
    assert bad == st.bad == 0
    assert relmax(gs["g"], st.g) < TOL[prec]
    if scale:
        assert relmax(gs["f"], st.f) < TOL[prec]
    else:
        assert not gs["f"].any()
