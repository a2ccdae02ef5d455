"""Uniform flows through the FP32 path over 2000 steps, on both lattices and every
energy split: the conserved fields must not drift.

The deviations that the step gathers vanish on a uniform field, so a step rounds
the same few numbers each time: the stored populations and the moments formed of
them.  Where those sums are free of bias (the sums of the stored weights are the
lattice's, formed as the kernel forms them), every field is off by a random walk
of one float rounding (2^-24 of its scale) per step at most, sqrt(2000) 2^-24 =
2.7e-6; the temperature, recovered from the total energy c_v T + u^2 / 2, by that
share of the energy.  A bias repeats in every step instead (2000 2^-24 = 1.2e-4).
"""
import math

import numpy as np
import pytest

from paper_2405_11489_amd import workloads
from parity_util import gpu_solver

pytestmark = pytest.mark.gpu

FP32 = 1
STEPS = 2000
WALK = math.sqrt(STEPS) * 2.0 ** -24
GAMMA = 1.4
VARIANTS = [(16, 0), (16, 1), (16, 2), (25, 0), (25, 2)]  # (lattice, split)


@pytest.mark.parametrize("lattice,split", VARIANTS)
@pytest.mark.parametrize("mach,T,rho", [(0.0, 1.0, 1.0), (2.0, 1.0, 1.0), (1.0, 0.04, 1.0),
                                        (0.0, 0.5, 1.3)])
def test_uniform_flow_does_not_drift(lattice, split, mach, T, rho):
    w = workloads.fourier_modes(n=8, ny=8, mach=mach, angle_deg=30.0, amplitude=0.0, seed=0,
                                tau=0.55, prandtl=1.0 if split == 2 else 0.71, T0=T, gamma=GAMMA,
                                steps=STEPS)
    w.rho = np.full_like(w.rho, rho)
    with gpu_solver(w, FP32, lattice=lattice, split=split) as s:
        s.step(STEPS)
        m = s.moments()
        assert s.stats().nonphysical == 0
    uscale = max(float(np.max(np.hypot(w.ux, w.uy))), math.sqrt(T))
    drho = float(np.max(np.abs(m["rho"] - rho))) / rho
    du = float(max(np.max(np.abs(m["ux"] - w.ux)), np.max(np.abs(m["uy"] - w.uy)))) / uscale
    dT = float(np.max(np.abs(m["T"] - w.T))) / T
    # energy over its thermal part: 1 + (u^2 / 2) / (c_v T)
    energy = 1.0 if split == 1 else 1.0 + 0.5 * GAMMA * (GAMMA - 1.0) * mach ** 2
    print(f"D2Q{lattice} split {split} Mach {mach} T {T} rho {rho}: rho {drho:.1e} u {du:.1e} "
          f"T {dT:.1e}")
    assert drho <= WALK and du <= WALK and dT <= WALK * energy
