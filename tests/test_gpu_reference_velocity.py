"""The reference velocity of a loaded state: its mass-weighted mean velocity.

The sums run over 256 partial sums in a fixed order; each of the three sums of N
doubles is within N eps of the sum of its magnitudes, so the quotient is compared
to the exact one within that.
"""
import math

import numpy as np
import pytest

from paper_2405_11489_amd import workloads
from parity_util import gpu_solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(1, 1), (3, 1), (255, 1), (17, 15), (257, 1), (263, 251)])
def test_reference_velocity_is_the_exact_mean(nx, ny):
    w = workloads.fourier_modes(n=nx, ny=ny, mach=1.1, amplitude=0.05, seed=9)
    with gpu_solver(w, 0) as s:
        u_ref = s.export_state()[3]
        f, g, frame, _ = s.export_state()
        s.import_state(f, g, frame, None)
        again = s.export_state()[3]
    rho = [math.fsum([r]) for r in w.rho.ravel()]
    mass = math.fsum(rho)
    for k, u in enumerate((w.ux, w.uy)):
        mom = [a * b for a, b in zip(rho, u.ravel().tolist())]
        bar = (nx * ny + 4) * np.finfo(float).eps * math.fsum(map(abs, mom)) / mass
        assert abs(u_ref[k] - math.fsum(mom) / mass) <= bar
        # from the populations: sums of 16 products more per node, weights to rounding
        assert abs(again[k] - u_ref[k]) <= (nx * ny + 64) * 1e-14 * 10
