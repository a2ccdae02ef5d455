"""The gather's two row paths at the edges of their ranges.

A node whose x-components' row stencils span at most 2 NP + 2 rows and lie in
the staged region takes the unrolled rows over a table of row weights; every
other node (and the whole HBM-tap kernel) the general rows.  Both form the same
numbers, so the tiled kernels equal the HBM-tap kernel bit for bit whichever
path a node takes, and either stays within the bars of the parity tests: FP64
1e-12 of the oracle, FP32 1e-5.
"""
import numpy as np
import pytest

import oracle
from paper_2405_11489_amd import workloads
from parity_util import field_errors, gpu_run, oracle_run, plane_errors

pytestmark = pytest.mark.gpu

FP64, FP32 = 0, 1


def _flow(T0, spread, n=37, ny=29, seed=5):
    """Temperature T0 (1 +- spread) along y: the row span of a node, 2 c_out sqrt(T)
    and a position-dependent row more, crosses the ends of the unrolled path."""
    w = workloads.fourier_modes(n=n, ny=ny, mach=0.6, amplitude=1e-2, seed=seed, tau=0.7,
                                prandtl=0.71, T0=T0)
    y = np.arange(ny, dtype=np.float64)[:, None]
    w.T = w.T * (1.0 + spread * np.sin(2 * np.pi * y / ny) * np.ones((1, n)))
    return w


# D2Q16: spans of NP and NP + 1 rows (cold), of 2 NP + 1 .. 2 NP + 4 (T about 2);
# D2Q25: the same about T = 1.4
CASES = [(16, 4, 0.03, 0.3), (16, 4, 1.95, 0.25), (16, 3, 1.1, 0.3), (25, 4, 0.02, 0.3),
         (25, 4, 1.35, 0.25)]


@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("lattice,npts,T0,spread", CASES)
def test_unrolled_and_general_rows_give_the_same_bits(lattice, npts, T0, spread, prec):
    from paper_2405_11489_amd import pond
    w = _flow(T0, spread)
    kw = dict(lattice=lattice, interp_points=npts)
    ref = gpu_run(w, prec, 3, tuning={"kernel": pond.KERNEL_GLOBAL}, **kw)
    for tile, cap in [(pond.TILE_16x8, 0), (pond.TILE_16x16, 0), (pond.TILE_32x8, 0),
                      (pond.TILE_8x8, 0), (pond.TILE_8x8, 90)]:
        out = gpu_run(w, prec, 3, tuning={"kernel": pond.KERNEL_TILED, "tile": tile,
                                          "lds_nodes": cap}, **kw)
        for x, y in zip(out[:3], ref[:3]):
            np.testing.assert_array_equal(x, y, err_msg=f"tile {tile} cap {cap}")
    P, s, ost = oracle_run(w, 3, **kw)
    assert ref[4].nonphysical == 0 and ost.nonphysical == 0
    if prec == FP64:
        assert max(plane_errors(*ref[:3], s)) <= 1e-12
    errs = field_errors(ref[5], oracle.moments(P, s))
    assert max(errs.values()) <= (1e-12 if prec == FP64 else 1e-5), errs


@pytest.mark.parametrize("prec,bar", [(FP64, 1e-12), (FP32, 1e-5)])
def test_far_state_keeps_its_mass(prec, bar):
    """A tube at rest in two uniform states, the right one an eighth of the
    density of the reference node's: the right half away from the interface is
    a uniform flow and keeps its density (10 steps reach no further than 40
    nodes), in FP32 to the rounding of the interpolated moments."""
    w = workloads.sod_tube(nx=240, ny=16, steps=10)
    _, _, _, _, _, m = gpu_run(w, prec, 10)
    right = m["rho"][:, 190:230]
    assert np.max(np.abs(right / 0.125 - 1.0)) <= bar
