"""Small D2Q16 grids run four lanes per node on the 64-node tiles.

Each lane gathers one x-component; the sums over the x-components are formed in
the order one lane per node forms them, so the tiled results equal the HBM-tap
kernel's bit for bit, at sizes that are no multiple of the tile, on both sides
of the largest such grid, and whatever part of the region LDS holds.
"""
import numpy as np
import pytest

from paper_2405_11489_amd import workloads
from parity_util import gpu_run

pytestmark = pytest.mark.gpu

FP64, FP32 = 0, 1
TOTAL, INTERNAL, NONTRANS = 0, 1, 2
LIMIT = {FP64: 36864, FP32: 49152}


def _flow(nx, ny):
    return workloads.fourier_modes(n=nx, ny=ny, mach=1.3, amplitude=2e-2, seed=3, tau=0.6,
                                   prandtl=1.0)


SIZES = [(1, 1), (3, 1), (129, 1), (5, 9), (61, 67)]


@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("split,npts", [(TOTAL, 4), (TOTAL, 3), (INTERNAL, 4), (NONTRANS, 3)])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_four_lanes_per_node_give_the_same_bits(nx, ny, split, npts, prec):
    from paper_2405_11489_amd import pond
    w = _flow(nx, ny)
    kw = dict(split=split, interp_points=npts)
    ref = gpu_run(w, prec, 3, tuning={"kernel": pond.KERNEL_GLOBAL}, **kw)
    for tile, cap in [(pond.TILE_8x8, 0), (pond.TILE_8x8, 100), (pond.TILE_64x1, 0)]:
        out = gpu_run(w, prec, 3, tuning={"kernel": pond.KERNEL_TILED, "tile": tile,
                                          "lds_nodes": cap}, **kw)
        for x, y in zip(out[:3], ref[:3]):
            np.testing.assert_array_equal(x, y, err_msg=f"tile {tile} cap {cap}")
        assert (out[4].pc_iterations, out[4].nonconverged) == (ref[4].pc_iterations,
                                                               ref[4].nonconverged)


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_largest_four_lane_grid_and_the_next(prec):
    from paper_2405_11489_amd import pond
    for n in (LIMIT[prec] // 192, LIMIT[prec] // 192 + 1):
        w = _flow(192, n)
        ref = gpu_run(w, prec, 2, tuning={"kernel": pond.KERNEL_GLOBAL})
        out = gpu_run(w, prec, 2, tuning={"kernel": pond.KERNEL_TILED, "tile": pond.TILE_8x8,
                                          "lds_nodes": 0})
        for x, y in zip(out[:3], ref[:3]):
            np.testing.assert_array_equal(x, y)
        assert out[4].pc_iterations == ref[4].pc_iterations
