"""Waves with few nodes left to converge gather them four lanes each.

The HBM-tap kernel keeps one lane per node throughout, so it is what the tiled
kernels must equal bit for bit: near a shock, where single nodes of a wave take
many iterations, and in ragged tiles.
"""
import numpy as np
import pytest

from paper_2405_11489_amd import workloads
from parity_util import gpu_run

pytestmark = pytest.mark.gpu

FP64, FP32 = 0, 1


@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("split,npts", [(0, 4), (0, 3), (1, 4), (2, 4)])
def test_shock_waves_give_the_same_bits(split, npts, prec):
    from paper_2405_11489_amd import pond
    w = workloads.sod_tube(nx=261, ny=201, steps=4)
    if split == 2:
        w.prandtl = 1.0
    kw = dict(split=split, interp_points=npts)
    ref = gpu_run(w, prec, 4, tuning={"kernel": pond.KERNEL_GLOBAL}, **kw)
    for tile in (pond.TILE_16x8, pond.TILE_32x8, pond.TILE_32x16, pond.TILE_8x8, pond.TILE_256x1):
        out = gpu_run(w, prec, 4, tuning={"kernel": pond.KERNEL_TILED, "tile": tile,
                                          "lds_nodes": 0}, **kw)
        for x, y in zip(out[:3], ref[:3]):
            np.testing.assert_array_equal(x, y, err_msg=f"tile {tile}")
        assert (out[4].pc_iterations, out[4].nonconverged) == (ref[4].pc_iterations,
                                                               ref[4].nonconverged)
    # some nodes took more than the two gathers of a smooth flow
    assert ref[4].pc_iterations > ref[4].node_updates
