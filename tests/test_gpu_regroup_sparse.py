"""Near a shock some waves do have a few nodes left after their first gathers.

Waves regroup once at most 16 of their nodes are left to converge.  The nodes that
take more than k gathers are those whose state after a step differs between k gathers
at most and as many as it takes; for some k they must come in such small numbers in
8 x 8 blocks, a wave each, and the tiled kernels must equal the HBM-tap kernel there.
"""
import numpy as np
import pytest

from paper_2405_11489_amd import workloads

pytestmark = pytest.mark.gpu

FP64, FP32 = 0, 1


def _step_from(state, w, prec, **kw):
    from paper_2405_11489_amd import pond
    with pond.Solver(w.nx, w.ny, tau=w.tau, gamma=w.gamma, prandtl=w.prandtl, bc_x=w.bc_x,
                     bc_y=w.bc_y, precision=prec, **kw) as s:
        s.import_state(*state)
        s.step(1)
        return s.export_state()


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_waves_with_few_nodes_left_regroup_to_the_same_bits(prec):
    from paper_2405_11489_amd import pond
    w = workloads.sod_tube(nx=261, ny=201, steps=4)
    with pond.Solver.from_workload(w, precision=prec) as s:
        s.step(3)
        state = s.export_state()
    ref_kernel = {"kernel": pond.KERNEL_GLOBAL}
    ref = _step_from(state, w, prec, tuning=ref_kernel)
    few = 0  # blocks with 1 .. 16 nodes left after k gathers
    for k in range(1, 7):
        cut = _step_from(state, w, prec, tuning=ref_kernel, pc_max_iter=k)
        left = np.zeros((208, 264), dtype=int)
        left[:w.ny, :w.nx] = np.any(ref[2] != cut[2], axis=0).reshape(w.ny, w.nx)
        left = left.reshape(26, 8, 33, 8).sum(axis=(1, 3))
        few += int(np.count_nonzero((left >= 1) & (left <= 16)))
    assert few > 0
    for tile in (pond.TILE_8x8, pond.TILE_16x8, pond.TILE_32x8):
        out = _step_from(state, w, prec, tuning={"kernel": pond.KERNEL_TILED, "tile": tile,
                                                 "lds_nodes": 0})
        for x, y in zip(out[:3], ref[:3]):
            np.testing.assert_array_equal(x, y, err_msg=f"tile {tile}")
