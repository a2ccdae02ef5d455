"""Autotuned classes keep grids with four lanes per node apart.

192 x 192 and 256 x 256 round to the same powers of two, but only the first runs its
64-node tiles with four lanes per node (up to 36864 nodes in FP64, 49152 in FP32).
What is tuned for that kernel -- its tile and a share of the LDS for one or two
blocks of four waves per CU -- would leave the larger grid one or two single-wave
blocks per CU.
"""
import pytest

from paper_2405_11489_amd import workloads

pytestmark = pytest.mark.gpu

FP64, FP32 = 0, 1


def _flow(n):
    return workloads.fourier_modes(n=n, mach=1.0, amplitude=1e-3, seed=0, tau=0.6)


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_a_four_lane_grid_does_not_tune_a_larger_one(prec):
    from paper_2405_11489_amd import pond
    pond.pond_tuning_cache_clear()
    try:
        with pond.Solver.from_workload(_flow(256), precision=prec) as s:
            want = pond.pond_get_tuning(s.ctx)
        with pond.Solver.from_workload(_flow(192), precision=prec) as s:
            small = pond.pond_autotune(s.ctx, 2)
        with pond.Solver.from_workload(_flow(256), precision=prec) as s:
            t = pond.pond_get_tuning(s.ctx)
        assert (t.tile, t.lds_nodes) == (want.tile, want.lds_nodes)
        # the class of the small grid itself is found again
        with pond.Solver.from_workload(_flow(190), precision=prec) as s:
            t = pond.pond_get_tuning(s.ctx)
        assert (t.tile, t.lds_nodes) == (small.tile, small.lds_nodes)
    finally:
        pond.pond_tuning_cache_clear()
