"""Members of a batch keep their order and their own flags.

The device tables of a batch hold its members sorted by stencil reach; what a caller
sees is in the order the contexts were given.  Walled batches replay captured
graphs, one per starting parity.
"""
import numpy as np
import pytest

from paper_2405_11489_amd import workloads
from parity_util import gpu_run

pytestmark = pytest.mark.gpu

FP64, FP32 = 0, 1


def _hot_channel():
    """Fluid that its walls heat beyond the ghost rows within three steps."""
    shape = (16, 4)
    return workloads.Workload("hot_channel", 4, 16, workloads.PERIODIC, workloads.WALL, 1.4, 1.0,
                              0.8, 20, np.ones(shape), np.zeros(shape), np.zeros(shape),
                              np.full(shape, 8.5), wall_ux=(0.0, 0.0), wall_T=(10.0, 10.0))


def _bad_tube():
    """Non-physical within 40 steps; stencils of longer reach than the channel's."""
    return workloads.sod_tube(nx=120, nu=1e-4, frame_mach=35.0)


def _solvers(ws, prec):
    from paper_2405_11489_amd import pond
    return [pond.Solver.from_workload(w, precision=prec) for w in ws]


def test_the_first_failed_member_gives_the_status():
    """The channel (first) leaves the ghost rows, the tube (second, of longer reach)
    goes non-physical: the status is the channel's, whatever order they step in."""
    from paper_2405_11489_amd import pond
    sols = _solvers([_hot_channel(), _bad_tube()], FP64)
    b = pond.pond_batch_create([s.ctx for s in sols])
    try:
        pond.pond_batch_step(b, 40)
        with pytest.raises(pond.PondError) as e:
            pond.pond_batch_synchronize(b)
        assert e.value.status == pond.ERR_UNSUPPORTED
    finally:
        pond.pond_batch_destroy(b)
        for s in sols:
            s.close()


def test_only_the_failed_member_is_flagged():
    """A failing member before a healthy one of longer reach: after the batch the
    failed context alone refuses to step."""
    from paper_2405_11489_amd import pond
    bad = workloads.sod_tube(nx=400, nu=1e-4)
    good = workloads.fourier_modes(n=48, ny=40, mach=2.0, amplitude=1e-2, seed=1, tau=0.6,
                                   prandtl=0.71)
    ref = gpu_run(good, FP64, 81)
    sols = _solvers([bad, good], FP64)
    b = pond.pond_batch_create([s.ctx for s in sols])
    try:
        pond.pond_batch_step(b, 80)
        with pytest.raises(pond.PondError) as e:
            pond.pond_batch_synchronize(b)
        assert e.value.status == pond.ERR_NONPHYSICAL
    finally:
        pond.pond_batch_destroy(b)
    try:
        with pytest.raises(pond.PondError) as e:
            sols[0].step(1)
        assert e.value.status == pond.ERR_STATE
        sols[1].step(1)
        for x, y in zip(sols[1].export_state()[:3], ref[:3]):
            np.testing.assert_array_equal(x, y)
    finally:
        for s in sols:
            s.close()


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_walled_batch_replays_either_parity(prec):
    """5 steps, then 8: the second call replays the graph of the odd parity."""
    from paper_2405_11489_amd import pond
    ws = [workloads.thermal_couette(ny=24, nx=6), workloads.sod_tube(nx=100, frame_mach=1.0)]
    for w in ws:
        w.prandtl = 0.71
    ref = [gpu_run(w, prec, 13) for w in ws]
    sols = _solvers(ws, prec)
    b = pond.pond_batch_create([s.ctx for s in sols])
    try:
        pond.pond_batch_step(b, 5)
        pond.pond_batch_step(b, 8)
        pond.pond_batch_synchronize(b)
        for s, r in zip(sols, ref):
            for x, y in zip(s.export_state()[:3], r[:3]):
                np.testing.assert_array_equal(x, y)
    finally:
        pond.pond_batch_destroy(b)
        for s in sols:
            s.close()


def test_batch_info_names_the_graph_in_use():
    """Walled batches replay graphs of several steps, the others launch each step."""
    from paper_2405_11489_amd import pond
    for ws, walled in (([workloads.thermal_couette(ny=24, nx=6)], True),
                       ([workloads.sod_tube(nx=100)], False)):
        sols = _solvers(ws, FP32)
        b = pond.pond_batch_create([s.ctx for s in sols])
        try:
            assert (pond.pond_batch_get_info(b).graph_steps > 0) == walled
        finally:
            pond.pond_batch_destroy(b)
            for s in sols:
                s.close()
