"""Periodic snapshots whose stage times leave a bracket and come back to it a period on
within one step: each stage still takes the field at its own time.  Two snapshots with a
wrap shorter than the step, and a bracket of three quarters of the period under a step
of more than half of it, forward and backward, against the FP64 oracle.
An infinite period, which holds the last snapshot for good."""

import numpy as np
import pytest

from oracle import oracle as O
from synthetic import configs as SC

from parity import compare_record, log, slice_record

pytestmark = pytest.mark.gpu

DAY = 86400.0
# snapshot times, period, step, steps, factor on the velocities
CASES = {
    "wrap of 600 s": ([0.0, DAY], 87000.0, 3600.0, 60, 1.0),
    "wrap of 60 s": ([0.0, DAY], 86460.0, 300.0, 350, 1.0),
    "long bracket": ([0.0, 3 * DAY, 3.5 * DAY], 4 * DAY, 2.4 * DAY, 20, 0.01),
}


def _workload(case, mesh):
    times, period, dt, nsteps, f = CASES[case]
    nt = len(times)
    if mesh == "spherical":
        w = SC.cfg1_global_eddies(nx=144, ny=72, nt=nt, n_particles=2000, nsteps=nsteps,
                                  period_days=4.0)
    else:
        w = SC.cfg3_ensemble(n_runs=1, side_min=64, side_max=64, np_min=2000, np_max=2000,
                             nsteps=nsteps, nt=5)[0]
    U, V = w.fields.U[:nt] * np.float32(f), w.fields.V[:nt] * np.float32(f)
    w.fields = SC.Fields(times=np.array(times), period=period, U=U, V=V)
    w.Kh = 0.0
    return w, dt, nsteps


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("mesh,dtype,batch", [("spherical", "f32", False), ("flat", "f32", False),
                                              ("spherical", "f64", False), ("flat", "f32", True)])
@pytest.mark.parametrize("case", list(CASES))
def test_stages_take_their_own_time(case, mesh, dtype, batch, sign):
    from paper_1707_05163_amd import FieldSet, ParticleSet, execute_batch
    w, dt, nsteps = _workload(case, mesh)
    dt *= sign
    log(f"{case}: {mesh} {dtype} batch={batch} dt {dt} x {nsteps}")
    fs = FieldSet.from_workload(w, dtype=dtype)
    ps = ParticleSet(fs, w.lon0, w.lat0)
    run = nsteps * abs(dt)
    if batch:
        execute_batch([ps], run, dt, opts=[ParticleSet.opts(output_stride=1)])
    else:
        ps.execute(run, dt, output_stride=1)
    recs = ps.records()
    ofs = O.OracleFieldSet.from_workload(w)
    st = O.make_state(w.lon0, w.lat0)
    orecs = O.run(ofs, st, dt, run, run)
    ext = 360.0 if mesh == "spherical" else float(w.grid.lon[-1])
    compare_record(slice_record(recs, -1), orecs[-1], w.grid, ext, label=case, ofs=ofs)
    c, status = ps.status()
    assert np.array_equal(status, st.status)
    assert (status == 0).sum() > 100


def test_infinite_period_is_no_period():
    """Between the snapshots the run is the one without a period; after the last it goes
    on in that snapshot."""
    from paper_1707_05163_amd import FieldSet, ParticleSet
    w, _, _ = _workload("wrap of 600 s", "spherical")
    out = []
    for period in (0.0, np.inf):
        fs = FieldSet.from_workload(w, time_period=period)
        ps = ParticleSet(fs, w.lon0, w.lat0)
        ps.execute(DAY, 3600.0)
        out.append(ps.get())
    assert np.isfinite(out[0]["lon"]).all()
    for k in out[0]:
        assert np.array_equal(out[0][k], out[1][k]), k
    ps.execute(DAY, 3600.0)
    w.fields = SC.Fields(times=np.zeros(1), U=w.fields.U[1:], V=w.fields.V[1:])
    last = ParticleSet(FieldSet.from_workload(w), out[1]["lon"], out[1]["lat"])
    last.execute(DAY, 3600.0)
    a, b = ps.get(), last.get()
    ok = ps.status()[1] == 0
    assert ok.sum() > 1000
    assert np.abs(a["lon"] - b["lon"])[ok].max() < 1e-9 * 360
    assert np.abs(a["lat"] - b["lat"])[ok].max() < 1e-9 * 360
