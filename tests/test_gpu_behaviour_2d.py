"""Age and tracer sampling along 2D trajectories in the cached kernel (the cell the step's
first stage sits in serves the sample) against the FP64 oracle and the gather kernel, in
every metric mode: cells of 15 (library cosine), 5 and 0.5 degrees (series) and 0.3
degrees (short series), and a flat mesh; snapshots, and a single steady one."""

import numpy as np
import pytest

from oracle import oracle as O
from synthetic import configs as SC

from parity import REL, compare_record, slice_record

pytestmark = pytest.mark.gpu

DAY = 86400.0


def _workload(nx, nt):
    if nx == 0:
        w = SC.cfg3_ensemble(n_runs=2, side_min=64, side_max=64, np_min=321, np_max=322,
                             nsteps=288, nt=nt, Kh=0.0)[0]
    else:
        w = SC.cfg1_global_eddies(nx=nx, ny=nx // 2, nt=nt, n_particles=321, nsteps=288,
                                  period_days=float(nt))
    if nt == 1:
        w.fields.period = 0.0
    rng = np.random.default_rng(nx + nt)
    w.fields.tracer = rng.uniform(0.0, 30.0, (nt, w.grid.ny, w.grid.nx)).astype(np.float32)
    return w


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("nx,nt", [(0, 5), (24, 3), (72, 3), (720, 3), (1200, 3), (1200, 1)])
def test_sample_and_age_in_2d(nx, nt, dtype):
    """Positions to the FP64 bar, ages and AGED deletions exactly, samples to the same bar
    (the tracer's values are at most 30)."""
    from paper_1707_05163_amd import FieldSet, ParticleSet
    w = _workload(nx, nt)
    fs = FieldSet.from_workload(w, dtype=dtype)
    runtime, maxage = 288 * w.dt, 0.7 * 288 * w.dt
    got = []
    for cache in (True, False):
        ps = ParticleSet(fs, w.lon0, w.lat0)
        ps.execute(runtime / 2, w.dt, runtime / 4, output_stride=1, sample=True, maxage=maxage,
                   stencil_cache=cache)
        ps.execute(runtime / 2, w.dt, runtime / 4, output_stride=1, sample=True, maxage=maxage,
                   stencil_cache=cache)
        got.append((ps.records(), ps.status()[1]))
    ofs = O.OracleFieldSet.from_workload(w)
    st = O.make_state(w.lon0, w.lat0)
    orecs = O.run(ofs, st, w.dt, runtime, runtime / 4, sample=True, maxage=maxage)
    extent = 360.0 if nx else float(w.grid.lon[-1])
    for recs, status in got:
        assert recs["lon"].shape[0] == len(orecs) == 5
        for k, o in enumerate(orecs):
            compare_record(slice_record(recs, k), o, w.grid, extent, label=f"rec {k}", ofs=ofs)
            assert np.array_equal(recs["age"][k], o["age"])
            nan = np.isnan(o["temp"])
            assert np.array_equal(np.isnan(recs["temp"][k]), nan)
            assert (np.abs(recs["temp"][k] - o["temp"])[~nan] <= REL * 30.0).all()
        assert np.array_equal(status, st.status)
        assert ((status & O.ST_AGED) != 0).any()
