"""Particles that stay at the ends of their cells: at a level or a row, just below one, at
the domain's last one and past it, in the cached kernels against the FP64 oracle, and in no
more time than in the middle of a cell."""

import numpy as np
import pytest

from oracle import oracle as O
from synthetic import configs as SC

from parity import compare_record, slice_record

pytestmark = pytest.mark.gpu


def _ends(axis):
    """Positions at and around the nodes of an axis, in the domain."""
    p = np.concatenate([axis, np.nextafter(axis, np.inf), np.nextafter(axis, -np.inf),
                        axis.astype(np.float32).astype(np.float64),
                        0.5 * (axis[1:] + axis[:-1])])
    return p[(p >= axis[0]) & (p <= axis[-1])]


@pytest.mark.parametrize("kernel", ["rk4", "euler"])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("kind", ["3d", "sphere", "flat"])
def test_rest_at_cell_ends(kind, dtype, kernel):
    from paper_1707_05163_amd import FieldSet, ParticleSet
    if kind == "3d":
        w = SC.cfg2_global_3d(nx=72, ny=36, nz=9, nt=2, n_particles=4000, nsteps=24)
        U, V, W = w.fields.materialise()
        w.fields = SC.Fields(times=w.fields.times, U=U, V=V, W=0.0 * W)
        w.depth0 = np.resize(_ends(w.grid.depth), w.n)
        ext = 360.0
    else:
        if kind == "sphere":
            w = SC.cfg1_global_eddies(nx=72, ny=36, nt=3, n_particles=4000, nsteps=24,
                                      period_days=3.0)
        else:  # a domain that ends at zero
            w = SC.cfg3_ensemble(n_runs=1, side_min=64, side_max=64, np_min=4000, np_max=4000,
                                 nsteps=24)[0]
            y = w.grid.lat - w.grid.lat[-1]
            w.grid = SC.Grid(lon=w.grid.lon, lat=y, spherical=False)
            w.Kh = 0.0
        w.fields = SC.Fields(times=w.fields.times, period=w.fields.period, U=w.fields.U,
                             V=0.0 * w.fields.V)
        w.lat0 = np.resize(_ends(w.grid.lat), w.n)
        ext = 360.0 if kind == "sphere" else float(w.grid.lon[-1])
    fs = FieldSet.from_workload(w, dtype=dtype)
    ps = ParticleSet(fs, w.lon0, w.lat0, w.depth0)
    run = 24 * w.dt
    ps.execute(run, w.dt, output_stride=1, kernel=kernel)
    recs = ps.records()
    ofs = O.OracleFieldSet.from_workload(w)
    st = O.make_state(w.lon0, w.lat0, w.depth0)
    orecs = O.run(ofs, st, w.dt, run, run,
                  **(dict(scheme=O.SCHEME_EULER) if kernel == "euler" else {}))
    compare_record(slice_record(recs, -1), orecs[-1], w.grid, ext, label=kind, ofs=ofs)
    _, status = ps.status()
    assert np.array_equal(status, st.status) and (status == 0).sum() > 1000


@pytest.mark.parametrize("at", ["below a level", "last level", "last row"])
def test_rest_at_cell_ends_takes_no_longer(at):
    """(Such points were once taken for points outside, reloaded at every stage: five times
    the time.)"""
    from paper_1707_05163_amd import FieldSet, ParticleSet
    n = 300_000
    if at == "last row":
        w = SC.cfg1_global_eddies(nx=360, ny=180, nt=3, n_particles=n, nsteps=96,
                                  period_days=3.0)
        w.grid.land = None
        a = w.grid.lat
        w.fields = SC.Fields(times=w.fields.times, period=w.fields.period, U=w.fields.U,
                             V=0.0 * w.fields.V)
        middle, rest = 0.5 * (a[-1] + a[-2]), a[-1]
    else:
        w = SC.cfg2_global_3d(nx=180, ny=90, nz=9, nt=2, n_particles=n, nsteps=96)
        U, V, W = w.fields.materialise()
        w.fields = SC.Fields(times=w.fields.times, U=U, V=V, W=0.0 * W)
        a = w.grid.depth
        middle, rest = ((0.5 * (a[-1] + a[-2]), a[-1]) if at == "last level" else
                        (0.5 * (a[4] + a[5]), np.nextafter(a[5], 0.0)))
    fs = FieldSet.from_workload(w)
    ms = []
    for p in (middle, rest):
        lat = np.full(n, p) if at == "last row" else w.lat0
        dep = None if at == "last row" else np.full(n, p)
        best = np.inf
        for _ in range(5):
            ps = ParticleSet(fs, w.lon0, lat, dep)
            ps.execute(96 * w.dt, w.dt, profile=True)
            best = min(best, ps.timing()[0])
            ps.close()
        ms.append(best)
    print(f"{at}: {ms[1]:.3f} ms, between {ms[0]:.3f}", flush=True)
    assert ms[1] < 2.0 * ms[0]
