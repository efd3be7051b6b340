"""The gathering adaptive lanes on both sides of the 0.3 degree cells from which the metric
is the library's: positions, step exponents and attempt counts of the FP64 oracle."""

import pytest

from synthetic import configs as SC

from test_gpu_rkf45 import _compare, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("kind,nx", [("2d", 1440), ("2d", 1200), ("2d", 1196), ("2d", 72),
                                     ("steady", 1440), ("3d", 1440), ("3d", 360)])
def test_both_metrics(kind, nx, dtype):
    if kind == "3d":
        w = SC.cfg2_global_3d(nx=nx, ny=nx // 2, nz=3, nt=2, n_particles=2000, nsteps=24)
    else:
        w = SC.cfg1_global_eddies(nx=nx, ny=nx // 2, nt=2, n_particles=2000, nsteps=24,
                                  period_days=2.0)
        if kind == "steady":
            w.fields = SC.Fields(times=w.fields.times[:1], U=w.fields.U[:1], V=w.fields.V[:1])
    day = 86400.0
    ps, recs, orecs, ofs, st = _run(w, 3600.0, day, day, tol=0.01, emin=-5, emax=3, dtype=dtype,
                                    cache=False)
    _compare(ps, recs, orecs, ofs, st, w, 360.0, f"{kind} {nx} {dtype}")
