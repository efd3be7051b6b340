"""Launches of up to 32768 particles carry 32 particles per wave, larger ones 64: a
particle's result does not depend on it, bit for bit, on either side of the line."""

import numpy as np
import pytest

from synthetic import configs as SC

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("is3d", [False, True])
@pytest.mark.parametrize("cache", [True, False])
def test_either_side_of_the_wave_split(is3d, cache):
    from paper_1707_05163_amd import FieldSet, ParticleSet
    n = 32769
    w = (SC.cfg2_global_3d(nx=72, ny=36, nz=5, nt=2, n_particles=n, nsteps=24) if is3d else
         SC.cfg1_global_eddies(nx=72, ny=36, nt=3, n_particles=n, nsteps=24, period_days=3.0))
    fs = FieldSet.from_workload(w)
    d = w.depth0
    out = []
    for m in (n, n - 1, 4097, 33):
        ps = ParticleSet(fs, w.lon0[:m], w.lat0[:m], None if d is None else d[:m])
        ps.execute(24 * w.dt, w.dt, stencil_cache=cache)
        out.append((ps.get(), ps.status()[1], m))
    g, st, _ = out[0]
    for h, st2, m in out[1:]:
        for k in g:
            assert np.array_equal(g[k][:m], h[k]), k
        assert np.array_equal(st[:m], st2)
