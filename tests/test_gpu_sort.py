"""The sorts keep every active particle once and drop the others: results with a sort after
every segment equal, bit for bit, those without one, for lists of one block, two, and more
than the largest number of blocks has steps for, and for as many bins as fit in LDS and one
level more."""

import numpy as np
import pytest

from synthetic import configs as SC

pytestmark = pytest.mark.gpu


def both_ways(w, Kh=0.0):
    from paper_1707_05163_amd import FieldSet, ParticleSet
    fs = FieldSet.from_workload(w)
    out = []
    for every in (0, 1):  # (the same launches of 3 steps: 3D coefficients follow them)
        ps = ParticleSet(fs, w.lon0, w.lat0, w.depth0)
        ps.execute(9 * w.dt, w.dt, outputdt=3 * w.dt, Kh=Kh, sort_every=every)
        out.append((ps.get(), ps.status()[1]))
    (a, sa), (b, sb) = out
    assert np.array_equal(sa, sb)
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    return sa


@pytest.mark.parametrize("n", [1, 2048, 2049, 20_481, 1_048_577])
def test_list_lengths(n):
    w = SC.cfg3_ensemble(n_runs=1, side_min=97, side_max=97, np_min=n, np_max=n, nsteps=9)[0]
    s = both_ways(w, Kh=1e5)
    if n > 1:
        assert 0 < np.count_nonzero(s) < n  # some left the grid between the sorts


@pytest.mark.parametrize("nz", [1025, 1026])  # 15 tiles x 1024 levels, and x 1025
@pytest.mark.parametrize("n", [9000, 40_000])
def test_bins(nz, n):
    both_ways(SC.cfg2_global_3d(nx=72, ny=36, nz=nz, nt=2, n_particles=n, nsteps=9))
