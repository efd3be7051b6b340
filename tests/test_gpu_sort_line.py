"""The sorts on both sides of the line between counting in LDS and by global atomics: 12
tiles of 512 levels are 6144 bins, the last in LDS, and of 513 one step past it."""

import pytest

from synthetic import configs as SC

from test_gpu_sort import both_ways

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz", [513, 514])
@pytest.mark.parametrize("n", [1, 1024, 1025, 30_000, 262_145])
def test_line(nz, n):
    both_ways(SC.cfg2_global_3d(nx=64, ny=36, nz=nz, nt=2, n_particles=n, nsteps=9))
