"""Scaled FP16 storage takes each level's scale from its largest value wherever that lies: the
first or last node of a plane of one block, of exactly one block's share, of one value more
and of many blocks, and every level of a 3D snapshot.  Stored values equal the reference
quantiser's bit for bit."""

import numpy as np
import pytest

from oracle import quantize as Q
from synthetic import configs as SC

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(18, 9), (128, 64), (8193 // 3, 3), (721, 363)])
@pytest.mark.parametrize("node", [0, -1])
def test_largest_value_anywhere(nx, ny, node):
    from paper_1707_05163_amd import FieldSet
    w = SC.cfg1_global_eddies(nx=nx, ny=ny, nt=2, n_particles=4, nsteps=2)
    for s in range(2):
        w.fields.U[s].reshape(-1)[node] = -37.25 * (s + 1)
        w.fields.V[s].reshape(-1)[node] = 0.013
        w.fields.V[s][np.abs(w.fields.V[s]) > 0.013] = 0.0
    fs = FieldSet.from_workload(w, dtype="f16s")
    for s in range(2):
        U, V, _ = fs.get_snapshot(w.fields.times[s])
        assert np.array_equal(U, Q.f16_scaled_round(w.fields.U[s]))
        assert np.array_equal(V, Q.f16_scaled_round(w.fields.V[s]))


@pytest.mark.parametrize("nx,ny,nz", [(36, 18, 3), (180, 90, 700)])
def test_every_level(nx, ny, nz):
    from paper_1707_05163_amd import FieldSet
    w = SC.cfg2_global_3d(nx=nx, ny=ny, nz=nz, nt=2, n_particles=4)
    fs = FieldSet.from_workload(w, dtype="f16s", capacity=2)
    for s in range(2):
        for got, ref in zip(fs.get_snapshot(w.fields.times[s]), w.fields.snapshot(s)):
            assert np.array_equal(got, Q.f16_scaled_round(ref))
