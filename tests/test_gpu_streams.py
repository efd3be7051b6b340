"""Sets on streams that the default stream does not wait for."""

import numpy as np
import pytest

from synthetic import configs as SC

pytestmark = pytest.mark.gpu


def _workload():
    return SC.cfg1_global_eddies(nx=72, ny=36, nt=3, n_particles=1000, nsteps=24, period_days=3.0)


@pytest.mark.parametrize("maxage", [0.0, 1e9])
def test_records_grow_behind_queued_ones(maxage):
    """Record arrays that grow while the records of the call before are still queued hold
    what they hold when every call is waited for."""
    import torch
    from paper_1707_05163_amd import FieldSet, ParticleSet
    w = _workload()
    fs = FieldSet.from_workload(w)
    n = 300_000
    x, y = np.resize(w.lon0, n), np.resize(w.lat0, n)
    out = []
    for wait in (True, False):
        stream = torch.cuda.Stream()
        ps = ParticleSet(fs, x, y)
        for nrec, age in ((2, 0.0), (3, maxage), (7, maxage)):
            ps.execute(nrec * 7200.0, 300.0, 7200.0, output_stride=1, maxage=age, stream=stream)
            if wait:
                torch.cuda.synchronize()
        out.append(ps.records())
    assert out[0]["lon"].shape == (13, n)
    for k in out[0]:
        assert np.array_equal(out[0][k], out[1][k], equal_nan=True), k


@pytest.mark.parametrize("elsewhere", [False, True])
def test_results_of_a_run_on_the_threads_own_stream(elsewhere):
    """hipStreamPerThread (2): results large enough for several host threads, asked for in
    the thread that ran and in another, are those of a run on the default stream."""
    import threading
    from paper_1707_05163_amd import FieldSet, ParticleSet
    w = _workload()
    fs = FieldSet.from_workload(w)
    n = 900_000
    x, y = np.resize(w.lon0, n), np.resize(w.lat0, n)
    out = []
    for stream in (0, 2):
        ps = ParticleSet(fs, x, y)
        got = {}

        def ask():
            got.update(ps.get(), status=ps.status()[1], rec=ps.records()["lon"])

        for _ in range(3):
            ps.execute(24 * 300.0, 300.0, output_stride=3, stream=stream)
            if stream and elsewhere:
                t = threading.Thread(target=ask)
                t.start()
                t.join()
            else:
                ask()
        out.append(dict(got))
    for k in out[0]:
        assert np.array_equal(out[0][k], out[1][k]), k
