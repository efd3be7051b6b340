"""Results through the pinned staging, around its chunk and thread boundaries, and sets
made from the blocks that earlier sets freed."""

import threading

import numpy as np
import pytest

from synthetic import configs as SC

pytestmark = pytest.mark.gpu

CHUNK = (1 << 20) // 8  # doubles per chunk


def _set(fs, w, n):
    from paper_1707_05163_amd import ParticleSet
    k = -(-n // w.n)
    d = None if w.depth0 is None else np.tile(w.depth0, k)[:n]
    return ParticleSet(fs, np.tile(w.lon0, k)[:n], np.tile(w.lat0, k)[:n], d)


@pytest.mark.parametrize("is3d", [False, True])
@pytest.mark.parametrize("n", [1, 17, CHUNK - 1, CHUNK, CHUNK + 1, 5 * CHUNK + 3])
def test_every_query_agrees(n, is3d):
    """Positions of the set, its stride-1 record and the allocation-free query are the same
    arrays, byte for byte; counts are those of the status bytes."""
    from paper_1707_05163_amd import FieldSet
    from paper_1707_05163_amd import _lib as L
    w = (SC.cfg2_global_3d(nx=72, ny=36, nz=5, nt=2, n_particles=1000, nsteps=24) if is3d else
         SC.cfg1_global_eddies(nx=72, ny=36, nt=3, n_particles=1000, nsteps=24, period_days=3.0))
    fs = FieldSet.from_workload(w)
    ps = _set(fs, w, n)
    ps.execute(24 * w.dt, w.dt, output_stride=1)
    g, r = ps.get(), ps.records()
    counts, st = ps.status()
    for k in g:
        assert np.array_equal(g[k], r[k][-1]), k
    assert np.array_equal(st, r["status"][-1])
    assert counts["active"] == (st == 0).sum() and counts["n"] == n
    assert counts["oob"] == ((st & 1) != 0).sum() and counts["land"] == ((st & 2) != 0).sum()
    assert counts["deleted"] == ((st & 4) != 0).sum()
    h = {k: np.empty_like(v) for k, v in g.items()}
    ptr = lambda k: h[k].ctypes.data if k in h else None  # noqa: E731
    assert L.lib.pset_get_noalloc(ps.handle, ptr("lon"), ptr("lat"), ptr("depth"), ptr("ci"),
                                  ptr("cj"), ptr("ck")) == L.LP_OK
    for k in g:
        assert np.array_equal(g[k], h[k]), k


def test_blocks_of_freed_sets_and_queries_from_threads():
    """The same run again and again on reused blocks, larger and smaller sets in between,
    queried from several threads at once: always the first answer."""
    from paper_1707_05163_amd import FieldSet
    w = SC.cfg1_global_eddies(nx=72, ny=36, nt=3, n_particles=1000, nsteps=24, period_days=3.0)
    fs = FieldSet.from_workload(w)
    want = None
    for n in (200_000, 1000, 150_000, 200_000, 400_000, 200_000):
        ps = _set(fs, w, n)
        ps.execute(24 * w.dt, w.dt, output_stride=7, sample=False)
        got, bad = [None] * 4, []

        def ask(t):
            try:
                got[t] = (ps.get(), ps.status()[1], ps.records())
            except Exception as e:  # noqa: BLE001
                bad.append(e)

        th = [threading.Thread(target=ask, args=(t,)) for t in range(4)]
        for t in th:
            t.start()
        for t in th:
            t.join()
        assert not bad
        for g, st, r in got:
            for k in g:
                assert np.array_equal(g[k], got[0][0][k]), k
            assert np.array_equal(st, got[0][1])
            assert np.array_equal(r["lon"], got[0][2]["lon"])
        if n == 200_000:
            want = want or got[0]
            assert all(np.array_equal(want[0][k], got[0][0][k]) for k in want[0])
            assert all(np.array_equal(want[2][k], got[0][2][k]) for k in want[2])
        ps.close()


def test_stage_times_bracket_as_fmod_does():
    """Times of a periodic run far from the snapshots, before and after them: the run from
    t0 + k periods is the run from t0 (whole periods, exact in binary)."""
    from paper_1707_05163_amd import FieldSet, ParticleSet
    w = SC.cfg1_global_eddies(nx=72, ny=36, nt=4, n_particles=500, nsteps=96, period_days=4.0)
    fs = FieldSet.from_workload(w)
    out = []
    for k in (0, 1, 1000, -1, -777):
        ps = ParticleSet(fs, w.lon0, w.lat0, t0=43200.0 + k * 4 * 86400.0)
        ps.execute(96 * 900.0, 900.0)
        out.append(ps.get())
    for g in out[1:]:
        assert np.array_equal(g["lon"], out[0]["lon"]) and np.array_equal(g["lat"], out[0]["lat"])
