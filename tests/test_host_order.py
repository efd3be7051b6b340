"""The order of the library's runtime calls, on a stand-in for the HIP runtime (no GPU):
what has to wait for what when record arrays grow and when results come back, what
memory a query writes, and what gives way when memory runs out."""

import pytest

import host_only


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return host_only.build(str(tmp_path_factory.mktemp("fake") / "fakehip.so"))


@pytest.mark.parametrize("behave", ["", "behave"])
def test_growing_records_waits_for_queued_ones(so, behave):
    host_only.run(so, __file__, "grow", behave)


def grow(fake, behave):
    """Two executes on a stream that does not wait for the default one, no query between
    them, the second with more records than fit: the copies of the old arrays come after
    a wait for the first call's records, and nothing is launched before they are done."""
    import numpy as np

    from paper_1707_05163_amd import FieldSet, ParticleSet
    stream = 0x770
    x = np.arange(11) * 1000.0
    fs = FieldSet(x, x, capacity=1)
    z = np.zeros((11, 11), np.float32)
    fs.push_snapshot(0.0, z, z, stream=0)
    p = np.full(100, 5000.0)
    ps = ParticleSet(fs, p, p)
    ps.execute(72000.0, 60.0, 72000.0, output_stride=1, stream=stream)
    fake.fake_clear()
    ps.execute(36000.0, 60.0, 3600.0, output_stride=1, maxage=1e9 if behave else 0.0,
               stream=stream)
    log = host_only.calls(fake)
    old = 2 * 100 * 8
    copies = [i for i, c in enumerate(log) if c.op in ("memcpy", "memset") and c.bytes == old]
    assert len(copies) == (4 if behave else 2), log
    waits = [i for i, c in enumerate(log) if c.op == "devicesync" or
             (c.op == "streamsync" and c.stream == stream)]
    assert any(i < copies[0] for i in waits), log
    # (on the default stream: a wait for it, or for the device, ends them)
    ends = [i for i, c in enumerate(log) if c.op == "devicesync" or
            (c.op == "streamsync" and c.stream == 0)]
    launch = next(i for i, c in enumerate(log) if c.op == "launch" and i > copies[0])
    assert any(copies[-1] < i < launch for i in ends), log


@pytest.mark.parametrize("stream", ["2", "0x770", "0"])
@pytest.mark.parametrize("where", ["here", "elsewhere"])
@pytest.mark.parametrize("n", ["1000", "700000"])
def test_results_wait_for_the_run(so, stream, where, n):
    host_only.run(so, __file__, "results", stream, where, n)


def results(fake, stream, where, n):
    """What a query launches comes after the run it reads, in the thread that ran it or in
    another and in the query's own helper threads: on the run's stream, or on one that
    waits for an event of it.  Stream 2 is the calling thread's own (hipStreamPerThread):
    the same number is another stream in every thread."""
    import threading

    import numpy as np

    from paper_1707_05163_amd import FieldSet, ParticleSet
    stream, n = int(stream, 0), int(n)
    x = np.arange(11) * 1000.0
    fs = FieldSet(x, x, capacity=1)
    z = np.zeros((11, 11), np.float32)
    fs.push_snapshot(0.0, z, z, stream=0)
    p = np.full(n, 5000.0)
    ps = ParticleSet(fs, p, p)
    for ask in (ps.get, ps.status, ps.behaviour, ps.records, ps.step_exponents):
        fake.fake_clear()
        ps.execute(600.0, 60.0, 600.0, output_stride=1, maxage=1e9, stream=stream)
        run = host_only.calls(fake)
        key = lambda c: (c.stream, c.tid if c.stream == 2 else 0)  # noqa: E731
        done = [key(c) for c in run if c.op == "launch"][-1]
        marks = {c.a for c in run[[c.op for c in run].index("launch"):]
                 if c.op == "eventrecord" and key(c) == done}
        if where == "here":
            ask()
        else:
            t = threading.Thread(target=ask)
            t.start()
            t.join()
        after = {done}  # streams whose work comes after the run
        seen = 0
        for c in host_only.calls(fake)[len(run):]:
            if c.op == "waitevent" and c.a in marks:
                after.add(key(c))
            elif c.op in ("launch", "memcpyasync"):
                assert key(c) in after, (ask.__name__, c, done)
                seen += 1
            elif c.op == "memcpy":
                assert False, c
        assert seen


@pytest.mark.parametrize("n", ["1000", "700000"])
def test_a_query_writes_no_array_of_the_set(so, n):
    host_only.run(so, __file__, "scratch", n)


def scratch(fake, n):
    """The cell indices that a query computes are in memory of its own: another thread may
    be queueing sorts and launches of the set meanwhile, which use every array it has."""
    import numpy as np

    from paper_1707_05163_amd import FieldSet, ParticleSet
    n = int(n)
    x = np.arange(11) * 1000.0
    fs = FieldSet(x, x, np.arange(3.0), capacity=1)
    z = np.zeros((3, 11, 11), np.float32)
    fs.push_snapshot(0.0, z, z, z, stream=0)
    fake.fake_clear()
    lon = np.arange(n) * 1e-3
    ps = ParticleSet(fs, lon, lon, lon)
    ps.execute(600.0, 60.0, stream=0)
    blocks = [(c.a, c.a + c.bytes) for c in host_only.calls(fake) if c.op == "malloc"]
    fake.fake_clear()
    got = ps.get()
    assert np.array_equal(got["lon"], lon) and np.array_equal(got["depth"], lon)
    out = [c for c in host_only.calls(fake) if c.op == "copyout"]
    mine = sum(c.bytes for c in out if any(a <= c.b < b for a, b in blocks))
    assert mine == 24 * n and sum(c.bytes for c in out) == 36 * n


@pytest.mark.parametrize("what", ["push", "push_device", "batch", "forward", "train_step",
                                  "gradients", "features", "surrogate", "set", "records"])
def test_kept_blocks_give_way(so, what):
    host_only.run(so, __file__, "full", what)


def full(fake, what):
    """With no memory left but the blocks kept from a closed set, every call that needs
    some gets it; without those it says that there is none."""
    import numpy as np

    import paper_1707_05163_amd as lp
    from paper_1707_05163_amd import _lib
    from paper_1707_05163_amd.core import surrogate_features
    x = np.arange(11) * 1000.0
    u = np.zeros((11, 11), np.float32)
    fs = lp.FieldSet(x, x, capacity=2)
    if what != "push":
        fs.push_snapshot(0.0, u, u, stream=0)
    p = np.full(2000, 5000.0)
    small = lp.ParticleSet(fs, p, p)
    net = lp.Surrogate()
    X, T = np.zeros((256, 64), np.float32), np.zeros((256, 2), np.float32)
    tracer = np.zeros((11, 11), np.float32)
    call = {"push": lambda: fs.push_snapshot(0.0, u, u, stream=0),
            "push_device": lambda: fs.push_tracer(0.0, tracer, stream=0),
            "batch": lambda: lp.execute_batch([small], 600.0, 60.0, stream=0),
            "forward": lambda: net.forward(X), "train_step": lambda: net.train_step(X, T, 1e-3),
            "gradients": lambda: net.gradients(X, T),
            "features": lambda: surrogate_features(fs, p, p, 0.0),
            "surrogate": lambda: lp.Surrogate(1), "set": lambda: lp.ParticleSet(fs, p, p),
            "records": lambda: small.execute(600.0, 60.0, output_stride=1, stream=0)}[what]
    big = np.full(300_000, 5000.0)
    before = fake.fake_in_use()
    lp.ParticleSet(fs, big, big).close()
    kept = fake.fake_in_use() - before
    assert kept > 300_000 * 40, "the closed set's blocks are not kept"
    fake.fake_limit(fake.fake_in_use())
    call()
    fake.fake_limit(fake.fake_in_use())
    with pytest.raises(_lib.LPError) as e:
        lp.ParticleSet(fs, big, big)
    assert e.value.code == _lib.LP_ENOMEM



@pytest.mark.parametrize("n", ["1000", "700000"])
def test_a_set_stays_on_its_device(so, n):
    host_only.run(so, __file__, "device", n)


def device(fake, n):
    """A set made and run with device 1 current, on a field set of device 0 (as peers read
    each other's memory): its memory is device 1's, and so is whatever a query or its end
    does, with any device current."""
    import numpy as np

    from paper_1707_05163_amd import FieldSet, ParticleSet
    x = np.arange(11) * 1000.0
    fs = FieldSet(x, x, capacity=1)
    z = np.zeros((11, 11), np.float32)
    fs.push_snapshot(0.0, z, z, stream=0)
    fake.fake_clear()
    fake.hipSetDevice(1)
    p = np.full(int(n), 5000.0)
    ps = ParticleSet(fs, p, p)
    ps.execute(600.0, 60.0, 600.0, output_stride=1, maxage=1e9, stream=0x770)
    for now in (1, 0):
        fake.hipSetDevice(now)
        for ask in (ps.get, ps.status, ps.behaviour, ps.records, ps.step_exponents):
            ask()
    ps.close()
    log = host_only.calls(fake)
    assert {c.dev for c in log if c.op in ("malloc", "launch", "waitevent", "devicesync")} == {1}


if __name__ == "__main__":
    import sys
    globals()[sys.argv[2]](host_only.load(sys.argv[1]), *sys.argv[3:])
