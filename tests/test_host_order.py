"""The order of the library's runtime calls, on a stand-in for the HIP runtime (no GPU):
what has to wait for what when record arrays grow."""

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


if __name__ == "__main__":
    import sys
    globals()[sys.argv[2]](host_only.load(sys.argv[1]), *sys.argv[3:])
