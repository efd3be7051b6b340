"""The field at a step's middle with FP32 coefficients: (1 - tau) earlier + tau later,
rounded as it is written, in each row of a flow along the rows, where the positions after
one RK4 step from x = 0 show the stages' velocities to FP64 rounding.  (A mean of the
step's rounded ends is up to an FP32 unit off, 6e-8; the bound is far below that.)"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f16s"])
def test_middle_is_taken_at_its_own_time(dtype, batch):
    from paper_1707_05163_amd import FieldSet, ParticleSet, execute_batch
    g = np.random.default_rng(11)
    ny, day, dt, t0 = 512, 86400.0, 300.0, 40000.0
    x = 1e4 * np.arange(-4.0, 60.0)
    y = 1e4 * np.arange(float(ny))
    fs = FieldSet(x, y, None, "flat", dtype, capacity=2)
    for t in range(2):
        U = np.repeat(g.uniform(0.5, 1.0, ny).astype(np.float32)[:, None], x.size, axis=1)
        fs.push_snapshot(t * day, U, np.zeros_like(U))
    a, b = (fs.get_snapshot(t * day)[0][:-1, 0] for t in range(2))
    ps = ParticleSet(fs, np.zeros(ny - 1), y[:-1], t0=t0)
    if batch:
        execute_batch([ps], dt, dt, opts=[ParticleSet.opts()])
    else:
        ps.execute(dt, dt)

    def velocity(t):
        tau = np.float32(t / day)
        wa = (np.float32(1.0) - tau) * a  # (one FP32 rounding)
        return (np.longdouble(tau) * b + wa).astype(np.float32).astype(np.float64)

    u = velocity(t0) + 4.0 * velocity(t0 + dt / 2) + velocity(t0 + dt)
    got = ps.get()
    assert np.array_equal(got["lat"], y[:-1])
    assert np.abs(got["lon"] / (u * dt / 6.0) - 1.0).max() < 1e-12
