"""The eastward metric of single Euler steps from the meridian 0 in a uniform eastward
flow, where the step itself is the position: against dt U / (M cos(lat)) in extended
precision, from the equator to a tenth of a degree from the poles, in the kernels that
took the library's cosine and a division from the first (the gathers, and the 2D runs
with an age, which run from the cached cell).

The cosine's argument is rounded (and the constant pi / 180 with it) to 2^-52 of up to
pi/2 radians, once for the point or for its row; the cosine, the row's sine and the series
between them round to 2^-53 of at most 1 each.  That is below 8e-16 absolute, divided by
cos(lat) relative; weights, products and quotient add below 1e-15 relative."""

import numpy as np
import pytest


pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["gather", "age", "steady age"])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("deg", [0.25, 1.0, 4.0, 10.0])
def test_step_along_a_parallel(deg, dtype, kind):
    from paper_1707_05163_amd import FieldSet, ParticleSet
    nx, ny = round(360 / deg), round(180 / deg) + 1
    lon = -180.0 + deg / 3 + deg * np.arange(nx)
    lat = np.linspace(-90.0, 90.0, ny)
    nt = 1 if kind == "steady age" else 2
    one = np.ones((ny, nx), np.float32)
    fs = FieldSet(lon, lat, None, "spherical", dtype, capacity=nt)
    for t in range(nt):
        fs.push_snapshot(86400.0 * t, one, 0.0 * one)
    g = np.random.default_rng(3)
    n = 20000
    y = g.uniform(-89.9, 89.9, n)
    y[:2000] = np.sign(y[:2000]) * g.uniform(85.0, 89.9, 2000)
    ps = ParticleSet(fs, np.zeros(n), y)
    dt = 3600.0
    kw = dict(stencil_cache=False) if kind == "gather" else dict(maxage=1e9)
    ps.execute(dt, dt, kernel="euler", **kw)
    got = ps.get()
    ext = np.longdouble
    pi = ext("3.14159265358979323846264338327950288")
    cos = np.cos(y.astype(ext) * pi / 180)
    want = ext(dt) / (ext(111120.0) * cos)
    err = np.abs((got["lon"] - want) / want).astype(float)
    tol = 8e-16 / cos.astype(float) + 1e-15
    worst = int(np.argmax(err / tol))
    print(f"{deg} {dtype} {kind}: largest error {err.max():.2e}, {(err / tol).max():.2f} of the "
          f"bound (at {y[worst]:.3f})", flush=True)
    assert (err <= tol).all()
    assert np.array_equal(got["lat"], y)
