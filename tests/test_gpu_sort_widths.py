"""The sort at the edges of its variants (one workgroup, wide digits, 8-bit
digits): stable by tile-major key, at load and after pushes."""
import numpy as np
import pytest

from paper_2009_13645_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _keys(cell, d):
    nx, ny, nz = d["nx"], d["ny"], d["nz"]
    t = d["tile"]
    nt = [-(-(n - 1) // k) for n, k in zip((nx, ny, nz), t)]
    i, j, k = cell % nx, cell // nx % ny, cell // (nx * ny)
    tile = ((k // t[2]) * nt[1] + j // t[1]) * nt[0] + i // t[0]
    loc = ((k % t[2]) * t[1] + j % t[1]) * t[0] + i % t[0]
    key = tile.astype(np.int64) * (t[0] * t[1] * t[2]) + loc
    return np.where(cell < 0, np.int64(1) << 40, key)


@pytest.mark.parametrize("n,shape,tile,sigma", [
    (4096, (20, 20, 40), (3, 2, 5), 3.0), (4097, (20, 20, 40), (3, 2, 5), 3.0), (6000, (60, 48, 200), (5, 3, 7), 40.0),
    (30001, (120, 100, 300), (1, 1, 1), 60.0), (1 << 18, (128, 64, 512), (4, 2, 2), 90.0),
    ((1 << 18) + 1, (64, 64, 64), (8, 8, 8), 9.0), (5000, (8, 8, 8), (8, 8, 8), 0.5), (9000, (24, 24, 24), (4, 4, 4), 500.0)])
def test_sort_is_stable_by_key(n, shape, tile, sigma):
    from paper_2009_13645_amd.engine import Engine
    w = wl.config1()
    w.nx, w.ny, w.nz = shape
    w.n_particles, w.tile, w.field_precision, w.charge_C = n, tile, 32, 1e-15
    d = w.descriptor()
    rng = np.random.default_rng(n)
    g = 0.5 * (np.array(shape) - 1) + sigma * rng.standard_normal((n, 3)) * np.array(shape) / max(shape)
    xyz = np.array([d["x0"], d["y0"], d["z0"]]) + g * np.array([d["dx"], d["dy"], d["dz"]])
    e = Engine(d, max_particles=n + 3)
    e.load_bunch(xyz, 0.4 * rng.standard_normal((n, 3)), -1e-15 / n)
    prev = np.arange(n)
    for step in range(3):
        if step:
            e.step(1)
        _, _, cell, order = e.read_particles()
        key = _keys(cell, d)
        assert np.array_equal(order, prev[np.argsort(key[prev], kind="stable")]), step
        prev = order
