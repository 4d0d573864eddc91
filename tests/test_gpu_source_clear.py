"""The clearing of a source set, whole (small boxes) and by the marks of the
sort tiles (boxes over 8 MB): particles over the grid that cross cells and
tiles every few steps leave no old current or charge behind."""
import numpy as np
import pytest

from paper_2009_13645_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,tile,prec,comp", [((48, 48, 260), (8, 8, 8), 64, 0), ((48, 48, 260), (4, 4, 4), 32, 1),
                                                  ((47, 50, 259), (1, 2, 3), 64, 0), ((24, 22, 40), (4, 4, 4), 64, 0)])
def test_no_deposit_of_an_earlier_step_is_left(shape, tile, prec, comp):
    from oracle.oracle import Oracle
    from paper_2009_13645_amd.engine import Engine
    n = 3000
    w = wl.config1()
    w.nx, w.ny, w.nz = shape
    w.n_particles, w.field_precision, w.charge_C, w.sort_every = n, prec, 1e-12, 3
    w.compensated = comp
    w.k_plane = shape[2] - 20
    w.tile = tile
    d = w.descriptor()
    rng = np.random.default_rng(4)
    g = 1.5 + rng.random((n, 3)) * (np.array(shape) - 4.0)
    xyz = np.array([d["x0"], d["y0"], d["z0"]]) + g * np.array([d["dx"], d["dy"], d["dz"]])
    u = 2.0 * rng.standard_normal((n, 3))  # a good part of a cell a step
    e, o = Engine(d, max_particles=n), Oracle(d)
    e.load_bunch(xyz, u, -1e-12 / n)
    o.load_bunch(xyz, u, -1e-12 / n)
    tol = 1e-10 if prec == 64 else 2e-4
    for step in range(7):
        e.step(1)
        o.step(1)
        for f in ("Jx", "Jy", "Jz", "Q"):
            a, b = e.read_field(f), o.field(f)
            assert np.linalg.norm(a - b) < tol * np.linalg.norm(b), (step, f)
