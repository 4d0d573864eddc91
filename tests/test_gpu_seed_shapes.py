"""Seeded runs on sweep tiles of every width and depth, and the shapes that a
seeded run takes once it is seeded: its default one and the scalar ones."""
import numpy as np
import pytest
import torch  # noqa: F401

from paper_2009_13645_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _seeded(prec, shape_before=None):
    from paper_2009_13645_amd.engine import Engine
    w = wl.config1()
    w.nx, w.ny, w.nz, w.n_particles = 36, 11, 24, 300
    w.sigma_cells, w.field_precision = (0.5, 0.5, 1.0), prec
    d = w.descriptor()
    lam = 2.25e-6
    seed = dict(type=1, signal=1, a0=0.02, wavelength=lam, ctau=2 * lam, ct0=1.5 * lam, cep_deg=10.0, pol_deg=30.0,
                w0=6 * d["dx"], z_focus=d["z0"] + 30 * d["dz"])
    e = Engine(d, max_particles=300)
    if shape_before is not None:
        e.set_sweep_shape(shape_before)
    e.set_seed(seed)
    e.load_bunch(*wl.make_bunch(w))
    return e, w, d, seed


def test_the_default_shape_can_be_restored():
    from paper_2009_13645_amd.engine import MithraError
    a, b = _seeded(64)[0], _seeded(64)[0]
    own = a.autotune_sweep(2)  # a seeded run keeps its shape and reports it
    a.set_sweep_shape(own)
    a.step(2)
    a.set_sweep_shape(0)  # scalar
    a.step(2)
    a.set_sweep_shape(own)
    a.step(2)
    b.step(6)
    for f in ("Ax", "Ay"):
        x, y = a.read_field(f), b.read_field(f)
        assert np.linalg.norm(x - y) <= 1e-12 * np.linalg.norm(y)
    for other in set(range(8, 18)) - {own}:  # as before, none of the other vector shapes
        with pytest.raises(MithraError):
            a.set_sweep_shape(other)


@pytest.mark.parametrize("prec", [64, 32])
def test_seed_on_every_shape(prec):
    from oracle.oracle import Oracle
    o = None
    for shape in range(18):
        e, w, d, seed = _seeded(prec, shape)  # a shape chosen before the seed stays
        if o is None:
            o = Oracle(d)
            o.set_seed(seed)
            o.load_bunch(*wl.make_bunch(w))
            o.step(40)
            norm = sum(float(np.sum(o.field(f) ** 2)) for f in ("Ax", "Ay", "Az")) ** 0.5
        e.step(40)
        for f in ("Ax", "Ay", "Az"):
            assert float(np.linalg.norm(e.read_field(f) - o.field(f))) < (1e-10 if prec == 64 else 2e-4) * norm, (shape, f)
        e.close()
