"""Sweeps that advance three potentials (no space charge), whose workgroups
end after A_z: scalar and vector tiles of a single run, and members with and
without space charge in one batch."""
import numpy as np
import pytest

from paper_2009_13645_amd import workloads as wl

pytestmark = pytest.mark.gpu


def make(shape, prec, sc, seed):
    from oracle.oracle import Oracle
    from paper_2009_13645_amd.engine import Engine
    w = wl.config1()
    w.nx, w.ny, w.nz = shape
    w.n_particles, w.field_precision, w.space_charge, w.seed = 2000, prec, sc, seed
    d = w.descriptor()
    xyz, u, q = wl.make_bunch(w)
    e, o = Engine(d, max_particles=len(xyz)), Oracle(d)
    e.load_bunch(xyz, u, q)
    o.load_bunch(xyz, u, q)
    return e, o


def check(e, o, prec, what):
    tol = 1e-10 if prec == 64 else 2e-4
    for f in ("Ax", "Ay", "Az", "F"):
        a, b = e.read_field(f), o.field(f)
        assert np.linalg.norm(a - b) <= tol * np.linalg.norm(b), (what, f)


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("tile", [0, 5, 8, 11, 12, 17])
def test_single_run(prec, tile):
    e, o = make((36, 28, 43), prec, 0, 3)
    e.set_sweep_shape(tile)
    e.step(20)
    o.step(20)
    check(e, o, prec, tile)


def test_mixed_batch():
    from paper_2009_13645_amd.engine import Batch
    kinds = [((32, 32, 48), 64, 0), ((40, 33, 40), 64, 1), ((36, 32, 64), 32, 0), ((32, 40, 41), 32, 1)]
    pairs = [make(s, p, sc, 5 + i) for i, (s, p, sc) in enumerate(kinds)]
    b = Batch([e for e, _ in pairs])
    b.run([20] * len(pairs))
    for (e, o), (s, p, sc) in zip(pairs, kinds):
        o.step(20)
        check(e, o, p, (s, p, sc))
