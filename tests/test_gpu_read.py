"""Read-back calls on the GPU: every field in both types against the oracle,
reads between steps leaving the run as it was, and partial particle reads."""
import ctypes as C

import numpy as np
import pytest

from paper_2009_13645_amd import workloads as wl

pytestmark = pytest.mark.gpu

FIELDS = ("Ex", "Ey", "Ez", "Bx", "By", "Bz", "Ax", "Ay", "Az", "Jx", "Jy", "Jz", "F", "Q")


def _rel(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


@pytest.mark.parametrize("shape,prec,comp,sc", [((12, 9, 21), 64, 0, 1), ((9, 12, 21), 32, 1, 1),
                                                ((8, 8, 40), 32, 0, 0), ((45, 7, 33), 64, 0, 0)])
def test_reads_between_steps(shape, prec, comp, sc):
    from oracle.oracle import Oracle
    from paper_2009_13645_amd.engine import Engine
    w = wl.config1()
    w.nx, w.ny, w.nz = shape
    w.sigma_cells, w.n_particles = (1.0, 1.0, 1.5), 777
    w.field_precision, w.compensated, w.space_charge = prec, comp, sc
    xyz, u, q = wl.make_bunch(w)
    e, o = Engine(w.descriptor(), max_particles=1000), Oracle(w.descriptor())
    e.load_bunch(xyz, u, q)
    o.load_bunch(xyz, u, q)
    tol = 1e-10 if prec == 64 else 2e-4
    for _ in range(3):
        e.step(2)
        o.step(2)
        scale = {"E": 0.0, "B": 0.0, "A": 0.0, "J": 0.0}
        for name in FIELDS:
            if len(name) == 2:
                scale[name[0]] += float(np.sum(o.field(name) ** 2))
        for name in FIELDS:
            f64, f32 = e.read_field(name, np.float64), e.read_field(name, np.float32)
            assert np.array_equal(f64.astype(np.float32), f32), name
            ref = o.field(name)
            norm = scale[name[0]] ** 0.5 if len(name) == 2 else float(np.linalg.norm(ref))
            assert float(np.linalg.norm(f64 - ref)) <= tol * norm, name
        px, pu, cell, order = e.read_particles()
        ox, ou, oc, oo = o.particles()
        assert np.array_equal(cell, oc) and np.array_equal(order, oo)
        assert _rel(px, ox) < 1e-10 and _rel(pu, ou) < 1e-10
    # any pointer may be null
    only = np.empty((777, 3))
    rc = e._L.mithra_read_particles(e._h, None, only.ctypes.data_as(C.POINTER(C.c_double)), None, None)
    assert rc == 0 and np.array_equal(only, pu)


@pytest.mark.parametrize("shape,n,prec", [((40, 30, 301), 60001, 64), ((64, 64, 80), 30000, 32)])
def test_repeated_reads_are_equal(shape, n, prec):
    """The first reads of a run are copied directly, later ones through the
    handle's pinned halves (1 MiB each): the same values either way."""
    from paper_2009_13645_amd.engine import Engine
    w = wl.config1()
    w.nx, w.ny, w.nz = shape
    w.n_particles, w.field_precision = n, prec
    xyz, u, q = wl.make_bunch(w)
    e = Engine(w.descriptor(), max_particles=n)
    e.load_bunch(xyz, u, q)
    e.step(5)
    first = [e.read_field("Ax"), e.read_field("Ey", np.float32), *e.read_particles(), e.power_history(5)]
    scalars = [e.radiated_power(), e.bunching()]
    for _ in range(10):
        again = [e.read_field("Ax"), e.read_field("Ey", np.float32), *e.read_particles(), e.power_history(5)]
        for a, b in zip(first, again):
            assert np.array_equal(a, b)
        assert [e.radiated_power(), e.bunching()] == scalars
