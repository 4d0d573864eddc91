"""The step-fields launch where its stages meet: particles and the power
plane beside the boundary, whose n+1 values the vertex fields compute
themselves, with fused and unfused x faces, both Mur orders and the spectrum."""
import numpy as np
import pytest

from paper_2009_13645_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,prec,order,sc,plane", [((8, 8, 12), 64, 2, 1, 1), ((8, 10, 12), 64, 1, 0, 10),
                                                       ((9, 8, 14), 64, 2, 1, 12), ((12, 9, 12), 32, 2, 1, 5),
                                                       ((7, 11, 12), 32, 1, 1, 1)])
def test_fields_beside_the_boundary(shape, prec, order, sc, plane):
    from oracle.oracle import Oracle
    from paper_2009_13645_amd.engine import Engine
    w = wl.config1()
    w.nx, w.ny, w.nz = shape
    w.n_particles, w.field_precision, w.truncation_order, w.space_charge = 600, prec, order, sc
    w.center_frac_z, w.k_plane, w.charge_C = 0.5, plane, 1e-9
    d = dict(w.descriptor(), n_freq=2, nu_min=0.8, nu_max=1.2)
    # particles over the whole active region, so that every face is beside one
    rng = np.random.default_rng(9)
    g = 1.0 + rng.random((600, 3)) * (np.array(shape) - 3.0)
    xyz = np.array([d["x0"], d["y0"], d["z0"]]) + g * np.array([d["dx"], d["dy"], d["dz"]])
    u = 0.05 * rng.standard_normal((600, 3))
    e, o = Engine(d, max_particles=600), Oracle(d)
    o.set_spectrum(2, 0.8, 1.2)
    e.load_bunch(xyz, u, -1e-9 / 600)
    o.load_bunch(xyz, u, -1e-9 / 600)
    power = []
    for _ in range(6):
        e.step(1)
        o.step(1)
        power.append(o.radiated_power())
    tol = 1e-10 if prec == 64 else 2e-4
    rel = lambda a, b: float(np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(b))  # noqa: E731
    _, gu, gc, _ = e.read_particles()
    _, ou, oc, _ = o.particles()
    assert rel(gu, ou) < tol and rel(e.power_history(6), power) < tol
    assert rel(e.spectral_power(), o.spectral_power()) < tol
    for f in ("Ax", "Ay", "Az"):
        assert rel(e.read_field(f), o.field(f)) < tol, f
    if prec == 64:
        assert np.array_equal(gc, oc)
