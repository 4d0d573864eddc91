"""Sub-steps of the push in each of its bodies (field type, compensation, single
module, arrays, optical), alone against the oracle and in a batch that mixes
them against the same runs alone; and steps whose end the next sweep carries, at
FP32 with and without compensation.

Bars: 1e-10 at FP64 and 2e-4 at FP32 against the oracle; 1e-11 and 1e-5 between
two runs of one program (the deposit's additions come in another order)."""
import numpy as np
import pytest
import torch  # noqa: F401

from paper_2009_13645_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(b))


def _recipe(prec, comp, n_sub, und_type=0, n=3000, every=1, shape=(32, 24, 48)):
    w = wl.config1()
    w.nx, w.ny, w.nz = shape
    w.n_particles, w.field_precision, w.compensated, w.sort_every, w.n_periods = n, prec, comp, every, 4
    w.und_type = 1 if und_type == 1 else 0
    d = dict(w.descriptor(), n_sub=n_sub, und_type=und_type)
    return d, wl.make_bunch(w)


def _engine(d, bunch, und=None):
    from paper_2009_13645_amd.engine import Engine
    e = Engine(d, max_particles=len(bunch[0]))
    if und:
        e.set_undulator(und)
    e.load_bunch(*bunch)
    return e


ARRAY = dict(n_modules=3, gap=0.03, dK=0.04)
PULSE = dict(signal=1, ctau=0.3, ct0=0.35, cep_deg=30.0)


@pytest.mark.parametrize("prec,comp,n_sub,und_type,und", [
    (64, 0, 3, 1, None), (32, 0, 2, 0, None), (32, 1, 3, 0, None), (64, 0, 2, 0, ARRAY), (32, 0, 3, 1, ARRAY),
    (32, 1, 2, 0, ARRAY), (64, 0, 2, 2, PULSE)])
def test_alone(prec, comp, n_sub, und_type, und):
    from oracle.oracle import Oracle
    d, bunch = _recipe(prec, comp, n_sub, und_type)
    o = Oracle(d)
    if und:
        o.set_undulator(und)
    o.load_bunch(*bunch)
    e = _engine(d, bunch, und)
    o.step(40)
    e.step(40)
    tol = 1e-10 if prec == 64 else 2e-4
    gx, gu = e.read_particles()[:2]
    ox, ou = o.particles()[:2]
    assert _rel(gx, ox) < tol and _rel(gu, ou) < tol
    for f in ("Ax", "Jz", "Q", "Ey"):
        if np.any(o.field(f)):
            assert _rel(e.read_field(f), o.field(f)) < tol, f


def test_batch_of_all_bodies():
    from paper_2009_13645_amd.engine import Batch
    kinds = [(p, c, n) for p, c in ((64, 0), (32, 0), (32, 1)) for n in (1, 3)]
    recipes = [_recipe(*k, und_type=i & 1, n=1000 + 700 * i) for i, k in enumerate(kinds)]
    members, alone = [_engine(*r) for r in recipes], [_engine(*r) for r in recipes]
    b = Batch(members)
    b.run(20)
    b.sync()
    for k, m, a in zip(kinds, members, alone):
        a.step(20)
        tol = 1e-11 if k[0] == 64 else 1e-5
        for x, y in list(zip(m.read_particles()[:2], a.read_particles()[:2])) + [
                (m.read_field("Ax"), a.read_field("Ax")), (m.power_history(20), a.power_history(20))]:
            assert _rel(x, y) < tol, k
    b.close()


@pytest.mark.parametrize("comp", [0, 1])
def test_fp32_steps_that_leave_their_end(comp):
    d, bunch = _recipe(32, comp, 1, n=9000, every=4)
    many, single = _engine(d, bunch), _engine(d, bunch)
    many.step(30)  # one call: the sweeps end the steps that no sort follows
    for _ in range(30):
        single.step(1)
    assert many.constants()["steps"] == 30
    assert _rel(many.power_history(30), single.power_history(30)) < 1e-5
    for x, y in zip(many.read_particles()[:2], single.read_particles()[:2]):
        assert _rel(x, y) < 1e-5
    for f in ("Ax", "Jz", "Q"):
        assert _rel(many.read_field(f), single.read_field(f)) < 1e-5, f
