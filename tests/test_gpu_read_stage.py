"""Reads through a handle's pinned memory (a handle has it after 48 read calls
or MiB): the non-finite report, calls that return nothing, its release, members
of a batch."""
import numpy as np
import pytest
import torch  # noqa: F401

from paper_2009_13645_amd import workloads as W

pytestmark = pytest.mark.gpu


def _stage(e):
    for _ in range(50):
        e.read_field("Ax")


def _run(n, q, prec, steps=0):
    from paper_2009_13645_amd.engine import Engine
    w = W.config1()
    w.n_particles, w.field_precision = n, prec
    d = w.descriptor()
    d["k_plane"] = int(round(w.center_z_cells))  # the power plane through the bunch
    xyz, u, _ = W.make_bunch(w)
    e = Engine(d, max_particles=n)
    e.load_bunch(xyz, u, q)
    e.step(steps)
    return e


def test_non_finite_run_is_reported_by_every_read():
    from paper_2009_13645_amd.engine import MithraError
    e = _run(256, -1e30, 32)  # rho ~ 1e42 C/m^3: above the FP32 range
    _stage(e)
    assert not np.any(e.read_field("Ex")) and not np.any(e.read_field("Bz"))  # step 0: zero
    assert e._L.mithra_read_particles(e._h, None, None, None, None) == 0
    e.step(3)
    for read in (lambda: e.read_field("Az"), lambda: e.read_field("Ex"), e.read_particles):
        with pytest.raises(MithraError) as ei:
            read()
        assert ei.value.code == -5
    assert e._L.mithra_read_particles(e._h, None, None, None, None) == -5


def test_destroy_does_not_wait_for_another_handle():
    a, b = _run(4096, -1e-15, 64), _run(4096, -1e-15, 64)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        c = _run(4096, -1e-15, 64)  # on the other stream
    for e in (a, b):
        _stage(e)
    torch.cuda.synchronize()
    c.step(8000)  # some 200 ms of work
    done = torch.cuda.Event()
    done.record(side)
    a.close()
    assert not done.query()  # c still steps
    field = b.read_field("Ax")
    _stage(c)
    assert not np.any(field) and np.all(np.isfinite(c.read_field("Ax")))
    b.close()
    c.close()


def test_members_of_a_batch():
    from paper_2009_13645_amd.engine import Batch
    sizes = [(4096, 64), (1500, 32)]
    alone = [_run(n, -1e-15, p, 12) for n, p in sizes]
    members = [_run(n, -1e-15, p) for n, p in sizes]
    for e in members:
        _stage(e)
    b = Batch(members)
    b.run([12, 12])  # the reads wait for the batch
    for (n, p), e, a in zip(sizes, members, alone):
        tol = 1e-11 if p == 64 else 1e-5  # the deposit's additions come in another order
        pairs = [(e.read_field(f), a.read_field(f)) for f in ("Ay", "Q", "By")]
        pairs += list(zip(e.read_particles()[:2], a.read_particles()[:2]))
        pairs += [(e.power_history(12), a.power_history(12)), (e.bunching(), a.bunching())]
        for x, y in pairs:
            assert np.linalg.norm(np.asarray(x) - y) <= tol * np.linalg.norm(y), p
    b.close()
