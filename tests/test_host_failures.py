"""The host side of the library under failures that a device rarely gives, over a stand-in for the
HIP runtime (host_runtime.cpp): every runtime call of an entry point made to fail in turn.  No GPU is
touched."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_1709_02733_amd import build as B
from paper_1709_02733_amd import el

HERE = os.path.dirname(os.path.abspath(__file__))
vp = ctypes.c_void_p


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("host") / "host.so")
    srcs = [os.path.join(B.CSRC, f) for f in ("el_api.hip", "el_exec.hip", "el_group.hip")]
    subprocess.run([B.HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared",
                    "-I" + os.path.join(B.ROOT, "include"), "-I" + B.CSRC, *srcs, os.path.join(HERE, "host_runtime.cpp"),
                    "-Wl,-Bsymbolic", "-o", so], check=True)
    lib = ctypes.CDLL(so)
    for name in ("fail_call", "fail_new"):
        getattr(lib, name).argtypes = [ctypes.c_longlong]
        getattr(lib, name).restype = None
    for name in ("calls", "news", "handles"):
        getattr(lib, name).restype = ctypes.c_longlong
    lib.fail_call(-1)
    lib.fail_new(-1)
    return lib


class Plan:
    """A plan over host memory (the stand-in classifies every other tile as fluid)."""

    def __init__(self, lib, shape=(70, 21, 40), npml=3, nsteps=9, nrec=20):
        self.lib = lib
        nx, ny, nz = shape
        self.grid = el.make_grid(nx, ny, nz, 1e-4, 1e-8, nsteps, npml)
        n = ctypes.c_size_t(0)
        assert lib.el_plan_bytes(ctypes.byref(self.grid), nrec, ctypes.byref(n)) == 0
        self.nbytes = n.value
        raw = np.zeros(n.value + 256, np.uint8)
        off = -raw.ctypes.data % 256
        self.ws = raw[off:off + n.value]
        self.maps = np.zeros(nx * ny * nz, np.float32)
        self.rec = np.ascontiguousarray(np.random.default_rng(1).uniform(size=(nrec, 3)) * (np.array(shape) - 1) * 1e-4)
        self.traces = np.zeros((nsteps, nrec))
        self.image = np.zeros(nx * ny * nz, np.float32)
        self.nrec = nrec
        self.h = vp(None)

    def create(self):
        m = vp(self.maps.ctypes.data)
        return self.lib.el_plan_create(ctypes.byref(self.h), ctypes.byref(self.grid), m, m, m, m, None,
                                       vp(self.rec.ctypes.data), self.nrec, vp(self.ws.ctypes.data),
                                       ctypes.c_size_t(self.nbytes), None)

    def fluid(self, enable):
        return self.lib.el_plan_fluid_path(self.h, enable, None)

    def tables(self):
        return [getattr(self.lib, "table_" + n)(self.h) for n in ("per", "of", "inc", "rec", "entries")]

    def forward(self):
        return self.lib.el_forward(self.h, vp(self.image.ctypes.data), vp(self.traces.ctypes.data), None)

    def adjoint(self):
        return self.lib.el_adjoint(self.h, vp(self.traces.ctypes.data), vp(self.image.ctypes.data), None)

    def destroy(self):
        self.lib.el_plan_destroy(self.h)
        self.h = vp(None)


def _tables_of_both(host):
    p = Plan(host)
    assert p.create() == el.EL_OK
    on = p.tables()
    assert p.fluid(0) == el.EL_OK
    off = p.tables()
    assert p.fluid(1) == el.EL_OK and p.tables() == on
    p.destroy()
    assert on[1:4] == [1, 1, 3] and off[1:4] == [0, 0, 0] and on != off
    return on, off


def test_a_failed_change_of_the_fluid_update_leaves_the_plan_as_it_was(host):
    """Every runtime call of the first change fails in turn; so does the list's room.  The plan's
    passes still take the list of the setting it had, and a later change succeeds."""
    on, off = _tables_of_both(host)
    n = 0
    while True:
        p = Plan(host)
        assert p.create() == el.EL_OK
        host.fail_call(n)
        st = p.fluid(0)
        reached = host.calls() > n
        host.fail_call(-1)
        if not reached:
            assert st == el.EL_OK and p.tables() == off
            p.destroy()
            break
        assert st == el.EL_EDEVICE
        assert p.tables() == on
        stats = el.FluidStats()
        assert host.el_plan_fluid_path(p.h, -1, ctypes.byref(stats)) == el.EL_OK and stats.tiles > 0
        assert p.fluid(0) == el.EL_OK and p.tables() == off
        assert p.fluid(1) == el.EL_OK and p.tables() == on
        p.destroy()
        n += 1
    assert n >= 4
    p = Plan(host)
    assert p.create() == el.EL_OK
    room = host.room(p.h)
    host.set_room(p.h, 1)
    assert p.fluid(0) == el.EL_EINVAL and p.tables() == on
    host.set_room(p.h, room)
    assert p.fluid(0) == el.EL_OK and p.tables() == off
    p.destroy()


def test_a_failed_creation_leaves_nothing_behind(host):
    n, before = 0, host.handles()
    while True:
        p = Plan(host)
        host.fail_call(n)
        st = p.create()
        reached = host.calls() > n
        host.fail_call(-1)
        if not reached:
            assert st == el.EL_OK
            p.destroy()
            break
        assert st == el.EL_EDEVICE and not p.h.value
        assert host.handles() == before
        n += 1
    assert n > 10 and host.handles() == before


def _each_failed_allocation(host, call, check):
    """call() with its 0th, 1st, ... allocation failing until it makes no more: it returns EL_ENOMEM
    each time (an exception that left it would end the process) and check() holds after it."""
    n = 0
    while True:
        host.fail_new(n)
        st = call()
        reached = host.news() > n
        host.fail_new(-1)
        if not reached:
            return n, st
        assert st == el.EL_ENOMEM
        check()
        n += 1


def test_no_exception_leaves_the_plan_entry_points(host):
    before = host.handles()
    p = Plan(host)

    def nothing():
        assert not p.h.value and host.handles() == before

    n, st = _each_failed_allocation(host, p.create, nothing)
    assert st == el.EL_OK and n > 10
    on, off = _tables_of_both(host)

    def as_it_was():
        assert p.tables() == on

    n, st = _each_failed_allocation(host, lambda: p.fluid(0), as_it_was)
    assert st == el.EL_OK and n > 4 and p.tables() == off
    for call in (p.forward, p.adjoint):   # the events of the timed launches
        assert host.el_plan_timing(p.h, 1) == el.EL_OK
        assert _each_failed_allocation(host, call, lambda: None)[1] == el.EL_OK
    p.destroy()
    assert host.handles() == before


def test_no_exception_leaves_the_executor_and_the_group(host):
    before = host.handles()
    p = Plan(host)
    assert p.create() == el.EL_OK
    held = host.handles()
    ex, g, slot = vp(None), vp(None), ctypes.c_int32(-1)

    def nothing():
        assert host.handles() == held

    n, st = _each_failed_allocation(host, lambda: host.el_exec_create(ctypes.byref(ex), 3, 4), nothing)
    assert st == el.EL_OK and n >= 2
    assert _each_failed_allocation(host, lambda: host.el_exec_set_ahead(ex, 5), lambda: None)[1] == el.EL_OK
    n, st = _each_failed_allocation(
        host, lambda: host.el_exec_start(ex, p.h, el.OP_FORWARD, vp(p.image.ctypes.data), vp(p.traces.ctypes.data), None,
                                         ctypes.byref(slot)), lambda: None)
    assert st == el.EL_OK and host.el_exec_wait(ex, slot) == el.EL_OK
    assert host.el_exec_destroy(ex) == el.EL_OK
    nothing()
    n, st = _each_failed_allocation(host, lambda: host.el_group_create(ctypes.byref(g), 3, el.EL_F32), nothing)
    assert st == el.EL_OK and n >= 2
    n, st = _each_failed_allocation(
        host, lambda: host.el_group_add(g, p.h, el.OP_ADJOINT, vp(p.traces.ctypes.data), vp(p.image.ctypes.data), None,
                                        ctypes.byref(slot)), lambda: None)
    assert st == el.EL_OK
    steps = ctypes.c_int32(0)

    def no_half_step():
        assert host.el_group_poll(g, slot, ctypes.byref(steps), None) == el.EL_OK and steps.value in (0, 2)

    n, st = _each_failed_allocation(host, lambda: host.el_group_run(g, 2), no_half_step)
    assert st == el.EL_OK and n >= 2
    assert host.el_group_destroy(g) == el.EL_OK
    nothing()
    p.destroy()
    assert host.handles() == before
