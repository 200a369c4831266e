"""Device memory that set-up calls hand from one to another, on the host: libhgnn.so runs on a runtime that executes nothing but
knows which streams have work in flight (fake_hip.cpp).  A block may go back only when nothing in flight uses it."""
import ctypes
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2411_01109_amd", "libhgnn.so")
OK, ENOMEM, EHIP = 0, 3, 4
vp, i32, i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
V, E, F = 1000, 20000, 64


class Csr(ctypes.Structure):
    _fields_ = [("nrows", i32), ("ncols", i32), ("nnz", i64), ("rowptr", vp), ("col", vp), ("row", vp), ("eid", vp)]


class Host:
    """The library on the fake runtime."""

    def __init__(self, fake, lib):
        self.fake = ctypes.CDLL(fake, mode=ctypes.RTLD_GLOBAL)
        self.lib = ctypes.CDLL(lib)
        self.path = lib.encode()
        self.keep = [(ctypes.c_int32 * (E + V + 2))() for _ in range(4)]
        self.data = ctypes.addressof((ctypes.c_char * (E * F * 4)).from_buffer(bytearray(E * F * 4)))
        self.data = (self.data + 255) // 256 * 256
        a = [ctypes.addressof(k) for k in self.keep]
        self.g = Csr(V, V, E, a[0], a[1], None, None)
        self.out = a[2], a[3]
        self.lib.hgnn_plan_destroy.argtypes = [vp]
        self.lib.hgnn_plan_destroy.restype = None
        self.fake.fake_launched.restype = ctypes.c_char_p
        self.reset()

    def reset(self):
        self.lib.hgnn_release_cached_memory()
        self.fake.fake_reset(self.path)

    def plan(self, stream, col_blocks=1):
        p = vp()
        st = self.lib.hgnn_plan_create(ctypes.byref(self.g), 256, F, 1, col_blocks, ctypes.byref(p), vp(stream))
        return st, p

    def compute(self, p, stream):
        """An asynchronous call that uses the plan."""
        x = vp(self.data)
        return self.lib.hgnn_edge_softmax(ctypes.byref(self.g), p, 1, x, x, vp(stream))


A, B = 0x1001, 0x1002  # streams of device 0
C = 0x2001             # of device 1


def destroy_on_another_device(h):
    """The plan's device is waited for, whatever device is current when it is destroyed."""
    h.fake.hipSetDevice(1)
    st, p = h.plan(C)
    assert st == OK and h.compute(p, C) == OK and h.fake.fake_busy(1) == 1
    h.fake.hipSetDevice(0)
    h.lib.hgnn_plan_destroy(p)
    assert h.fake.fake_freed_busy() == 0
    d = ctypes.c_int()
    h.fake.hipGetDevice(ctypes.byref(d))
    assert d.value == 0


def failed_wait(h):
    """A plan whose wait failed may still be in use: its blocks go back to the runtime, not to the next plan."""
    st, p = h.plan(A)
    assert st == OK
    before = h.fake.fake_mallocs()
    st, q = h.plan(A)
    blocks = h.fake.fake_mallocs() - before  # of one plan: the temporaries were there
    assert st == OK and h.compute(q, A) == OK
    h.fake.fake_fail_waits(1)
    h.lib.hgnn_plan_destroy(q)
    h.fake.fake_fail_waits(0)
    before = h.fake.fake_mallocs()
    st, q = h.plan(B)
    assert st == OK and blocks > 0 and h.fake.fake_mallocs() - before == blocks
    h.lib.hgnn_plan_destroy(q)
    h.lib.hgnn_plan_destroy(p)


def destroyed_during_a_capture(h):
    """Neither the capture nor the blocks are spoiled when a plan is destroyed by the thread that captures."""
    st, p = h.plan(A)
    assert st == OK and h.compute(p, A) == OK
    h.fake.fake_capture(1)
    h.lib.hgnn_plan_destroy(p)
    assert h.fake.fake_spoiled() == 0 and h.fake.fake_freed_busy() == 0
    h.fake.fake_capture(0)


def replaced_groups(h):
    """Groups that a call on the plan still uses are not given to another set-up call."""
    st, p = h.plan(A)
    add = lambda: h.lib.hgnn_plan_add_groups(p, ctypes.byref(h.g), 32, vp(B))
    assert st == OK and add() == OK and h.compute(p, A) == OK and h.fake.fake_busy(0) == 1
    assert add() == OK and h.fake.fake_freed_busy() == 0
    h.lib.hgnn_plan_destroy(p)


def replaced_slices(h):
    st, p = h.plan(A)
    add = lambda: h.lib.hgnn_plan_add_slices(p, ctypes.byref(h.g), 0, vp(B))
    assert st == OK and add() == OK and h.compute(p, A) == OK and h.fake.fake_busy(0) == 1
    assert add() == OK and h.fake.fake_freed_busy() == 0
    h.lib.hgnn_plan_destroy(p)


def failed_calls(h):
    """Set-up calls that fail half-way leave nothing in flight that uses the blocks they give back: every allocation fails
    in turn, and every wait."""
    st, p = h.plan(A)
    assert st == OK
    g = ctypes.byref(h.g)
    r, c = vp(h.out[0]), vp(h.out[1])
    calls = [lambda: h.lib.hgnn_csr_validate(g, vp(A)), lambda: h.lib.hgnn_plan_add_groups(p, g, 32, vp(A)),
             lambda: h.lib.hgnn_plan_add_slices(p, g, 0, vp(A)), lambda: h.plan(A)[0], lambda: h.plan(A, 3)[0],
             lambda: h.lib.hgnn_transpose(g, r, c, c, vp(A)),
             lambda: h.lib.hgnn_coo_to_csr(V, V, i64(E), vp(h.g.rowptr), vp(h.g.col), r, c, c, vp(A))]
    for k, call in enumerate(calls):
        for n in range(60):
            h.lib.hgnn_release_cached_memory()
            h.fake.fake_fail_malloc(n)
            st = call()
            h.fake.fake_fail_malloc(-1)
            assert h.fake.fake_freed_busy() == 0 and h.fake.fake_busy(0) == 0, (k, n)
            if st == OK:
                break
        assert st == OK and n > 0, (k, n)
        h.fake.fake_fail_waits(1)
        assert call() == EHIP, k
        assert h.fake.fake_freed_busy() == 0, k
        h.fake.fake_fail_waits(0)
        h.fake.hipDeviceSynchronize()
    h.lib.hgnn_plan_destroy(p)


def bytes_per_non_zero(h):
    """What a plan holds for every non-zero of a graph that the automatic rule cuts into column blocks: a 16-bit column id, its slot
    where the graph has a map, and two row ids per segment (lists of pieces aside, which depend on the rows)."""
    h.fake.fake_live_bytes.restype = ctypes.c_size_t
    for eid, most in ((None, 2.2), (h.g.rowptr, 6.2)):
        total = []
        for nnz in (1 << 24, 1 << 25):
            h.reset()
            h.g = Csr(20000, 120000, nnz, h.g.rowptr, h.g.col, None, eid)  # a table of 15 MB, rows of 800 and more
            st, p = h.plan(A, 0)
            assert st == OK and h.lib.hgnn_plan_col_blocks(p) == 2 and h.lib.hgnn_plan_col_blocks_fine(p) == 4
            h.lib.hgnn_release_cached_memory()
            total.append(h.fake.fake_live_bytes())
            h.lib.hgnn_plan_destroy(p)
        assert total[1] - total[0] <= most * (1 << 24), (eid, total)


SCENARIOS = [destroy_on_another_device, failed_wait, destroyed_during_a_capture, replaced_groups, replaced_slices, failed_calls, bytes_per_non_zero]


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I/opt/rocm/include",
                           os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", so, "-ldl"])
    return so


@pytest.mark.parametrize("name", [s.__name__ for s in SCENARIOS])
def test_blocks_in_flight(hgnn, fake, name):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), fake, LIB, name], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    host = Host(sys.argv[1], sys.argv[2])
    {s.__name__: s for s in SCENARIOS}[sys.argv[3]](host)
    print("ok")
