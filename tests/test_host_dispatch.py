"""The plan-free SpMM's choice of kernels, on the host: libhgnn.so on a runtime that executes nothing and writes launches down
(fake_hip.cpp)."""
import ctypes
import os
import re
import subprocess
import sys

import pytest

from test_host_memory import A, LIB, ROOT, Csr, Host, fake, i64, vp  # noqa: F401

V, E, F = 200000, 4000000, 64


def up(n):
    return (n + 255) // 256 * 256


def chunk_bytes(nrows, nnz, f):
    """What the chunks of the long rows need: lists of chunks and of long rows, a partial row in fp32 for every chunk."""
    long_row = min(max(256, 8 * (nnz // nrows)), 1024)
    if nnz <= long_row:
        return 0
    rows = nnz // long_row + 1
    chunks = nnz // 512 + rows + 1
    return 256 + 2 * up(4 * chunks) + 2 * up(4 * rows) + up(4 * chunks * ((f + 7) // 8 * 8))


def launches(h, call):
    h.fake.fake_reset(h.path)
    st = call()
    names = h.fake.fake_launched().decode().split()
    return st, [re.sub(r"^_ZN4hgnn\d+", "", n) for n in names]


def spmm(h, g, f, nbytes, w=None):
    x = vp(h.data)
    return launches(h, lambda: h.lib.hgnn_spmm(ctypes.byref(g), w, 1, x, i64(f), x, i64(f), f, 0, None, x if nbytes else None,
                                               ctypes.c_size_t(nbytes), vp(A)))


def graph(h, nrows, ncols, nnz, eid=False):
    return Csr(nrows, ncols, nnz, h.g.rowptr, h.g.col, None, h.g.rowptr if eid else None)


def smaller_workspaces(h):
    """A workspace that holds the chunks of the long rows is enough, as before rows were listed as pieces; one byte less is not."""
    for nrows, nnz, f in ((V, E, 64), (1200001, 31000001, 64), (100003, 1300001, 42), (3000000, 18000000, 128), (30000, 300000, 512)):
        for eid in (False, True):
            g = graph(h, nrows, nrows, nnz, eid)
            w = vp(h.data)
            least = chunk_bytes(nrows, nnz, f)
            st, names = spmm(h, g, (f + 7) // 8 * 8, least, w)
            assert st == 0 and names, (nrows, nnz, f, st)
            st, names = spmm(h, g, (f + 7) // 8 * 8, least - 1, w)
            assert st == 1 and not names, (nrows, nnz, f, st)
            st, names = spmm(h, g, (f + 7) // 8 * 8, 0, w)
            assert st == 0 and len(names) == 1
            full = h.lib.hgnn_spmm_workspace(nrows, 0, i64(nnz), f)  # a few bytes less than named: refused, unless those are the chunks'
            for short in (1, 256, 512):
                st, names = spmm(h, g, (f + 7) // 8 * 8, full - short, w)
                assert st == (0 if full - short == least else 1), (nrows, nnz, f, short)
    # column passes with their own room behind the chunks
    nrows, nnz, f = 233000, 114000000, 64
    g = graph(h, nrows, nrows, nnz)
    passes = round(2.0 * nrows * f / (2 * (4 << 20)))
    room = up(4 * nrows * (passes + 1)) + up(4 * passes * nrows * f)
    for size in (chunk_bytes(nrows, nnz, f) + room, h.lib.hgnn_spmm_workspace(nrows, nrows, i64(nnz), f)):
        st, names = spmm(h, g, f, size)
        assert st == 0 and any("row_pass" in n for n in names), names
    st, names = spmm(h, g, f, h.lib.hgnn_spmm_workspace(nrows, 0, i64(nnz), f))
    assert st == 0 and not any("row_pass" in n for n in names), names


def static_form(h):
    """hgnn_spmm_static launches what hgnn_spmm does with hgnn_spmm_workspace(nrows, 0, nnz, F) bytes, and refuses what needs more
    than its array: also where the pieces of all rows do not fit it and the chunks of the long rows do, and where passes would."""
    limit = h.lib.hgnn_spmm_static_limit()
    seen = set()
    for nrows in (30, 1000, 30000, 300000, 1700000, 3000000):
        for nnz in (200, 2000, 100000, 1500000, 8000000, 30000000, 90000000):
            for f in (8, 40, 64, 128, 512):
                for weighted, eid in ((False, False), (True, False), (True, True)):
                    if f == 512 and (nrows > 100000 or nnz > 30000000):
                        continue
                    ld = (f + 7) // 8 * 8
                    g = graph(h, nrows, 200000, nnz, eid)
                    w, x = (vp(h.data) if weighted else None), vp(h.data)
                    need = h.lib.hgnn_spmm_workspace(nrows, 0, i64(nnz), f)
                    st, names = launches(h, lambda: h.lib.hgnn_spmm_static(ctypes.byref(g), w, 1, x, i64(ld), x, i64(ld), f, 0, None, vp(A)))
                    assert (st == 0) == (need <= limit), (nrows, nnz, f, st, need)
                    if st:
                        assert st == 2 and not names
                        seen.add("refused")
                        continue
                    st, same = spmm(h, g, ld, need, w)
                    assert st == 0 and same == names, (nrows, nnz, f, weighted, eid, names, same)
                    seen.add(names[0][:8])
                    if need < h.lib.hgnn_spmm_workspace(nrows, 200000, i64(nnz), f):
                        seen.add("smaller")
    assert {"refused", "smaller", "task_cou", "hub_zero", "spmm_row"} <= seen, seen


def narrow_features(h):
    """Whatever the workspace, narrow features keep the kernels that take rows in storage order, unless values are behind a map."""
    for nrows, nnz in ((100000, 1300000), (1200001, 31000001)):
        for eid in (False, True):
            g = graph(h, nrows, nrows, nnz, eid)
            for f in (8, 24, 32, 56, 64, 128):
                n = h.lib.hgnn_spmm_workspace(nrows, nrows, i64(nnz), f)
                for w, least in ((None, 64), (vp(h.data), 8 if eid else 32)):
                    st, names = spmm(h, g, f, n, w)
                    assert st == 0 and any("task" in x for x in names) == (f >= least), (f, eid, names)


def column_ranges(h):
    """Long rows are cut at column ranges where the workspace is the query's for the graph's columns and that pays, never below 4 Mi
    non-zeros or over a table that the L2s hold together, and never in the static form."""
    for nrows, ncols, nnz, f, eid, want in ((1200001, 1200001, 31000001, 64, True, True), (1200001, 1200001, 31000001, 64, False, False),
                                            (2400000, 2400000, 54000000, 64, False, True), (600000, 600000, 12000000, 128, False, True),
                                            (262144, 262144, 5505024, 64, True, False), (600000, 600000, 4000000, 128, True, False)):
        g = graph(h, nrows, ncols, nnz, eid)
        w = vp(h.data)
        full, less = (h.lib.hgnn_spmm_workspace(nrows, c, i64(nnz), f) for c in (ncols, 0))
        for size, take in ((full, want), (full + 4096, want), (full - 1, False), (less, False)):
            if size < less:  # the answer has no room for ranges, and one byte less has none for the pieces
                continue
            st, names = spmm(h, g, f, size, w)
            assert st == 0 and any("free_count" in x for x in names) == take, (nrows, nnz, f, eid, size, names)


def room_for_column_ranges(h):
    """Beside the pieces of all rows the query counts at most a staged row and a list entry per 128 non-zeros, the cuts and an entry for every
    256, and ten counts per 1024 rows; nothing for features that no call over pieces takes."""
    for nrows, nnz, f in ((1200001, 31000001, 64), (2400000, 62000000, 128), (600000, 14000000, 256), (20000000, 40000000, 8), (200000, 6000000, 128)):
        ld = (f + 7) // 8 * 8
        full, less = (h.lib.hgnn_spmm_workspace(nrows, n, i64(nnz), f) for n in (nrows, 1))
        room = nnz // 128 * (4 * ld + 16) + (nnz // 256 + 1) * (28 + 16) + (nrows // 1024 + 1) * 48 + 4096
        assert 0 < full - less <= room, (nrows, nnz, f, full, less, room)
    assert h.lib.hgnn_spmm_workspace(1200001, 1200001, i64(31000001), 520) == h.lib.hgnn_spmm_workspace(1200001, 1, i64(31000001), 520)


def many_windows(h):
    """Beyond 400 windows of 1024 rows a launch scans their counts, for pieces and with column ranges, instead of every workgroup."""
    for nrows in (409600, 409601, 20000000):
        g = graph(h, nrows, 5000000, 41000000, True)
        for ncols, kind in ((1, "task_write"), (5000000, "free_write")):
            st, names = spmm(h, g, 16, h.lib.hgnn_spmm_workspace(nrows, ncols, i64(41000000), 16), vp(h.data))
            assert st == 0 and any(kind in n for n in names), names
            assert any("free_scan" in n for n in names) == (nrows > 409600), (nrows, names)


def weight_gradient(h):
    """One launch for few rows, the more the larger dW is, while its workgroups fit the chip at once; two beyond."""
    x = vp(h.data)
    for K, F, most in ((16, 16, 2400), (64, 16, 2400), (64, 64, 1700), (128, 64, 1700), (128, 128, 3000), (256, 128, 4096), (256, 256, 2560)):
        for n in (1, most, most + 1):
            st, names = launches(h, lambda: h.lib.hgnn_linear_wgrad(i64(n), K, F, x, i64(K), x, i64(F), x, i64(F), x, ctypes.c_size_t(1 << 30), vp(A)))
            assert st == 0 and len(names) == (1 if n <= most else 2), (n, K, F, names)


def shared_columns(h):
    """Waves share a tile's columns up to as many rows as that pays for, by the columns; for 128 of them by the weight, too."""
    x = vp(h.data)
    for K, F, trans, most in ((608, 64, 0, 32768), (264, 128, 1, 32768), (256, 128, 0, 28672), (136, 8, 0, 28672), (128, 128, 0, 20480), (128, 64, 1, 20480),
                              (128, 64, 0, 8191), (128, 40, 0, 8191), (128, 32, 0, 0), (120, 64, 1, 0)):
        for n in (1, most, most + 1):
            st, names = launches(h, lambda: h.lib.hgnn_linear(i64(n), K, F, x, i64(K), x, i64(K if trans else F), trans, x, i64(F), vp(A)))
            assert st == 0 and len(names) == (n > 0), (n, K, F, names)
            if n:
                assert ("linear_split" in names[0]) == (n <= most), (n, K, F, trans, names)


def rounds(h):
    """Rounds of 64 non-zeros where lane groups have longer pieces: not in small graphs, nor where most rows are pieces of whole waves, an eighth of
    which to a lane group is no longer than a round of 32 (of 16 lanes, a quarter)."""
    w = vp(h.data)
    for f, nnz, mean, most in ((64, 4000000, 20, 32), (64, 12000000, 40, 64), (64, 12000000, 128, 64), (64, 12000000, 130, 32), (64, 12000000, 200, 32),
                               (64, 12000000, 256, 32), (64, 12000000, 258, 64), (64, 12000000, 500, 64), (128, 12000000, 200, 64)):
        g = graph(h, nnz // mean, nnz // mean, nnz, True)
        st, names = spmm(h, g, f, h.lib.hgnn_spmm_workspace(nnz // mean, 0, i64(nnz), f), w)
        kernel = [n for n in names if n.startswith("spmm_task_kernel")]
        assert st == 0 and len(kernel) == 1 and f"Li{most}EEE" in kernel[0], (f, nnz, mean, names)


def waves_of_a_projection(h):
    """Workgroups of eight waves for small weights where they take most places, else of four; of larger weights eight, or 16 and more of them than the
    chip holds at once where that leaves nobody with more blocks of rows; all with the same number of blocks, to one."""
    x = vp(h.data)
    for n, K, F, trans, waves, most in (
            (288000, 64, 64, 1, 4, 1024), (144000, 128, 128, 0, 4, 1024), (131072, 128, 128, 0, 8, 512), (288000, 128, 128, 1, 8, 512), (800000, 128, 128, 0, 8, 512),
            (2400000, 128, 128, 0, 8, 1024), (288000, 64, 256, 0, 4, 1024), (400000, 64, 256, 0, 8, 1024), (800000, 64, 256, 1, 8, 1024), (288000, 128, 256, 0, 8, 512),
            (400000, 128, 256, 1, 8, 512), (131072, 64, 608, 1, 8, 512), (288000, 64, 608, 1, 8, 512), (233000, 64, 608, 1, 16, 512), (233000, 608, 64, 0, 8, 512),
            (1200000, 128, 256, 0, 8, 512), (70000, 64, 64, 0, 4, 1024)):
        st, names = launches(h, lambda: h.lib.hgnn_linear(i64(n), K, F, x, i64(K), x, i64(K if trans else F), trans, x, i64(F), vp(A)))
        assert st == 0 and len(names) == 1, (n, K, F, names)
        got, grid = h.fake.fake_last_block() // 64, h.fake.fake_last_grid()
        assert got == waves and grid <= most, (n, K, F, trans, got, grid)
        rows = 16 * (1 if K > 64 else (2 if K > 32 else 4))
        blocks = -(-n // (rows * waves))
        each = -(-blocks // most)
        assert grid == -(-blocks // each), (n, K, F, grid, blocks)


def lanes_of_a_row(h):
    """Softmax and row sums: half of the lanes that the mean row fills only if its registers hold a quarter more than the mean and waves are many, by how
    much more they hold; never without a plan, for the backward and for sums of eight heads by whole waves.  (The runtime's graphs list no rows.)"""
    x = vp(h.data)
    for nrows, mean, H, lanes in ((1000, 20, 4, 16), (8000, 20, 4, 16), (20000, 20, 4, 8), (300000, 10, 4, 4), (2000, 6, 8, 8), (25000, 6, 8, 8), (60000, 6, 8, 8),
                                  (130000, 6, 8, 4), (1000, 40, 4, 32), (10000, 40, 4, 16), (30000, 50, 4, 32), (31000, 50, 4, 16), (100000, 50, 1, 8), (130000, 50, 1, 4),
                                  (200000, 28, 8, 32), (3000, 70, 4, 64), (5000, 70, 4, 32), (300000, 14, 1, 4), (60000, 100, 8, 64)):
        g = graph(h, nrows, nrows, nrows * mean)
        p = vp()
        assert h.lib.hgnn_plan_create(ctypes.byref(g), 256, 64, 8, 1, ctypes.byref(p), vp(A)) == 0
        full = 4
        while full < 64 and full < mean * H / 8:
            full *= 2
        for plan in (p, None):
            for what, args in (("Li0", (x, x)), ("Li1", (x, x, None, ctypes.c_float(0.2), x)), ("Li2", (x, x))):
                f = {"Li0": h.lib.hgnn_edge_softmax, "Li1": h.lib.hgnn_edge_softmax_bwd, "Li2": h.lib.hgnn_edge_rowsum}[what]
                st, names = launches(h, lambda: f(ctypes.byref(g), plan, H, *args, vp(A)))
                want = lanes if plan and what != "Li1" and not (what == "Li2" and H == 8 and full == 64) else full
                kernel = [n for n in names if "edge_rows_kernel" in n]
                assert st == 0 and len(kernel) == 1 and f"I{what}ELi{want}ELi{H}E" in kernel[0], (nrows, mean, H, what, plan, want, names)
        h.lib.hgnn_plan_destroy(p)


SCENARIOS = [lanes_of_a_row, waves_of_a_projection, smaller_workspaces, static_form, narrow_features, column_ranges, room_for_column_ranges, many_windows, weight_gradient, shared_columns, rounds]


@pytest.mark.parametrize("name", [s.__name__ for s in SCENARIOS])
def test_choice_of_kernels(hgnn, fake, name):  # noqa: F811
    r = subprocess.run([sys.executable, os.path.abspath(__file__), fake, LIB, name], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    host = Host(sys.argv[1], sys.argv[2])
    host.lib.hgnn_spmm_workspace.restype = ctypes.c_size_t
    host.lib.hgnn_spmm_static_limit.restype = ctypes.c_size_t
    {s.__name__: s for s in SCENARIOS}[sys.argv[3]](host)
    print("ok")
