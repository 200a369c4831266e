"""Long rows cut at the borders of column ranges (plans of more than 4 Mi non-zeros over a table beyond four L2s): row lengths around
the segment size, rows inside one range, rows that touch only the columns at the borders, empty ranges, every walk that takes them."""
import time

import numpy as np
import pytest
import torch

import oracle
from parity import compare, down, f16, up

pytestmark = pytest.mark.gpu

V, NCOLS, S, MAX_F = 30000, 1100003, 64, 288  # tables of 17.6 MB and more
# 50021 rows, 130003 columns, segments of 36: at 64 features 16.6 MB to gather from in attention and dot products and 6.4 in their backward,
# where a plan for MAX_F has column ranges, which those calls take, and one for 64 has none
WIDE = (50021, 130003, 36, 60, 120)


def make(V, NCOLS, S, least, most):
    r = np.random.default_rng(7)
    width = -(-NCOLS // 8)
    deg = r.integers(least, most, size=V)
    deg[r.permutation(V)[:3000]] = r.integers(0, 70, size=3000)
    lens = (0, 1, S - 1, S, S + 1, S + 2, 2 * S, 8 * S - 1, 8 * S, 8 * S + 1, 2047, 4097, 9000)
    deg[:len(lens)] = lens
    deg[-len(lens):] = lens
    col = [np.sort(r.integers(0, NCOLS, size=d)) for d in deg]
    borders = np.array([b for x in range(1, 8) for b in (x * width - 1, x * width)])
    special = [np.zeros(300), np.full(300, NCOLS - 1), r.integers(0, width, size=700), r.integers(3 * width, 4 * width, size=1000),
               np.tile(borders, 20), np.concatenate([np.zeros(100), np.full(1, NCOLS - 1)]), np.full(2 * S + 1, width)]
    for i, c in enumerate(special):
        deg[50 + i] = c.size
        col[50 + i] = np.sort(c)
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    col = np.concatenate(col).astype(np.int32)
    assert 4 << 20 < col.size < 8 << 20
    return rowptr, col


@pytest.fixture(scope="module")
def graph():
    return make(V, NCOLS, S, 110, 200)


@pytest.fixture(scope="module")
def wide():
    return make(*WIDE)


@pytest.mark.parametrize("F,H", [(8, 1), (42, 1), (32, 4), (24, 3)])
@pytest.mark.parametrize("what", ["plain", "w", "map", "scaled"])
def test_spmm(hgnn, dev, graph, F, H, what):
    print(f"ranges F={F} H={H} {what}", flush=True)
    r = np.random.default_rng(F + H)
    rowptr, col = graph
    pitch = (F + 7) // 8 * 8
    w = None if what == "plain" else f16(r.standard_normal((col.size, H)))
    H = 1 if w is None else H
    g, ncols, eid = hgnn.Csr(up(rowptr, dev), up(col, dev), ncols=NCOLS), NCOLS, None
    if what == "map":  # the long rows again, now with a map
        t = hgnn.hgnn_transpose(g)
        g = hgnn.hgnn_transpose(hgnn.Csr(t.rowptr, t.col, ncols=V))
        eid = down(g.eid)
    Xh = np.zeros((ncols, pitch), dtype=np.float16)
    Xh[:, :F] = f16(r.standard_normal((ncols, F)))
    p = hgnn.hgnn_plan_create(g, S, MAX_F, H, col_blocks=1)
    Y = torch.full((V, pitch), 3.0, dtype=torch.float16, device=dev)
    wd = None if w is None else up(w, dev)
    if what == "scaled":
        cs = r.uniform(0.5, 2.0, size=ncols).astype(np.float32)
        hgnn.hgnn_spmm_discretized_fused(p, g, wd, H, up(Xh, dev), Y, op=hgnn.HGNN_MEAN, col_scale=up(cs, dev), F=F)
        ref, sabs = scaled(rowptr, col, Xh[:, :F], w, cs, H)
    else:
        hgnn.hgnn_spmm_discretized(p, g, wd, H, up(Xh, dev), Y, F=F)
        ref, sabs = oracle.spmm(rowptr, col, np.ascontiguousarray(Xh[:, :F]), w=w, H=H, want_sabs=True, **({} if eid is None else {"eid": eid}))
    compare("ranges", np.ascontiguousarray(down(Y)[:, :F]), ref, sabs)
    hgnn.hgnn_plan_destroy(p)


@pytest.mark.parametrize("S", [64, 1000])
def test_table_beyond_the_last_level_cache(hgnn, dev, graph, S):
    """Most rows, or a few, have pieces at column ranges: more waves in flight, or fewer."""
    print(f"ranges, 282 MB table, S={S}", flush=True)
    rowptr, col = graph
    F = 128
    X = torch.randn((NCOLS, F), generator=torch.Generator(device=dev).manual_seed(S), device=dev).half()
    w = f16(np.random.default_rng(S).standard_normal((col.size, 1)))
    g = hgnn.Csr(up(rowptr, dev), up(col, dev), ncols=NCOLS)
    p = hgnn.hgnn_plan_create(g, S, F, 1, col_blocks=1)
    Y = torch.full((V, F), 3.0, dtype=torch.float16, device=dev)
    hgnn.hgnn_spmm_discretized(p, g, up(w, dev), 1, X, Y)
    ref, sabs = oracle.spmm(rowptr, col, down(X), w=w, H=1, want_sabs=True)
    compare("large table", down(Y), ref, sabs)
    hgnn.hgnn_plan_destroy(p)


def scaled(rowptr, col, X, w, cs, H):
    """Mean of w * cs[col] * X[col], and the same over magnitudes, in float64."""
    F = X.shape[1]
    out = []
    for f in (lambda a: a, np.abs):
        t = f(w.astype(np.float64)).repeat(F // H, axis=1) * (f(X.astype(np.float64)) * cs[:, None].astype(np.float64))[col]
        y = np.add.reduceat(np.concatenate([t, np.zeros((1, F))]), rowptr[:-1], axis=0)
        deg = np.diff(rowptr)
        y[deg == 0] = 0
        out.append(y / np.maximum(deg, 1)[:, None])
    return out


@pytest.mark.parametrize("H,D", [(1, 64), (4, 16), (8, 8)])
def test_attention(hgnn, dev, wide, H, D):
    """Saving forward and its backward against the oracle (forward) and the walk over rows in one range (backward)."""
    print(f"ranges attention H={H} D={D}", flush=True)
    rowptr, col = wide
    V, NCOLS, S = WIDE[:3]
    F = H * D
    r = np.random.default_rng(H)
    U, X, dO = (f16(r.standard_normal((n, F))) for n in (V, NCOLS, V))
    a_l, a_r = f16(0.2 * r.standard_normal(F)), f16(0.2 * r.standard_normal(F))
    ref, ref_lse, sabs = oracle.gat_forward(rowptr, col, U, X, a_l, a_r, H, slope=0.2)
    g = hgnn.Csr(up(rowptr, dev), up(col, dev), ncols=NCOLS)
    gt = hgnn.hgnn_transpose(g)
    Ud, Xd, dOd, al, ar = up(U, dev), up(X, dev), up(dO, dev), up(a_l, dev), up(a_r, dev)
    got = []
    for max_f in (F, MAX_F):
        p, pt = (hgnn.hgnn_plan_create(x, S, max_f, H, col_blocks=1) for x in (g, gt))
        half = lambda *n: torch.full(n, 7.0, dtype=torch.float16, device=dev)
        f32 = lambda *n: torch.full(n, 7.0, dtype=torch.float32, device=dev)
        out, outm, lse, csum = half(V, F), half(V, F), f32(V, H), f32(V, H)
        hgnn.hgnn_gat_forward_fused_save(g, p, H, D, Ud, Xd, al, ar, out, lse, outm, csum)
        out0, lse0 = half(V, F), f32(V, H)
        hgnn.hgnn_gat_forward_fused(g, p, H, D, Ud, Xd, al, ar, out0, lse0)
        assert torch.equal(out, out0) and torch.equal(lse, lse0)
        dV, d_el, d_er = half(NCOLS, F), half(V, H), half(NCOLS, H)
        hgnn.hgnn_gat_backward_fused_saved(g, p, gt, pt, H, D, Ud, Xd, al, ar, out, lse, outm, csum, dOd, dV, d_el, d_er)
        dot = torch.full((col.size, H), 7.0, dtype=torch.float16, device=dev)
        hgnn.hgnn_sddmm(g, p, hgnn.HGNN_SDDMM_DOT, H, D, dOd, Xd, dot)
        sums = half(NCOLS, H)
        hgnn.hgnn_edge_rowsum(gt, pt, H, dot, sums)
        got.append([down(t) for t in (out, outm, lse, csum, dV, d_el, d_er, dot, sums)])
        hgnn.hgnn_plan_destroy(p)
        hgnn.hgnn_plan_destroy(pt)
    compare("out", got[1][0], ref, sabs)
    deg = np.diff(rowptr)
    assert np.abs(got[1][2][deg > 0] - ref_lse[deg > 0]).max() <= 2e-3 + 1e-3 * np.abs(ref_lse).max()
    for name, a, b in zip(("out", "outm", "lse", "csum", "dV", "d_el", "d_er", "dot", "sums"), got[0], got[1]):
        if name == "dot":  # the same products in the same order
            assert np.array_equal(a.view(np.uint16), b.view(np.uint16))
            continue
        a, b = a.astype(np.float64), b.astype(np.float64)
        # two results of sums that are rounded to fp16 up to three times each; 2^-11 relative to the terms of a cancelling sum
        assert np.linalg.norm(a - b) <= 4e-3 * np.linalg.norm(a), (name, np.linalg.norm(a - b) / np.linalg.norm(a))


# without a plan: beyond 4 Mi non-zeros and 34 MB of table, rows below 128 non-zeros on average (no column passes)
@pytest.mark.parametrize("F,H,ncols,mapped,has_w", [(32, 1, 600011, True, True), (32, 4, 600011, True, True), (42, 1, 500009, True, True),
                                                    (128, 1, 600011, False, True), (128, 1, 600011, False, False)])
def test_without_a_plan(hgnn, dev, F, H, ncols, mapped, has_w):
    print(f"ranges without a plan F={F} H={H} ncols={ncols} mapped={mapped} values={has_w}", flush=True)
    r = np.random.default_rng(F + H)
    nrows, width = 40003, -(-ncols // 8)
    deg = r.integers(60, 160, size=nrows)
    lens = (0, 1, 255, 256, 257, 258, 511, 512, 513, 2047, 2048, 2049, 9000, 30000)
    deg[:len(lens)] = lens
    deg[-len(lens):] = lens
    col = [np.sort(r.integers(0, ncols, size=d)) for d in deg]
    borders = np.array([b for x in range(1, 8) for b in (x * width - 1, x * width)])
    for i, c in enumerate((np.zeros(300), np.full(300, ncols - 1), r.integers(3 * width, 4 * width, size=1000), np.tile(borders, 20))):
        deg[2000 * i + 1500] = c.size
        col[2000 * i + 1500] = np.sort(c)
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    col = np.concatenate(col).astype(np.int32)
    E = col.size
    assert 4 << 20 < E < 128 * nrows
    pitch = (F + 7) // 8 * 8
    X = np.zeros((ncols, pitch), dtype=np.float16)
    X[:, :F] = f16(r.standard_normal((ncols, F)))
    w = f16(r.standard_normal((E, H))) if has_w else None
    eid = r.permutation(E).astype(np.int32) if mapped else None
    g = hgnn.Csr(up(rowptr, dev), up(col, dev), ncols=ncols, eid=None if eid is None else up(eid, dev))
    need, less = hgnn.hgnn_spmm_workspace(nrows, ncols, E, F), hgnn.hgnn_spmm_workspace(nrows, 0, E, F)
    assert need > less > 0
    Xd, wd = up(X, dev), None if w is None else up(w, dev)
    out = []
    for n, fill in ((need, 255), (need, 0), (less, 0)):  # what the workspace holds beforehand does not matter
        ws = torch.full((n,), fill, dtype=torch.uint8, device=dev)
        Y = torch.full((nrows, pitch), 3.0, dtype=torch.float16, device=dev)
        hgnn.hgnn_spmm(g, wd, H, Xd, Y, F=F, workspace=ws)
        out.append(down(Y))
    assert np.array_equal(out[0].view(np.uint16), out[1].view(np.uint16))
    ref, sabs = oracle.spmm(rowptr, col, np.ascontiguousarray(X[:, :F]), w=w, H=H, want_sabs=True, **({} if eid is None else {"eid": eid}))
    for y in (out[0], out[2]):
        compare("without a plan", np.ascontiguousarray(y[:, :F]), ref, sabs)


@pytest.mark.parametrize("spread", [True, False])
@pytest.mark.parametrize("rows,least,most", [(18000, 257, 300), (18000, 257, 480), (70000, 257, 260)])
def test_without_a_plan_many_long_rows(hgnn, dev, rows, least, most, spread):
    """Most non-zeros in rows that are barely long: more of them than there are pieces of 512, and more than take a wave each.  Over all
    columns they have more pieces at column ranges than there is room for, inside one range two each."""
    print(f"ranges without a plan, {rows} rows of {least} to {most}", flush=True)
    F, ncols = 8, 2200003
    r = np.random.default_rng(rows + most)
    deg = np.zeros(3 * rows, dtype=np.int64)
    deg[::3] = r.integers(least, most + 1, size=rows)
    deg[1::3] = r.integers(0, 3, size=rows)
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    E = int(rowptr[-1])
    assert 4 << 20 < E < 128 * deg.size and rows > E // 512 + 1
    row = np.repeat(np.arange(deg.size), deg)
    c = r.integers(0, ncols, size=E)
    if not spread:
        width = -(-ncols // 8)
        c = np.minimum(c % width + row % 8 * width, ncols - 1)
    col = (np.sort(row * ncols + c) - row * ncols).astype(np.int32)
    assert (8 * rows > E // 128) and (2 * rows <= E // 128)
    Xh, w, eid = f16(r.standard_normal((ncols, F))), f16(r.standard_normal((E, 1))), r.permutation(E).astype(np.int32)
    n = hgnn.hgnn_spmm_workspace(deg.size, ncols, E, F)
    assert n > hgnn.hgnn_spmm_workspace(deg.size, 0, E, F)
    Y = torch.full((deg.size, F), 3.0, dtype=torch.float16, device=dev)
    hgnn.hgnn_spmm(hgnn.Csr(up(rowptr, dev), up(col, dev), ncols=ncols, eid=up(eid, dev)), up(w, dev), 1, up(Xh, dev), Y, F=F,
                   workspace=torch.full((n,), 255, dtype=torch.uint8, device=dev))
    ref, sabs = oracle.spmm(rowptr, col, Xh, w=w, H=1, want_sabs=True, eid=eid)
    compare("many long rows", down(Y), ref, sabs)


@pytest.mark.parametrize("spare", [0, -1])
def test_without_a_plan_room(hgnn, dev, spare):
    """Exactly as many pieces at column ranges as there is room for, and one more than that."""
    print(f"ranges without a plan, {spare} pieces to spare", flush=True)
    F, ncols, n = 8, 2200003, 5000
    width = -(-ncols // 8)
    r = np.random.default_rng(3)
    E = 1024 * n + spare
    deg = np.concatenate([np.full(n, 304), np.full((E - 304 * n) // 100, 100), [(E - 304 * n) % 100]])
    deg = deg[r.permutation(deg.size)]
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    assert rowptr[-1] == E and E // 128 == 8 * n + spare and E < 128 * deg.size
    row = np.repeat(np.arange(deg.size), deg)
    k = np.arange(E) - rowptr[:-1].astype(np.int64)[row]
    c = np.where(deg[row] == 304, np.minimum(k // 38 * width + r.integers(0, width, size=E), ncols - 1), r.integers(0, ncols, size=E))
    col = (np.sort(row * ncols + c) - row * ncols).astype(np.int32)  # 38 non-zeros in every range
    Xh, w, eid = f16(r.standard_normal((ncols, F))), f16(r.standard_normal((E, 1))), r.permutation(E).astype(np.int32)
    Y = torch.full((deg.size, F), 3.0, dtype=torch.float16, device=dev)
    hgnn.hgnn_spmm(hgnn.Csr(up(rowptr, dev), up(col, dev), ncols=ncols, eid=up(eid, dev)), up(w, dev), 1, up(Xh, dev), Y, F=F,
                   workspace=torch.full((hgnn.hgnn_spmm_workspace(deg.size, ncols, E, F),), 255, dtype=torch.uint8, device=dev))
    ref, sabs = oracle.spmm(rowptr, col, Xh, w=w, H=1, want_sabs=True, eid=eid)
    compare("room", down(Y), ref, sabs)


@pytest.mark.parametrize("n", [409600, 409601])
def test_without_a_plan_many_windows(hgnn, dev, n):
    """400 windows of rows add up their counts, more have them scanned; in pieces and with column ranges."""
    print(f"ranges without a plan, {n} rows", flush=True)
    F, ncols = 8, 2200003
    r = np.random.default_rng(n)
    deg = r.integers(0, 20, size=n)
    deg[r.permutation(n)[:1000]] = r.integers(200, 1200, size=1000)
    deg[-3:] = (0, 700, 2000)
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    E = int(rowptr[-1])
    assert E > 4 << 20
    row = np.repeat(np.arange(n), deg)
    col = (np.sort(row * ncols + r.integers(0, ncols, size=E)) - row * ncols).astype(np.int32)
    Xh, w, eid = f16(r.standard_normal((ncols, F))), f16(r.standard_normal((E, 1))), r.permutation(E).astype(np.int32)
    g = hgnn.Csr(up(rowptr, dev), up(col, dev), ncols=ncols, eid=up(eid, dev))
    ref, sabs = oracle.spmm(rowptr, col, Xh, w=w, H=1, want_sabs=True, eid=eid)
    for cols in (1, ncols):
        Y = torch.full((n, F), 3.0, dtype=torch.float16, device=dev)
        hgnn.hgnn_spmm(g, up(w, dev), 1, up(Xh, dev), Y, F=F,
                       workspace=torch.full((hgnn.hgnn_spmm_workspace(n, cols, E, F),), 255, dtype=torch.uint8, device=dev))
        compare("many windows", down(Y), ref, sabs)


def test_without_a_plan_any_order(hgnn, dev):
    """Rows whose columns do not ascend: still every non-zero once."""
    print("ranges without a plan, columns in any order", flush=True)
    F, ncols, n = 8, 2200003, 60000
    r = np.random.default_rng(4)
    deg = r.integers(0, 120, size=n)
    deg[:2000] = r.integers(257, 3000, size=2000)
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    E = int(rowptr[-1])
    assert 4 << 20 < E < 128 * n
    col = r.integers(0, ncols, size=E).astype(np.int32)
    Xh, w, eid = f16(r.standard_normal((ncols, F))), f16(r.standard_normal((E, 1))), r.permutation(E).astype(np.int32)
    Y = torch.full((n, F), 3.0, dtype=torch.float16, device=dev)
    hgnn.hgnn_spmm(hgnn.Csr(up(rowptr, dev), up(col, dev), ncols=ncols, eid=up(eid, dev)), up(w, dev), 1, up(Xh, dev), Y, F=F,
                   workspace=torch.full((hgnn.hgnn_spmm_workspace(n, ncols, E, F),), 255, dtype=torch.uint8, device=dev))
    ref, sabs = oracle.spmm(rowptr, col, Xh, w=w, H=1, want_sabs=True, eid=eid)
    compare("any order", down(Y), ref, sabs)


@pytest.mark.parametrize("S", [4, 64, 256])
def test_a_very_long_row(hgnn, dev, S):
    """Half of all non-zeros in one row, most of them in one column range: its many pieces are written by a wave, so a plan with column
    ranges takes about as long as one without (a lane alone took ten times as long at S = 4, twice at 256)."""
    print(f"ranges, very long row S={S}", flush=True)
    n, E, F = 200000, 6000000, 64
    r = np.random.default_rng(S)
    deg = np.bincount(r.integers(0, n, size=E // 2), minlength=n)
    deg[77] += E - deg.sum()
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    row = np.repeat(np.arange(n), deg)
    c = r.integers(0, n, size=E)
    hub = np.arange(rowptr[77], rowptr[78])
    c[hub[: hub.size * 3 // 4]] %= 1000
    col = (np.sort(row * n + c) - row * n).astype(np.int32)
    g = hgnn.Csr(up(rowptr, dev), up(col, dev), ncols=n)

    def plan_time(max_f):
        best = 1e9
        for _ in range(5):
            t = time.perf_counter()
            hgnn.hgnn_plan_destroy(hgnn.hgnn_plan_create(g, S, max_f, 1, col_blocks=1))
            best = min(best, time.perf_counter() - t)
        return best

    narrow, wide = plan_time(8), plan_time(F)
    assert wide <= 3 * narrow + 100e-6, (narrow, wide)
    w, Xh = f16(r.standard_normal((E, 1))), f16(r.standard_normal((n, F)))
    ref, sabs = oracle.spmm(rowptr, col, Xh, w=w, H=1, want_sabs=True)
    Y = torch.full((n, F), 3.0, dtype=torch.float16, device=dev)
    p = hgnn.hgnn_plan_create(g, S, F, 1, col_blocks=1)
    hgnn.hgnn_spmm_discretized(p, g, up(w, dev), 1, up(Xh, dev), Y)
    compare("very long row", down(Y), ref, sabs)
    hgnn.hgnn_plan_destroy(p)
    ident = hgnn.Csr(g.rowptr, g.col, ncols=n, eid=torch.arange(E, dtype=torch.int32, device=dev))
    X2 = np.concatenate([Xh, Xh], axis=1)  # beyond eight L2s
    Y2 = torch.full((n, 2 * F), 3.0, dtype=torch.float16, device=dev)
    hgnn.hgnn_spmm(ident, up(w, dev), 1, up(X2, dev), Y2,
                   workspace=torch.full((hgnn.hgnn_spmm_workspace(n, n, E, 2 * F),), 255, dtype=torch.uint8, device=dev))
    compare("very long row without a plan", np.ascontiguousarray(down(Y2)[:, F:]), ref, sabs)


@pytest.mark.parametrize("S,most", [(32, 180), (64, 60)])
def test_memory_of_short_segments(hgnn, dev, S, most):
    """Rows of about 50 non-zeros in segments of 32 have two pieces, in eight column ranges they would have eight: 417 MB of staging."""
    print(f"ranges, memory S={S}", flush=True)
    n, E, F = 100000, 5000000, 128
    r = np.random.default_rng(S)
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(r.integers(0, n, size=E), minlength=n))]).astype(np.int32)
    row = np.repeat(np.arange(n), np.diff(rowptr))
    col = (np.sort(row * n + r.integers(0, n, size=E)) - row * n).astype(np.int32)
    g = hgnn.Csr(up(rowptr, dev), up(col, dev), ncols=n)
    hgnn.hgnn_release_cached_memory()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    p = hgnn.hgnn_plan_create(g, S, F, 1, col_blocks=1)
    used = free - torch.cuda.mem_get_info()[0]
    hgnn.hgnn_plan_destroy(p)
    hgnn.hgnn_release_cached_memory()
    assert used < most << 20, used


def test_calls_that_keep_ordinary_pieces(hgnn, dev, wide):
    """Calls over a narrow table walk the same pieces whatever the plan was made for; only the row sums gather from something else."""
    print("ranges, narrow calls", flush=True)
    rowptr, col = wide
    V, NCOLS, S = WIDE[:3]
    F, r = 8, np.random.default_rng(1)
    g = hgnn.Csr(up(rowptr, dev), up(col, dev), ncols=NCOLS)
    t = hgnn.hgnn_transpose(g)
    gm = hgnn.hgnn_transpose(hgnn.Csr(t.rowptr, t.col, ncols=V))
    X, U = up(f16(r.standard_normal((NCOLS, F))), dev), up(f16(r.standard_normal((V, F))), dev)
    w = up(f16(r.standard_normal((col.size, 1))), dev)
    a_l, a_r = (up(f16(r.standard_normal(F)), dev) for _ in range(2))
    got = []
    for max_f in (F, MAX_F):
        p, pm = (hgnn.hgnn_plan_create(x, S, max_f, 1, col_blocks=1) for x in (g, gm))
        half = lambda *n: torch.full(n, 3.0, dtype=torch.float16, device=dev)
        Y, Yw, Ym, out, lse, dot = half(V, F), half(V, F), half(V, F), half(V, F), half(V, 1).float(), half(col.size, 1)
        hgnn.hgnn_spmm_discretized(p, g, None, 1, X, Y)
        hgnn.hgnn_spmm_discretized(p, g, w, 1, X, Yw)
        hgnn.hgnn_spmm_discretized(pm, gm, w, 1, X, Ym)
        hgnn.hgnn_gat_forward_fused(g, p, 1, F, U, X, a_l, a_r, out, lse)
        hgnn.hgnn_sddmm(g, p, hgnn.HGNN_SDDMM_DOT, 1, F, U, X, dot)
        got.append([down(x).view(np.uint8) for x in (Y, Yw, Ym, out, lse, dot)])
        for x in (p, pm):
            hgnn.hgnn_plan_destroy(x)
    for a, b in zip(*got):
        assert np.array_equal(a, b)


def test_atomic_additions(hgnn, dev, graph):
    """The variant that adds every piece to the row in fp16 rounds as often as there are segments, whatever the plan was made for: the
    expected square of the error is a sum over the additions, so twice the additions would show as 1.4 times the error."""
    print("ranges, atomic additions", flush=True)
    rowptr, col = graph
    F, r = 8, np.random.default_rng(2)
    g = hgnn.Csr(up(rowptr, dev), up(col, dev), ncols=NCOLS)
    Xh = f16(r.standard_normal((NCOLS, F)))
    ref = oracle.spmm(rowptr, col, Xh)
    deg = np.diff(rowptr)
    rows = (deg > 2 * S) & (deg <= 3 * S)  # of three segments' pieces; with column ranges of eight
    X, err = up(Xh, dev), {}
    n = int(rowptr[V // 2])  # half of the graph has no column ranges
    assert n < 4 << 20
    for name, h in (("half", hgnn.Csr(up(rowptr[: V // 2 + 1].copy(), dev), up(col[:n].copy(), dev), ncols=NCOLS)), ("all", g)):
        m = h.rowptr.numel() - 1
        Y = torch.full((m, F), 3.0, dtype=torch.float16, device=dev)
        p = hgnn.hgnn_plan_create(h, S, MAX_F, 1, col_blocks=1)
        hgnn.hgnn_spmm_discretized_variant(p, h, None, 1, X, Y, variant=hgnn.HGNN_EDGE_SEGMENTS_ATOMIC)
        k = rows[: V // 2]
        d = down(Y)[: V // 2][k].astype(np.float64) - ref[: V // 2][k]
        err[name] = np.linalg.norm(d) / np.linalg.norm(ref[: V // 2][k])
        hgnn.hgnn_plan_destroy(p)
    assert err["all"] <= 1.1 * err["half"], err
