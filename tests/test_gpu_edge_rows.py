"""The row passes over edge tensors at the borders of their vectors, teams and chunks: rows of every length around them, beginning at every
offset inside a vector, with neighbours whose values must not leak."""
import numpy as np
import pytest
import torch

import oracle
from parity import compare, down, f16, up

pytestmark = pytest.mark.gpu

# around a vector of 8 elements, a team's and a wave's registers, the listed rows (32), the chunks (2048)
EDGES = (1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1025, 2047, 2048, 2049, 2056,
         4096, 4097)


def lengths(short_rows, seed):
    r = np.random.default_rng(seed)
    some = np.concatenate([np.array([n, k], np.int64) for k in range(8) for n in EDGES])  # each from eight offsets on
    return np.concatenate([some, r.integers(0, 6, short_rows)])


@pytest.mark.parametrize("H", [1, 2, 4, 8])
@pytest.mark.parametrize("short_rows", [0, 1500, 60000])
def test_row_passes_at_borders(hgnn, dev, H, short_rows):
    print(f"edge rows H={H} short={short_rows}", flush=True)
    deg = lengths(short_rows, H)
    V = deg.size
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    E = int(rowptr[-1])
    r = np.random.default_rng(H)
    col = np.zeros(E, np.int32)  # (one column: the passes only read the offsets)
    rows = np.repeat(np.arange(V), deg)
    e16, da16, t16 = f16(3 * r.standard_normal((E, H))), f16(r.standard_normal((E, H))), f16(r.standard_normal((E, H)))
    lone = np.flatnonzero(deg == 1)[::3]  # rows of one non-zero between others: infinite there, and nowhere else
    at = rowptr[lone]
    t16[at] = np.float16(np.inf)
    da_inf = da16.copy()
    da_inf[at] = np.float16(np.inf)
    e16[rowptr[np.flatnonzero(deg > 4)], 0] = np.float16(-np.inf)  # weight zero
    others = np.ones(V, bool)
    others[lone] = False
    g = hgnn.Csr(up(rowptr, dev), up(col, dev), ncols=1)
    p = hgnn.hgnn_plan_create(g, 256, 64, 8)
    ref = oracle.edge_softmax(rowptr, e16.astype(np.float64))
    t64 = np.where(np.isfinite(t16), t16, 0).astype(np.float64)
    for plan in (p, None):
        alpha = torch.full((E, H), -1.0, dtype=torch.float16, device=dev)
        hgnn.hgnn_edge_softmax(g, plan, H, up(e16, dev), alpha)
        a16 = down(alpha).copy()
        # exp and the division in fp32, one rounding to fp16: half an ulp, and 2^-20 for what precedes it
        assert np.all(np.abs(a16.astype(np.float64) - ref) <= ref * (2.0 ** -11 + 2.0 ** -18) + 2.0 ** -24)
        de = torch.full((E, H), 9.0, dtype=torch.float16, device=dev)
        for e in (None, e16):
            hgnn.hgnn_edge_softmax_bwd(g, plan, H, alpha, up(da_inf, dev), de, e=None if e is None else up(e, dev), neg_slope=0.2)
            a64, d64 = a16.astype(np.float64), da16.astype(np.float64)
            want = oracle.edge_softmax_bwd(rowptr, a64, d64, e=None if e is None else e.astype(np.float64))
            mag = np.zeros((V, H))
            np.add.at(mag, rows, np.abs(a64 * d64))
            keep = others[rows]
            compare("de", down(de)[keep], want[keep], (a64 * (np.abs(d64) + mag[rows]) + 2.0 ** -14)[keep])
        out = torch.full((V, H), 9.0, dtype=torch.float16, device=dev)
        hgnn.hgnn_edge_rowsum(g, plan, H, up(t16, dev), out)
        got = down(out)
        assert np.all(np.isinf(got[lone]))
        compare("row sums", got[others], oracle.edge_rowsum(rowptr, t64)[others], oracle.edge_rowsum(rowptr, np.abs(t64))[others])
    hgnn.hgnn_plan_destroy(p)


def median_ms(call):
    ms = []
    for _ in range(9):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            call()
        b.record()
        b.synchronize()
        ms.append(a.elapsed_time(b) / 5)
    return sorted(ms)[4]


def csr_of(hgnn, dev, deg):
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    return hgnn.Csr(up(rowptr, dev), torch.zeros(int(rowptr[-1]), dtype=torch.int32, device=dev), ncols=1)


# the last rows of a stretch that is dealt out to workgroups, and few of the next
@pytest.mark.parametrize("V", [1, 17, 1023, 1025, 4095, 4096, 4097, 12290])
@pytest.mark.parametrize("H", [1, 4])
def test_rows_dealt_out(hgnn, dev, V, H):
    print(f"dealt rows V={V} H={H}", flush=True)
    r = np.random.default_rng(V)
    deg = r.choice([0, 3, 33, 40, 70, 130, 600], V)
    deg[-1] = 517
    E, rows = int(deg.sum()), np.repeat(np.arange(V), deg)
    g = csr_of(hgnn, dev, deg)
    rowptr = np.concatenate([[0], np.cumsum(deg)])
    e16, da16 = f16(3 * r.standard_normal((E, H))), f16(r.standard_normal((E, H)))
    ref = oracle.edge_softmax(rowptr.astype(np.int32), e16.astype(np.float64))
    for plan in (None, hgnn.hgnn_plan_create(g, 256, 64, 8)):
        alpha, de = (torch.full((E, H), 9.0, dtype=torch.float16, device=dev) for _ in range(2))
        out = torch.full((V, H), 9.0, dtype=torch.float16, device=dev)
        hgnn.hgnn_edge_softmax(g, plan, H, up(e16, dev), alpha)
        a64, d64 = down(alpha).astype(np.float64), da16.astype(np.float64)
        assert np.all(np.abs(a64 - ref) <= ref * (2.0 ** -11 + 2.0 ** -18) + 2.0 ** -24)
        hgnn.hgnn_edge_softmax_bwd(g, plan, H, alpha, up(da16, dev), de, e=up(e16, dev), neg_slope=0.2)
        mag = np.zeros((V, H))
        np.add.at(mag, rows, np.abs(a64 * d64))
        compare("de", down(de), oracle.edge_softmax_bwd(rowptr.astype(np.int32), a64, d64, e=e16.astype(np.float64)),
                a64 * (np.abs(d64) + mag[rows]) + 2.0 ** -14)
        hgnn.hgnn_edge_rowsum(g, plan, H, up(da16, dev), out)
        compare("row sums", down(out), oracle.edge_rowsum(rowptr.astype(np.int32), d64), oracle.edge_rowsum(rowptr.astype(np.int32), np.abs(d64)))


# mean lengths at which half of the lanes take a row, or just not any more; rows beyond what those hold at once, from a whole wave's lanes on
@pytest.mark.parametrize("mean,H", [(5, 8), (12, 8), (13, 8), (10, 4), (20, 2), (25, 4), (26, 4), (35, 8), (48, 1), (100, 4), (400, 1), (420, 1)])
def test_half_of_the_lanes(hgnn, dev, mean, H):
    print(f"half of the lanes mean={mean} H={H}", flush=True)
    V = 3000
    r = np.random.default_rng(mean + H)
    deg = r.integers(0, mean, V)
    deg[::7] = r.integers(mean, 2 * mean, deg[::7].size)
    deg[5::100] = 3 * mean + r.integers(0, 40, deg[5::100].size)
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    E = int(rowptr[-1])
    e16 = f16(3 * r.standard_normal((E, H)))
    g = csr_of(hgnn, dev, deg)
    p = hgnn.hgnn_plan_create(g, 256, 64, 8)
    alpha, out = (torch.full((n, H), 9.0, dtype=torch.float16, device=dev) for n in (E, V))
    hgnn.hgnn_edge_softmax(g, p, H, up(e16, dev), alpha)
    ref = oracle.edge_softmax(rowptr, e16.astype(np.float64))
    assert np.all(np.abs(down(alpha).astype(np.float64) - ref) <= ref * (2.0 ** -11 + 2.0 ** -18) + 2.0 ** -24)
    hgnn.hgnn_edge_rowsum(g, p, H, up(e16, dev), out)
    e64 = e16.astype(np.float64)
    compare("row sums", down(out), oracle.edge_rowsum(rowptr, e64), oracle.edge_rowsum(rowptr, np.abs(e64)))
    hgnn.hgnn_plan_destroy(p)


# so many rows that half of the lanes take them (16, 60 or 96 waves of all lanes a compute unit), or just not; some rows at and beyond what the half hold
@pytest.mark.parametrize("V,mean,H,alike", [(17000, 20, 4, True), (9000, 20, 8, True), (8100, 20, 8, True), (33000, 40, 1, True), (4200, 140, 2, True), (124000, 50, 1, True),
                                            (200000, 6, 8, False), (60000, 6, 8, True), (200000, 6, 4, False)])
def test_half_of_the_lanes_of_many_rows(hgnn, dev, V, mean, H, alike):
    print(f"half of the lanes, many rows V={V} mean={mean} H={H} alike={alike}", flush=True)
    r = np.random.default_rng(V + mean + H)
    deg = r.integers(mean - 1, mean + 2, V) if alike else r.integers(0, 2 * mean, V)
    held = 1
    while held < mean:
        held *= 2
    for k, d in enumerate((held - 1, held, held + 1, 2 * held, 2 * held + 1, 33, 300, 0)):
        deg[11 + k::V // 9] = d
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    E = int(rowptr[-1])
    e16 = f16(3 * r.standard_normal((E, H)))
    g = csr_of(hgnn, dev, deg)
    p = hgnn.hgnn_plan_create(g, 256, 64, 8)
    alpha, out = (torch.full((n, H), 9.0, dtype=torch.float16, device=dev) for n in (E, V))
    hgnn.hgnn_edge_softmax(g, p, H, up(e16, dev), alpha)
    e64 = e16.astype(np.float64)
    ref = oracle.edge_softmax(rowptr, e64)
    assert np.all(np.abs(down(alpha).astype(np.float64) - ref) <= ref * (2.0 ** -11 + 2.0 ** -18) + 2.0 ** -24)
    hgnn.hgnn_edge_rowsum(g, p, H, up(e16, dev), out)
    compare("row sums", down(out), oracle.edge_rowsum(rowptr, e64), oracle.edge_rowsum(rowptr, np.abs(e64)))
    hgnn.hgnn_plan_destroy(p)


@pytest.mark.parametrize("H,planned", [(1, False), (4, False), (8, False), (1, True), (2, True)])
def test_rows_in_order_of_their_lengths(hgnn, dev, H, planned):
    """Vertices in the order of their degrees, longest rows side by side, take no longer than the same rows in any order: sixteen of the longest in
    a workgroup took 2.8 to 3.6 times as long without a plan, 1.7 to 2.2 times with one."""
    deg = np.minimum(8000 if not planned else 2000, 38000 * (np.arange(30000) + 1.0) ** -0.8).astype(np.int64) + 1
    E = int(deg.sum())
    e = torch.randn((E, H), dtype=torch.float16, device=dev)
    out = torch.empty_like(e)
    ms = []
    for order in (deg, np.random.default_rng(1).permutation(deg)):
        g = csr_of(hgnn, dev, order)
        p = hgnn.hgnn_plan_create(g, 256, 64, 8) if planned else None
        ms.append(median_ms(lambda: (hgnn.hgnn_edge_softmax(g, p, H, e, out), hgnn.hgnn_edge_softmax_bwd(g, p, H, e, e, out, e=e))))
    print(f"in order H={H} plan={planned}: {1e3 * ms[0]:.0f} us, in any {1e3 * ms[1]:.0f} us", flush=True)
    assert ms[0] < (1.4 if not planned else 1.2) * ms[1]


def test_backward_of_short_rows(hgnn, dev):
    """Rows of four non-zeros: two heads have half the bytes of four.  With every array and the row ends fetched apart they took 1.05 of its time
    (30.6 / 29.2 us), fetched together 0.79 (22.0 / 28.0); the bound is between the two."""
    V, call = 1000000, {}
    g = csr_of(hgnn, dev, np.random.default_rng(2).poisson(4, V))
    p = hgnn.hgnn_plan_create(g, 256, 64, 8)
    for H in (2, 4):
        e = torch.randn((g.nnz, H), dtype=torch.float16, device=dev)
        alpha, out = torch.rand_like(e), torch.empty_like(e)
        call[H] = lambda H=H, e=e, alpha=alpha, out=out: hgnn.hgnn_edge_softmax_bwd(g, p, H, alpha, e, out, e=e)
    tries = [median_ms(call[2]) / median_ms(call[4]) for _ in range(3)]
    hgnn.hgnn_plan_destroy(p)
    print("two heads / four: " + ", ".join(f"{t:.2f}" for t in tries), flush=True)
    assert min(tries) < 0.91


# scores by segments of the edge list: segments below, at and above the 256 non-zeros of one round, ids at every offset inside a
# vector, rows that are empty, longer than a segment or more than a wave to a segment, sides of different tables and sizes
@pytest.mark.parametrize("S", [64, 256, 320, 1000])
@pytest.mark.parametrize("H", [1, 2, 3, 4, 8])
def test_edge_scores_by_segments(hgnn, dev, H, S):
    print(f"scores H={H} S={S}", flush=True)
    r = np.random.default_rng(10 * S + H)
    deg = np.concatenate([[0, 0, 1], r.integers(0, 3, 700), [0, 700, 0, 2500, 0], r.integers(0, 40, 60), [1], np.zeros(3, np.int64)])
    V, ncols, D, E = deg.size, 333, 8, int(deg.sum())
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    row = np.repeat(np.arange(V), deg)
    col = r.integers(0, ncols, E).astype(np.int32)
    col = col[np.lexsort((col, row))]
    U, Vt = f16(r.standard_normal((V, H * D))), f16(r.standard_normal((ncols, H * D)))
    al, ar = f16(0.3 * r.standard_normal((H, D))), f16(0.3 * r.standard_normal((H, D)))
    parts = [np.einsum("vhd,hd->vh", f(X.astype(np.float64)).reshape(-1, H, D), f(a.astype(np.float64)))[i]
             for f in (np.asarray, np.abs) for X, a, i in ((U, al, row), (Vt, ar, col))]
    s = parts[0] + parts[1]
    ref, mag = np.where(s > 0, s, 0.2 * s), parts[2] + parts[3]
    for shift in (0, 1, 2):
        cbuf = torch.zeros(E + shift, dtype=torch.int32, device=dev)
        cbuf[shift:] = up(col, dev)
        g = hgnn.Csr(up(rowptr, dev), cbuf[shift:], ncols=ncols)
        p = hgnn.hgnn_plan_create(g, S, 64, 8)
        obuf = torch.full((E * H + 2,), 7.0, dtype=torch.float16, device=dev)
        out = obuf[shift:shift + E * H].view(E, H)
        hgnn.hgnn_sddmm(g, p, hgnn.HGNN_SDDMM_GAT_SCORE, H, D, up(U, dev), up(Vt, dev), out, up(al, dev), up(ar, dev), 0.2)
        compare("score", down(out), ref, mag)
        assert torch.all(obuf[:shift] == 7.0) and torch.all(obuf[shift + E * H:] == 7.0)
        hgnn.hgnn_plan_destroy(p)
