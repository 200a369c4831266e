"""The discretized SpMM over row tasks at the sizes where a piece of work changes shape: row lengths around a tile (8), a round
(32), the longest lane-group piece and the segment size; every lanes-per-row count; tables beyond 4 GiB."""
import numpy as np
import pytest
import torch

import oracle
from parity import compare, down, f16, spmm_plain, up

pytestmark = pytest.mark.gpu

EDGES = (1, 7, 8, 9, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 2049)


def border_graph(V, ncols, seed):
    """Rows of every border length, scattered among short and empty ones; columns ascending."""
    r = np.random.default_rng(seed)
    deg = r.integers(0, 6, size=V)
    deg[r.permutation(V)[:len(EDGES)]] = EDGES
    deg[V - 1] = 40
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    col = np.concatenate([np.sort(r.integers(0, ncols, size=d)) for d in deg]).astype(np.int32)
    return rowptr, col


@pytest.mark.parametrize("F,H,S,nb", [(8, 1, 256, 1), (16, 1, 256, 1), (32, 1, 100, 1), (42, 1, 256, 1), (64, 1, 256, 3), (64, 2, 64, 1),
                                      (64, 4, 256, 3), (64, 8, 256, 1), (100, 1, 2048, 1), (128, 1, 256, 2), (128, 16, 1, 1),
                                      (256, 8, 256, 1), (512, 1, 256, 1)])
@pytest.mark.parametrize("what", ["plain", "w", "map"])
def test_piece_borders(hgnn, dev, F, H, S, nb, what):
    print(f"row tasks F={F} H={H} S={S} nb={nb} {what}", flush=True)
    V = 2300  # more than two windows of rows
    rowptr, col = border_graph(V, V, F + S)
    r = np.random.default_rng(F)
    pitch = (F + 7) // 8 * 8
    Xh = np.zeros((V, pitch), dtype=np.float16)
    Xh[:, :F] = f16(r.standard_normal((V, F)))
    w = None if what == "plain" else f16(r.standard_normal((col.size, H)))
    H = 1 if w is None else H
    wd = None if w is None else up(w, dev)
    g = hgnn.Csr(up(rowptr, dev), up(col, dev))
    eid = None
    if what == "map":
        g = hgnn.hgnn_transpose(g)
        rowptr, col, eid = down(g.rowptr), down(g.col), down(g.eid)
    p = hgnn.hgnn_plan_create(g, S, pitch, H, col_blocks=nb)
    Y = torch.full((V, pitch), 3.0, dtype=torch.float16, device=dev)
    hgnn.hgnn_spmm_discretized(p, g, wd, H, up(Xh, dev), Y, F=F)
    ref, sabs = oracle.spmm(rowptr, col, np.ascontiguousarray(Xh[:, :F]), w=w, H=H, want_sabs=True, **({"eid": eid} if eid is not None else {}))
    compare("row tasks", np.ascontiguousarray(down(Y)[:, :F]), ref, sabs)
    hgnn.hgnn_plan_destroy(p)


@pytest.mark.parametrize("S,less,times", [(256, 0, 1), (256, 1, 1), (64, 0, 1), (50, 0, 1), (24, 0, 1), (256, 0, 2), (64, 0, 2), (50, 0, 3), (24, 0, 3)])
def test_windows_of_middle_rows(hgnn, dev, S, less, times):
    """Windows of 1024 rows whose rows of 33 to 64 non-zeros are left to lane groups or take a wave each: all of them, none, at the border of the
    rule, beside longer and empty ones, in pieces of several to a row; graphs of 2^18 non-zeros and one fewer; with a plan only graphs of 7000 such
    rows or more (4200 in one set of the windows)."""
    print(f"middle rows S={S} less={less} times={times}", flush=True)
    r = np.random.default_rng(S)
    window = lambda *kinds: r.permutation(np.concatenate([np.broadcast_to(v, n) for n, v in kinds]))
    wins = [window((1024, 47)), window((1024, r.integers(33, 65, 1024))), window((500, 64), (62, 65), (12, 1), (450, 0)),
            window((500, 33), (374, 3), (1, 300), (149, 40)), window((512, 32), (512, 64)), window((86, 50), (516, 9), (422, 0)),
            window((86, 50), (515, 9), (423, 0)), window((350, 64), (674, 0)), window((300, 8))]
    deg = np.concatenate(wins * times)
    deg[-1] = 0
    deg[-1] = (1 << 18) - less - deg.sum() if times == 1 else 1000  # one long row
    assert 300 < deg[-1] < 60000
    V, F = deg.size, 16
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    row = np.repeat(np.arange(V), deg)
    col = r.integers(0, V, row.size).astype(np.int32)
    col = col[np.lexsort((col, row))]
    X, w = f16(r.standard_normal((V, F))), f16(r.standard_normal((row.size, 1)))
    g, Xd, wd = hgnn.Csr(up(rowptr, dev), up(col, dev)), up(X, dev), up(w, dev)
    p = hgnn.hgnn_plan_create(g, S, F, 1, col_blocks=1)
    ref, sabs = oracle.spmm(rowptr, col, X, w=w, H=1, want_sabs=True)
    Y = torch.full((V, F), 3.0, dtype=torch.float16, device=dev)
    hgnn.hgnn_spmm_discretized(p, g, wd, 1, Xd, Y)
    compare("with a plan", down(Y), ref, sabs)
    Y.fill_(3.0)
    spmm_plain(hgnn, g, wd, 1, Xd, Y)
    compare("without", down(Y), ref, sabs)
    dot = torch.full((row.size, 1), 3.0, dtype=torch.float16, device=dev)
    hgnn.hgnn_sddmm(g, p, hgnn.HGNN_SDDMM_DOT, 1, F, Xd, Xd, dot)
    mag = np.einsum("ef,ef->e", np.abs(X[row].astype(np.float64)), np.abs(X[col].astype(np.float64)))[:, None]
    compare("dot", down(dot), oracle.sddmm_dot(rowptr, col, X, X, H=1), mag)
    hgnn.hgnn_plan_destroy(p)


def test_middle_rows_in_order_of_lengths(hgnn, dev):
    """A power law in the order of its degrees has windows of nothing but rows of 33 to 64 non-zeros, beside many others.  They stay with the waves
    they have when the rows are in any order (in lane groups, 1.06 times the time of any order; with waves 0.99)."""
    r = np.random.default_rng(1)
    deg = np.minimum(4000, 60000 * (np.arange(30000) + 20.0) ** -0.85).astype(np.int64) + 1
    F, both = 16, []
    for order in (deg, r.permutation(deg)):
        V, E = order.size, int(order.sum())
        row = torch.repeat_interleave(torch.arange(V, device=dev), up(order, dev))
        col = torch.sort(row * V + torch.randint(0, V, (E,), device=dev))[0] % V
        g = hgnn.Csr(up(np.concatenate([[0], np.cumsum(order)]).astype(np.int32), dev), col.int())
        p = hgnn.hgnn_plan_create(g, 256, F, 1, col_blocks=1)
        X = torch.randn((V, F), device=dev).half()
        Y, e = torch.empty_like(X), torch.empty((E, 1), dtype=torch.float16, device=dev)

        def call(g=g, p=p, X=X, Y=Y, e=e):
            hgnn.hgnn_sddmm(g, p, hgnn.HGNN_SDDMM_DOT, 1, F, X, X, e)
            hgnn.hgnn_spmm_discretized(p, g, None, 1, X, Y)

        both.append(call)

    def median_us(call):
        us = []
        for _ in range(11):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                call()
            b.record()
            b.synchronize()
            us.append(100 * a.elapsed_time(b))
        return sorted(us)[5]

    tries = [median_us(both[0]) / median_us(both[1]) for _ in range(4)]
    print("in order / in any order: " + ", ".join(f"{t:.3f}" for t in tries), flush=True)
    assert min(tries) < 1.03


@pytest.mark.parametrize("F,H,what", [(64, 1, "plain"), (64, 1, "w"), (64, 2, "map"), (64, 4, "w"), (64, 4, "map"), (64, 8, "w"), (128, 1, "norm"), (128, 8, "w"),
                                      (256, 4, "map"), (512, 1, "norm"), (16, 1, "w")])
def test_rounds_of_blocks_at_borders(hgnn, dev, F, H, what):
    """Pieces of column blocks around a batch of ids, a round of 64 and the longest lane-group piece (256), SpMM and dot products."""
    print(f"rounds F={F} H={H} {what}", flush=True)
    lens = (0, 1, 7, 8, 9, 31, 32, 33, 39, 40, 41, 63, 64, 65, 95, 96, 97, 127, 128, 129, 191, 193, 255, 256)
    V, half = 64 * len(lens), 32 * len(lens)
    r = np.random.default_rng(F + H)
    pick = lambda n, lo: np.sort(r.choice(half, n, replace=False)) + lo  # noqa: E731
    parts = [np.concatenate([pick(lens[i % len(lens)], 0), pick(lens[(i // len(lens) + i) % len(lens)], half)]) for i in range(V)]
    rowptr = np.concatenate([[0], np.cumsum([q.size for q in parts])]).astype(np.int32)
    col = np.concatenate(parts).astype(np.int32)
    X, U = f16(r.standard_normal((V, F))), f16(r.standard_normal((V, F)))
    w = f16(r.standard_normal((col.size, H))) if what in ("w", "map") else None
    g = hgnn.Csr(up(rowptr, dev), up(col, dev))
    eid = None
    if what == "map":  # (a graph that carries a map need not come from hgnn_transpose)
        eid = r.permutation(col.size).astype(np.int32)
        g = hgnn.Csr(up(rowptr, dev), up(col, dev), eid=up(eid, dev))
    p = hgnn.hgnn_plan_create(g, 256, F, H, col_blocks=2)
    Y = torch.full((V, F), 3.0, dtype=torch.float16, device=dev)
    kw = {}
    if what == "norm":
        cs, rs = (r.uniform(0.5, 2, V).astype(np.float32) for _ in range(2))
        kw = {"row_scale": up(rs, dev), "col_scale": up(cs, dev)}
    hgnn.hgnn_spmm_discretized_fused(p, g, None if w is None else up(w, dev), H, up(X, dev), Y, F=F, **kw)
    if what == "norm":
        dense = np.zeros((V, V))
        np.add.at(dense, (np.repeat(np.arange(V), np.diff(rowptr)), col), 1.0)
        ref = rs[:, None].astype(np.float64) * (dense @ (cs[:, None].astype(np.float64) * X.astype(np.float64)))
        sabs = rs[:, None].astype(np.float64) * (dense @ (cs[:, None].astype(np.float64) * np.abs(X.astype(np.float64))))
    else:
        ref, sabs = oracle.spmm(rowptr, col, X, w=w, H=H if w is not None else 1, want_sabs=True, **({"eid": eid} if eid is not None else {}))
    compare("rounds of blocks", down(Y), ref, sabs)
    D = F // H
    if what != "map" and D % 8 == 0:
        e = torch.full((col.size, H), 7.0, dtype=torch.float16, device=dev)
        hgnn.hgnn_sddmm(g, p, hgnn.HGNN_SDDMM_DOT, H, D, up(U, dev), up(X, dev), e)
        row = np.repeat(np.arange(V), np.diff(rowptr))
        mag = (np.abs(U[row].astype(np.float64)) * np.abs(X[col].astype(np.float64))).reshape(-1, H, D).sum(-1)
        compare("dot products of blocks", down(e), oracle.sddmm_dot(rowptr, col, U, X, H=H), mag)
    hgnn.hgnn_plan_destroy(p)


@pytest.mark.parametrize("bad", [np.inf, np.nan])
@pytest.mark.parametrize("nb", [1, 2])
@pytest.mark.parametrize("F,H,what", [(64, 1, "none"), (64, 1, "w"), (64, 1, "map"), (64, 2, "w"), (64, 2, "map"), (42, 1, "none"), (16, 1, "w"),
                                      (256, 1, "map")])
def test_values_that_no_non_zero_reaches(hgnn, dev, F, H, what, nb, bad):
    """Column factors and feature rows of columns without non-zeros (the first of the graph and of a block, the last), and the edge value of
    slot 0, which belongs to one row: none of them is in any other row, whatever the rows leave over of a batch, a round or a wave."""
    print(f"unreached values F={F} H={H} {what} nb={nb} {bad}", flush=True)
    lens = np.array([1, 2, 3, 4, 5, 6, 7, 8, 9, 0, 15, 17, 31, 32, 33, 40, 41, 63, 64, 65, 95, 127, 129, 191, 255, 256, 257, 300])
    deg = np.tile(lens, 12)
    V, D = deg.size, F // H
    r = np.random.default_rng(F + H + nb)
    dead = np.array([0, V // 2, V - 1])
    alive = np.setdiff1d(np.arange(V), dead)
    col = np.concatenate([np.sort(r.choice(alive, n)) for n in deg]).astype(np.int32)
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    row, E = np.repeat(np.arange(V), deg), col.size
    X, cs, rs = f16(r.standard_normal((V, F))), r.uniform(0.5, 2, V).astype(np.float32), r.uniform(0.5, 2, V).astype(np.float32)
    X[dead], cs[dead] = bad, bad
    w = eid = None
    keep = np.ones(V, bool)
    if what != "none":
        w = f16(r.standard_normal((E, H)))
    if what == "map":
        eid = r.permutation(E).astype(np.int32)
        w[0] = bad  # of one non-zero
        keep[row[eid == 0]] = False
    g = hgnn.Csr(up(rowptr, dev), up(col, dev), eid=None if eid is None else up(eid, dev))
    p = hgnn.hgnn_plan_create(g, 256, (F + 7) // 8 * 8, H, col_blocks=nb)
    pitch = (F + 7) // 8 * 8
    Xp = np.zeros((V, pitch), np.float16)
    Xp[:, :F] = X
    f = np.ones((E, H)) if w is None else w[slice(None) if eid is None else eid].astype(np.float64)
    f = np.repeat(f * cs[col][:, None], D, 1)
    for scaled in (None, torch.zeros((V, pitch), dtype=torch.float16, device=dev)):
        Y = torch.full((V, pitch), 3.0, dtype=torch.float16, device=dev)
        hgnn.hgnn_spmm_discretized_fused(p, g, None if w is None else up(w, dev), H, up(Xp, dev), Y, F=F, row_scale=up(rs, dev), col_scale=up(cs, dev),
                                         scaled_x=scaled)
        got = down(Y)[:, :F]
        terms = np.where(keep[row][:, None], f * X[col].astype(np.float64), 0.0)
        ref, mag = np.zeros((V, F)), np.zeros((V, F))
        np.add.at(ref, row, terms)
        np.add.at(mag, row, np.abs(terms))
        compare("unreached values", got[keep], (rs[:, None] * ref)[keep], (rs[:, None] * mag)[keep])
        assert not np.isfinite(got[~keep]).any()
    hgnn.hgnn_plan_destroy(p)


@pytest.mark.parametrize("H", [1, 4])
def test_table_beyond_4_gib(hgnn, dev, H):
    """Rows 2.2 M halves apart: the table spans 4.8 GB, its rows are read by 64-bit addresses."""
    V, F, ld = 1100, 64, 2200000
    rowptr, col = border_graph(V, V, 5)
    r = np.random.default_rng(9)
    Xh = f16(r.standard_normal((V, F)))
    w = f16(r.standard_normal((col.size, H)))
    far = torch.empty((V, ld), dtype=torch.float16, device=dev)
    X = far[:, :F]
    X.copy_(up(Xh, dev))
    g = hgnn.Csr(up(rowptr, dev), up(col, dev))
    p = hgnn.hgnn_plan_create(g, 256, F, H)
    Y = torch.empty((V, F), dtype=torch.float16, device=dev)
    for wd, wn, h in ((up(w, dev), w, H), (None, None, 1)):
        hgnn.hgnn_spmm_discretized(p, g, wd, h, X, Y, F=F)
        ref, sabs = oracle.spmm(rowptr, col, Xh, w=wn, H=h, want_sabs=True)
        compare("far table", down(Y), ref, sabs)
    hgnn.hgnn_plan_destroy(p)


@pytest.mark.parametrize("H,S,nb", [(1, 256, 1), (2, 64, 3), (4, 256, 2), (8, 256, 1), (8, 1, 3), (4, 2048, 1)])
def test_row_sums_through_the_map(hgnn, dev, H, S, nb):
    print(f"row sums H={H} S={S} nb={nb}", flush=True)
    V = 2300
    rowptr, col = border_graph(V, V, H + S)
    t = f16(np.random.default_rng(H).standard_normal((col.size, H)))
    gt = hgnn.hgnn_transpose(hgnn.Csr(up(rowptr, dev), up(col, dev)))
    g = hgnn.hgnn_transpose(hgnn.Csr(gt.rowptr, gt.col, ncols=V))  # the border rows again, now with a map
    rp, slots = down(g.rowptr), down(g.eid)
    p = hgnn.hgnn_plan_create(g, S, 8, H, col_blocks=nb)
    out = torch.full((V, H), 3.0, dtype=torch.float16, device=dev)
    hgnn.hgnn_edge_rowsum(g, p, H, up(t, dev), out)
    t64 = t.astype(np.float64)[slots]
    compare("row sums", down(out), oracle.edge_rowsum(rp, t64), oracle.edge_rowsum(rp, np.abs(t64)))
    hgnn.hgnn_plan_destroy(p)


def test_positions_up_to_the_last_one(hgnn, dev):
    """2^31 - 1 non-zeros: the walks over the last pieces form sums beyond 2^31.  Every column is 0, so the results are known."""
    if torch.cuda.get_device_properties(dev).total_memory < 100 << 30:
        pytest.skip("needs 60 GB of device memory")
    E, tail = (1 << 31) - 1, [1, 7, 0, 9, 33, 255, 300, 2000]
    rest = E - sum(tail)
    n = -(-rest // 2000)
    deg = torch.full((n + len(tail),), rest // n, dtype=torch.int64, device=dev)
    deg[:rest % n] += 1
    deg[n:] = torch.tensor(tail, device=dev)
    V, D = deg.numel(), 8
    rowptr = torch.zeros(V + 1, dtype=torch.int64, device=dev)
    torch.cumsum(deg, 0, out=rowptr[1:])
    assert int(rowptr[-1]) == E
    col = torch.zeros(E, dtype=torch.int32, device=dev)
    g = hgnn.Csr(rowptr.int(), col, ncols=8)
    x0 = torch.tensor([1, 0.5, 1, 0.5, 1, 1, 0.5, 1], dtype=torch.float16, device=dev)
    X = torch.zeros((8, D), dtype=torch.float16, device=dev)
    X[0] = x0
    want = deg[:, None].float() * x0.float()  # at most 2000, halves: exact in fp16, partial sums too
    Y = torch.empty((V, D), dtype=torch.float16, device=dev)

    def check(what):
        torch.cuda.synchronize()
        print(what, flush=True)
        assert torch.equal(Y.float(), want), what

    p = hgnn.hgnn_plan_create(g, 256, D, 1)
    hgnn.hgnn_spmm_discretized(p, g, None, 1, X, Y)
    check("discretized")
    w = torch.ones((E, 1), dtype=torch.float16, device=dev)
    hgnn.hgnn_spmm_discretized(p, g, w, 1, X, Y)
    check("edge values")
    ws = torch.empty(hgnn.hgnn_spmm_workspace(V, 8, E, D), dtype=torch.uint8, device=dev)
    hgnn.hgnn_spmm(g, w, 1, X, Y, workspace=ws)
    check("without a plan")
    hgnn.hgnn_spmm(g, w, 1, X, Y)
    check("without a workspace")
    gm = hgnn.Csr(g.rowptr, col, ncols=8, eid=torch.arange(E, dtype=torch.int32, device=dev))
    hgnn.hgnn_spmm_discretized(p, gm, w, 1, X, Y)
    check("through the map")
    sums = torch.empty((V, 1), dtype=torch.float16, device=dev)
    for q in (p, None):
        hgnn.hgnn_edge_rowsum(gm, q, 1, w, sums)
        assert torch.equal(sums[:, 0].float(), deg.float()), q
    del gm, ws
    print("row sums", flush=True)
    U = x0.repeat(V, 1)
    hgnn.hgnn_sddmm(g, p, hgnn.HGNN_SDDMM_DOT, 1, D, U, X, w)
    assert bool((w == float((x0.float() ** 2).sum())).all())
    print("sddmm", flush=True)
    zero = torch.zeros(D, dtype=torch.float16, device=dev)
    lse = torch.empty((V, 1), dtype=torch.float32, device=dev)
    hgnn.hgnn_gat_forward_fused(g, p, 1, D, U, X, zero, zero, Y, lse)
    full = (deg > 0)[:, None]
    assert ((Y.float() - x0.float() * full).abs() <= 1e-3).all()
    assert ((lse[:, 0] - deg.clamp(min=1).float().log()).abs() <= 1e-4).all()
    print("gat forward", flush=True)
    del w
    col_t = torch.repeat_interleave(torch.arange(V, dtype=torch.int32, device=dev), deg, output_size=E)
    rp_t = torch.full((9,), E, dtype=torch.int32, device=dev)
    rp_t[0] = 0
    gt = hgnn.Csr(rp_t, col_t, ncols=V)
    pt = hgnn.hgnn_plan_create(gt, 256, D, 1)
    dO = torch.full((V, D), 2.0 ** -6, dtype=torch.float16, device=dev)
    dV, d_el, d_er = torch.empty_like(X), torch.empty((V, 1), dtype=torch.float16, device=dev), torch.empty((8, 1), dtype=torch.float16, device=dev)
    hgnn.hgnn_gat_backward_fused(g, p, gt, pt, 1, D, U, X, zero, zero, Y, lse, dO, dV, d_el, d_er)
    total = float(full.sum()) * 2.0 ** -6  # each row's weights add up to one; 8.4 M pieces, rounded to fp16 once each
    assert ((dV[0].float() - total).abs() <= 2e-3 * total).all() and (dV[1:] == 0).all()
    assert (d_el.abs() <= 1e-3).all()
    hgnn.hgnn_plan_destroy(p)
    hgnn.hgnn_plan_destroy(pt)


def test_both_kinds_of_pieces_side_by_side(hgnn, dev):
    """A graph beyond the size from which whole-wave and lane-group pieces alternate: every piece is taken once, for every number
    of lane groups per wave, with one kind rare."""
    V = 30000
    r = np.random.default_rng(4)
    for long_rows in (5, 9000):
        deg = r.integers(0, 300, size=V)  # pieces up to 256, lane groups up to 32
        deg[deg > 32] //= 9
        deg[r.permutation(V)[:long_rows]] = 4_300_000 // long_rows if long_rows > 100 else 880_000
        rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
        assert rowptr[-1] > 4 << 20
        g = hgnn.Csr(up(rowptr, dev), torch.zeros(int(rowptr[-1]), dtype=torch.int32, device=dev), ncols=8)
        w = torch.full((g.nnz, 1), 2.0 ** -10, dtype=torch.float16, device=dev)
        for F in (8, 32, 64, 128, 512):
            X = torch.zeros((8, F), dtype=torch.float16, device=dev)
            X[0] = 1
            p = hgnn.hgnn_plan_create(g, 256, F, 1)
            Y = torch.full((V, F), 3.0, dtype=torch.float16, device=dev)
            hgnn.hgnn_spmm_discretized(p, g, w, 1, X, Y)
            got = down(Y).astype(np.float64)
            want = deg * 2.0 ** -10
            assert np.abs(got - want[:, None]).max() <= 2.0 ** -11 * want.max(), (long_rows, F)  # pieces are exact, one rounding
            assert np.array_equal(got[want <= 2], np.broadcast_to(want[:, None], got.shape)[want <= 2]), (long_rows, F)
            hgnn.hgnn_plan_destroy(p)


# (H, D, S, col_blocks): every number of lanes per row and per head, pieces of one non-zero, of a round, of the largest segment
SHAPES = [(1, 8, 1, 1), (1, 8, 256, 3), (2, 8, 32, 1), (1, 16, 64, 2), (4, 8, 256, 1), (2, 16, 33, 3), (1, 32, 2048, 1), (8, 8, 256, 1),
          (4, 16, 256, 2), (2, 32, 100, 1), (1, 64, 256, 3), (4, 32, 256, 1), (1, 128, 1, 3), (8, 32, 256, 1), (1, 256, 64, 2), (8, 64, 256, 1)]


@pytest.mark.parametrize("H,D,S,nb", SHAPES)
def test_sddmm_piece_borders(hgnn, dev, H, D, S, nb):
    """The dot products at the borders of pieces, over blocks too, at every width of the vector-width study."""
    print(f"sddmm borders H={H} D={D} S={S} nb={nb}", flush=True)
    V, F = 2300, H * D
    rowptr, col = border_graph(V, V, F + S)
    r = np.random.default_rng(F)
    U, X = f16(r.standard_normal((V, F))), f16(r.standard_normal((V, F)))
    g = hgnn.Csr(up(rowptr, dev), up(col, dev))
    p = hgnn.hgnn_plan_create(g, S, F, H, col_blocks=nb)
    ref = oracle.sddmm_dot(rowptr, col, U, X, H=H)
    row = np.repeat(np.arange(V), np.diff(rowptr))
    mag = (np.abs(U[row].astype(np.float64)) * np.abs(X[col].astype(np.float64))).reshape(-1, H, D).sum(-1)
    Ud, Xd = up(U, dev), up(X, dev)
    for vw in (8, 4, 2):
        if F > 64 * vw:
            continue
        hgnn.hgnn_plan_set_vector_halves(p, vw)
        e = torch.full((col.size, H), 7.0, dtype=torch.float16, device=dev)
        hgnn.hgnn_sddmm(g, p, hgnn.HGNN_SDDMM_DOT, H, D, Ud, Xd, e)
        compare(f"sddmm borders, {vw} halves per lane", down(e), ref, mag)
    hgnn.hgnn_plan_destroy(p)


@pytest.mark.parametrize("D,S,nb", [(2, 256, 1), (6, 64, 3), (42, 256, 2), (100, 1, 1), (250, 2048, 3)])
def test_sddmm_masked_piece_borders(hgnn, dev, D, S, nb):
    """One head whose length is no multiple of 8; the padding columns hold what must not count."""
    V, ld = 2300, (D + 7) // 8 * 8
    rowptr, col = border_graph(V, V, D + S)
    r = np.random.default_rng(D)
    U, X = np.full((V, ld), np.nan, np.float16), np.full((V, ld), np.inf, np.float16)
    U[:, :D], X[:, :D] = f16(r.standard_normal((V, D))), f16(r.standard_normal((V, D)))
    g = hgnn.Csr(up(rowptr, dev), up(col, dev))
    p = hgnn.hgnn_plan_create(g, S, ld, 1, col_blocks=nb)
    e = torch.full((col.size, 1), 7.0, dtype=torch.float16, device=dev)
    hgnn.hgnn_sddmm(g, p, hgnn.HGNN_SDDMM_DOT, 1, D, up(U, dev), up(X, dev), e)
    u, x = np.ascontiguousarray(U[:, :D]), np.ascontiguousarray(X[:, :D])
    row = np.repeat(np.arange(V), np.diff(rowptr))
    mag = (np.abs(u[row].astype(np.float64)) * np.abs(x[col].astype(np.float64))).sum(-1, keepdims=True)
    compare("masked sddmm borders", down(e), oracle.sddmm_dot(rowptr, col, u, x), mag)
    hgnn.hgnn_plan_destroy(p)


@pytest.mark.parametrize("flip", [False, True])  # border rows in the pass over the graph, or in the one over its transpose
@pytest.mark.parametrize("H,D,S,nb", SHAPES)
def test_gat_piece_borders(hgnn, dev, H, D, S, nb, flip):
    print(f"gat borders H={H} D={D} S={S} nb={nb} flip={flip}", flush=True)
    from test_gpu_gat_fused import bwd_reference, check_lse
    V, F = 2300, H * D
    rowptr, col = border_graph(V, V, F + S + 1)
    if flip:
        rowptr, col = oracle.transpose(rowptr, col, V)[:2]
    r = np.random.default_rng(F + 1)
    X, dOut = f16(r.standard_normal((V, F))), f16(r.standard_normal((V, F)))
    a_l, a_r = f16(0.3 * r.standard_normal(F)), f16(0.3 * r.standard_normal(F))
    oref, lref, oabs, mref, cref = oracle.gat_forward(rowptr, col, X, X, a_l, a_r, H, want_saved=True)
    (dV, dV_abs), (d_el, el_abs), (d_er, er_abs) = bwd_reference(rowptr, col, V, X, X, a_l, a_r, dOut, H)
    g = hgnn.Csr(up(rowptr, dev), up(col, dev))
    gt = hgnn.hgnn_transpose(g)
    p, pt = (hgnn.hgnn_plan_create(x, S, F, H, col_blocks=nb) for x in (g, gt))
    Xd, dOd, ald, ard = (up(t, dev) for t in (X, dOut, a_l, a_r))
    half = lambda *s: torch.full(s, 7.0, dtype=torch.float16, device=dev)  # noqa: E731
    f32 = lambda *s: torch.full(s, 7.0, dtype=torch.float32, device=dev)  # noqa: E731
    out, outm, lse, csum, out0 = half(V, F), half(V, F), f32(V, H), f32(V, H), half(V, F)
    hgnn.hgnn_gat_forward_fused_save(g, p, H, D, Xd, Xd, ald, ard, out, lse, outm, csum)
    hgnn.hgnn_gat_forward_fused(g, p, H, D, Xd, Xd, ald, ard, out0)
    compare("out", down(out), oref, oabs)
    assert np.array_equal(down(out0).view(np.uint16), down(out).view(np.uint16))
    check_lse("borders", down(lse), lref, np.diff(rowptr))
    compare("out_masked", down(outm), mref, oabs)
    assert np.abs(down(csum).astype(np.float64) - cref).max() <= 2e-3
    # dV of a column is staged in fp16 pieces and block partials: values below 2^-14 lose up to 2^-25 with each of them (compare
    # allows 2^-11 of the magnitude it is given)
    dV_abs = dV_abs + 2.0 ** 11 * 2.0 ** -25 * (np.bincount(col, minlength=V)[:, None] / S + nb + 1)
    for saved in (False, True):
        gV, gl, gr = half(V, F), half(V, H), half(V, H)
        if saved:
            hgnn.hgnn_gat_backward_fused_saved(g, p, gt, pt, H, D, Xd, Xd, ald, ard, out, lse, outm, csum, dOd, gV, gl, gr)
        else:
            hgnn.hgnn_gat_backward_fused(g, p, gt, pt, H, D, Xd, Xd, ald, ard, out, lse, dOd, gV, gl, gr)
        compare("dV", down(gV), dV, dV_abs)
        compare("d_el", down(gl), d_el, el_abs, rel_l2=2e-2)  # cancelling sums, as in the tests of the shapes
        compare("d_er", down(gr), d_er, er_abs, rel_l2=2e-2)
    hgnn.hgnn_plan_destroy(p)
    hgnn.hgnn_plan_destroy(pt)


@pytest.mark.parametrize("F,what", [(64, "w"), (42, "map"), (32, "none")])
def test_plain_spmm_with_a_smaller_workspace(hgnn, dev, F, what):
    """A workspace that holds the chunks of the long rows and not the pieces of all rows: the same sums in another order."""
    V, pitch = 5000, (F + 7) // 8 * 8
    r = np.random.default_rng(F)
    deg = r.integers(0, 12, V)
    deg[r.permutation(V)[:40]] = r.integers(300, 5000, 40)
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    col = np.concatenate([np.sort(r.integers(0, V, size=d)) for d in deg]).astype(np.int32)
    E = col.size
    Xh = np.zeros((V, pitch), dtype=np.float16)
    Xh[:, :F] = f16(r.standard_normal((V, F)))
    w = None if what == "none" else f16(r.standard_normal((E, 1)))
    eid = r.permutation(E).astype(np.int32) if what == "map" else None
    g = hgnn.Csr(up(rowptr, dev), up(col, dev), eid=None if eid is None else up(eid, dev))
    ref, sabs = oracle.spmm(rowptr, col, np.ascontiguousarray(Xh[:, :F]), w=w, want_sabs=True, **({} if eid is None else {"eid": eid}))
    long_row = min(max(256, 8 * (E // V)), 1024)
    chunks = E // 512 + E // long_row + 2
    least = 256 + 2 * (4 * chunks + 256) + 2 * (4 * (E // long_row + 1) + 256) + 4 * chunks * pitch + 256
    full = hgnn.hgnn_spmm_workspace(V, V, E, F)
    assert least < full
    for n in (least, full - 513, full):  # (513: up to 512 bytes short of what the query names is refused)
        Y = torch.full((V, pitch), 3.0, dtype=torch.float16, device=dev)
        hgnn.hgnn_spmm(g, None if w is None else up(w, dev), 1, up(Xh, dev), Y, F=F, workspace=torch.empty(n, dtype=torch.uint8, device=dev))
        compare(f"workspace of {n}", np.ascontiguousarray(down(Y)[:, :F]), ref, sabs)


# up to 8192 rows of several pieces, and up to 65536 of nine on average (of six where a wave holds 32 rows or more), take a wave each in the
# follow-up kernels, others a lane group: both sides of every line, the average by one piece; a piece is one non-zero
@pytest.mark.parametrize("V,least,most,fewer,D", [(8192, 2, 6, 0, 8), (8193, 2, 6, 0, 8), (8192, 2, 6, 0, 32), (8193, 2, 6, 0, 32),
                                                  (65536, 6, 14, 0, 8), (65537, 6, 14, 0, 8), (65536, 9, 14, 0, 32), (65537, 9, 14, 0, 32),
                                                  (9000, 6, 6, 0, 8), (9000, 6, 6, 1, 8), (9000, 9, 9, 0, 32), (9000, 9, 9, 1, 32)])
def test_many_rows_of_several_pieces(hgnn, dev, V, least, most, fewer, D):
    print(f"follow-up rows V={V} pieces {least}..{most} less {fewer} D={D}", flush=True)
    r = np.random.default_rng(V)
    deg = r.integers(least, most + 1, size=V)
    if least < most:
        deg[:12] = (8, 9, 10, 16, 17, 31, 33, 40, 64, 65, 66, 300)
    deg[V // 2] -= fewer
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    col = np.concatenate([np.sort(r.integers(0, V, size=d)) for d in deg]).astype(np.int32)
    H = 2
    F = H * D
    X, dO = f16(r.standard_normal((V, F))), f16(r.standard_normal((V, F)))
    w = f16(r.standard_normal((col.size, H)))
    a_l, a_r = f16(0.3 * r.standard_normal(F)), f16(0.3 * r.standard_normal(F))
    g = hgnn.Csr(up(rowptr, dev), up(col, dev))
    gt = hgnn.hgnn_transpose(g)
    p, pt, pt1 = (hgnn.hgnn_plan_create(x, s, F, H, col_blocks=1) for x, s in ((g, 1), (gt, 256), (gt, 1)))
    half = lambda *s: torch.full(s, 7.0, dtype=torch.float16, device=dev)
    f32 = lambda *s: torch.full(s, 7.0, dtype=torch.float32, device=dev)
    Y = half(V, F)
    hgnn.hgnn_spmm_discretized(p, g, up(w, dev), H, up(X, dev), Y)
    ref, sabs = oracle.spmm(rowptr, col, X, w=w, H=H, want_sabs=True)
    compare("follow-up", down(Y), ref, sabs)
    Xd, ald, ard, dOd = up(X, dev), up(a_l, dev), up(a_r, dev), up(dO, dev)
    out, outm, lse, csum = half(V, F), half(V, F), f32(V, H), f32(V, H)
    hgnn.hgnn_gat_forward_fused_save(g, p, H, D, Xd, Xd, ald, ard, out, lse, outm, csum)
    oref, lref, oabs, mref, cref = oracle.gat_forward(rowptr, col, X, X, a_l, a_r, H, slope=0.2, want_saved=True)
    compare("out", down(out), oref, oabs)
    compare("out_masked", down(outm), mref, oabs)
    assert np.abs(down(csum) - cref).max() <= 2e-3 and np.abs(down(lse) - lref).max() <= 2e-3 + 1e-3 * np.abs(lref).max()
    got = []
    for q in (pt, pt1):
        dV, d_el, d_er = half(V, F), half(V, H), half(V, H)
        hgnn.hgnn_gat_backward_fused_saved(g, p, gt, q, H, D, Xd, Xd, ald, ard, out, lse, outm, csum, dOd, dV, d_el, d_er)
        got.append([down(t).astype(np.float64) for t in (dV, d_el, d_er)])
    for a, b in zip(*got):  # one rounding of a row against one of each of its pieces beside it
        assert np.linalg.norm(a - b) <= 2e-3 * np.linalg.norm(a)


# rows of about 32 pieces for each lane group of a wave, one more and several times as many, side by side: beyond them all waves of a workgroup add the
# pieces; with a row for each wave and for each lane group; in the pass over the graph or over its transpose; a piece is one non-zero
@pytest.mark.parametrize("flip", [False, True])
@pytest.mark.parametrize("V,D", [(700, 8), (700, 32), (700, 64), (300, 256), (9000, 32)])
def test_rows_of_many_pieces(hgnn, dev, V, D, flip):
    print(f"rows of many pieces V={V} D={D} flip={flip}", flush=True)
    H, r = 2, np.random.default_rng(V + D)
    F = H * D
    many = 32 * 64 * 8 // F
    deg = r.integers(2, 4, size=V)
    deg[40:47] = (many - 1, many, many + 1, 2 * many, 5 * many + 3, 4 * many, many + 1)
    deg[200], deg[V - 1] = many + 5, 9 * many
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    col = np.concatenate([np.sort(r.integers(0, V, size=d)) for d in deg]).astype(np.int32)
    if flip:
        rowptr, col = oracle.transpose(rowptr, col, V)[:2]
    X, dO = f16(r.standard_normal((V, F))), f16(r.standard_normal((V, F)))
    w = f16(r.standard_normal((col.size, H)))
    a_l, a_r = f16(0.3 * r.standard_normal(F) / np.sqrt(D)), f16(0.3 * r.standard_normal(F) / np.sqrt(D))
    g = hgnn.Csr(up(rowptr, dev), up(col, dev))
    gt = hgnn.hgnn_transpose(g)
    p, pt, pt1 = (hgnn.hgnn_plan_create(x, s, F, H, col_blocks=1) for x, s in ((g, 1), (gt, 256), (gt, 1)))
    half = lambda *s: torch.full(s, 7.0, dtype=torch.float16, device=dev)  # noqa: E731
    f32 = lambda *s: torch.full(s, 7.0, dtype=torch.float32, device=dev)  # noqa: E731
    Xd, ald, ard, dOd = up(X, dev), up(a_l, dev), up(a_r, dev), up(dO, dev)
    bits = []
    for _ in range(2):  # the same bits on a second run
        Y, out, outm, lse, csum, out0 = half(V, F), half(V, F), half(V, F), f32(V, H), f32(V, H), half(V, F)
        hgnn.hgnn_spmm_discretized(p, g, up(w, dev), H, Xd, Y)
        hgnn.hgnn_gat_forward_fused_save(g, p, H, D, Xd, Xd, ald, ard, out, lse, outm, csum)
        hgnn.hgnn_gat_forward_fused(g, p, H, D, Xd, Xd, ald, ard, out0)
        bits.append([down(t) for t in (Y, out, outm, lse, csum)])
        assert np.array_equal(down(out0).view(np.uint16), bits[-1][1].view(np.uint16))
    assert all(np.array_equal(a, b) for a, b in zip(*bits))
    ref, sabs = oracle.spmm(rowptr, col, X, w=w, H=H, want_sabs=True)
    compare("sum", down(Y), ref, sabs)
    oref, lref, oabs, mref, cref = oracle.gat_forward(rowptr, col, X, X, a_l, a_r, H, slope=0.2, want_saved=True)
    compare("out", down(out), oref, oabs)
    compare("out_masked", down(outm), mref, oabs)
    assert np.abs(down(csum) - cref).max() <= 2e-3 and np.abs(down(lse) - lref).max() <= 2e-3 + 1e-3 * np.abs(lref).max()
    got = []
    for q in (pt, pt1):
        dV, d_el, d_er = half(V, F), half(V, H), half(V, H)
        hgnn.hgnn_gat_backward_fused_saved(g, p, gt, q, H, D, Xd, Xd, ald, ard, out, lse, outm, csum, dOd, dV, d_el, d_er)
        got.append([down(t).astype(np.float64) for t in (dV, d_el, d_er)])
    for a, b in zip(*got):  # one rounding of a row against one of each of its pieces beside it
        assert np.linalg.norm(a - b) <= 2e-3 * np.linalg.norm(a)
    for q in (p, pt, pt1):
        hgnn.hgnn_plan_destroy(q)


# one row of 32 pieces for each lane group of a wave, alone or beside one of two pieces, and one piece more: up to there no row can have more, and the
# follow-up kernels look for none; a piece is one non-zero
@pytest.mark.parametrize("more", [0, 1])
@pytest.mark.parametrize("beside", [0, 1])
@pytest.mark.parametrize("D", [8, 64, 256])
def test_as_many_pieces_as_a_wave_adds(hgnn, dev, D, beside, more):
    print(f"as many pieces D={D} beside={beside} more={more}", flush=True)
    V, H, r = 90, 2, np.random.default_rng(D + 2 * beside + more)
    F = H * D
    deg = np.ones(V, dtype=np.int64)
    deg[41] = 32 * 64 * 8 // F + more
    deg[70] += beside
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    col = np.concatenate([np.sort(r.integers(0, V, size=d)) for d in deg]).astype(np.int32)
    X, w = f16(r.standard_normal((V, F))), f16(r.standard_normal((col.size, H)))
    a_l, a_r = f16(0.3 * r.standard_normal(F) / np.sqrt(D)), f16(0.3 * r.standard_normal(F) / np.sqrt(D))
    g = hgnn.Csr(up(rowptr, dev), up(col, dev))
    turned = hgnn.hgnn_transpose(g)
    gt = hgnn.Csr(turned.rowptr, turned.col, ncols=V)
    p, pt, back = hgnn.hgnn_plan_create(g, 1, F, H, col_blocks=1), hgnn.hgnn_plan_create(gt, 256, F, H, col_blocks=1), hgnn.hgnn_transpose(gt)
    half = lambda *s: torch.full(s, 7.0, dtype=torch.float16, device=dev)  # noqa: E731
    f32 = lambda *s: torch.full(s, 7.0, dtype=torch.float32, device=dev)  # noqa: E731
    Xd, ald, ard = up(X, dev), up(a_l, dev), up(a_r, dev)
    Y, out, outm, lse, csum = half(V, F), half(V, F), half(V, F), f32(V, H), f32(V, H)
    hgnn.hgnn_spmm_discretized(p, g, up(w, dev), H, Xd, Y)
    ref, sabs = oracle.spmm(rowptr, col, X, w=w, H=H, want_sabs=True)
    compare("sum", down(Y), ref, sabs)
    hgnn.hgnn_gat_forward_fused_save(g, p, H, D, Xd, Xd, ald, ard, out, lse, outm, csum)
    oref, lref, oabs, mref, cref = oracle.gat_forward(rowptr, col, X, X, a_l, a_r, H, slope=0.2, want_saved=True)
    compare("out", down(out), oref, oabs)
    compare("out_masked", down(outm), mref, oabs)
    # the pass over the transpose has the long row where the graph itself is the transpose
    o2, m2, l2, c2 = half(V, F), half(V, F), f32(V, H), f32(V, H)
    hgnn.hgnn_gat_forward_fused_save(gt, pt, H, D, Xd, Xd, ald, ard, o2, l2, m2, c2)
    got = []
    for q in (hgnn.hgnn_plan_create(back, 1, F, H, col_blocks=1), hgnn.hgnn_plan_create(back, 256, F, H, col_blocks=1)):
        dV, d_el, d_er = half(V, F), half(V, H), half(V, H)
        hgnn.hgnn_gat_backward_fused_saved(gt, pt, back, q, H, D, Xd, Xd, ald, ard, o2, l2, m2, c2, Xd, dV, d_el, d_er)
        got.append([down(t).astype(np.float64) for t in (dV, d_el, d_er)])
    for a, b in zip(*got):  # one rounding of a row against one of each of its pieces beside it
        assert np.linalg.norm(a - b) <= 2e-3 * np.linalg.norm(a)
