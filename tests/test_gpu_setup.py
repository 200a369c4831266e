"""Set-up calls at the edges of their dispatch: edge lists and transposes whose fields do and do not fit one 64-bit sort key,
row lists of every kind, graphs rejected by each rule, and the memory that set-up calls keep for one another."""
import threading
import time

import numpy as np
import pytest
import torch

from parity import up

pytestmark = pytest.mark.gpu


def down(t):
    return t.cpu().numpy()


def check_lists(hgnn, dev, V, row, col):
    E = row.size
    g, eid = hgnn.hgnn_coo_to_csr(up(row, dev), up(col, dev), V, V)
    order = np.lexsort((np.arange(E), col, row))
    assert np.array_equal(down(eid), order) and np.array_equal(down(g.col), col[order])
    rowptr = np.searchsorted(row[order], np.arange(V + 1))
    assert np.array_equal(down(g.rowptr), rowptr)
    h, none = hgnn.hgnn_coo_to_csr(up(row, dev), up(col, dev), V, V, want_eid=False)
    assert none is None and torch.equal(h.col, g.col) and torch.equal(h.rowptr, g.rowptr)
    gt = hgnn.hgnn_transpose(g)
    t = np.argsort(col[order], kind="stable")
    assert np.array_equal(down(gt.eid), t) and np.array_equal(down(gt.col), row[order][t])
    assert np.array_equal(down(gt.rowptr), np.searchsorted(col[order][t], np.arange(V + 1)))
    return g, gt


# 2^25 vertices and 2^15 edges: 65 bits for row, column and position; with 2^24 vertices they fit
@pytest.mark.parametrize("V,E", [(1, 1), (3, 2047), (5, 2049), (1000, 4096), (40000, 100001), (1 << 24, 1 << 14), ((1 << 24) + 1, (1 << 15) + 1)])
def test_sort_keys(hgnn, dev, V, E):
    print(f"setup V={V} E={E}", flush=True)
    r = np.random.default_rng(V + E)
    row, col = (r.integers(0, V, E).astype(np.int32) for _ in range(2))
    row[: E // 3] = row[0]  # a hub, and duplicates
    col[: E // 8] = col[0]
    check_lists(hgnn, dev, V, row, col)


# tiles of 8192 words at most, few tiles add up their counts themselves; digits of 1 to 9 bits
@pytest.mark.parametrize("V,E", [(2, 8191), (512, 8192), (513, 8193), (1 << 18, 64 * 8192), ((1 << 18) + 1, 64 * 8192 + 1), (37, 600000),
                                 (1 << 20, 1200000)])
def test_sort_tiles(hgnn, dev, V, E):
    print(f"setup tiles V={V} E={E}", flush=True)
    r = np.random.default_rng(V + E)
    row, col = (r.integers(0, V, E).astype(np.int32) for _ in range(2))
    row[E // 2:E // 2 + E // 5] = V - 1  # a hub in the last row, long stretches of empty rows beside it
    row[row > V * 3 // 4] = V - 1
    col[: E // 8] = col[0]
    check_lists(hgnn, dev, V, row, col)


# two, four and eight words a thread, counts added up by the tiles or scanned, with each number of words; one, two and four passes
@pytest.mark.parametrize("E", [128 * 2048, 128 * 2048 + 1, 256 * 2048, 256 * 2048 + 1, 256 * 4096, 256 * 4096 + 1])
@pytest.mark.parametrize("V", [20, 511, 70000])
def test_sort_items_of_a_thread(hgnn, dev, V, E):
    test_sort_tiles(hgnn, dev, V, E)


@pytest.mark.parametrize("V,E", [(70000, 256 * 6144), (70000, 256 * 6144 + 1), (511, 256 * 8192), (511, 256 * 8192 + 1), (70000, 512 * 6144),
                                 (300000, 512 * 6144 - 6143), (20, 512 * 6144 + 1)])
def test_sort_six_items_of_a_thread(hgnn, dev, V, E):
    test_sort_tiles(hgnn, dev, V, E)


@pytest.mark.parametrize("E", [3072 * 8192, 3072 * 8192 + 1])
def test_many_tiles(hgnn, dev, E):
    """The counts of up to 3072 tiles are scanned in one, of more in shares."""
    V = 100003
    print(f"setup E={E}", flush=True)
    gen = torch.Generator(device=dev).manual_seed(E)
    row, col = (torch.randint(0, V, (E,), generator=gen, device=dev, dtype=torch.int32) for _ in range(2))
    row[E // 2:E // 2 + E // 5] = 3
    g, eid = hgnn.hgnn_coo_to_csr(row, col, V, V)
    key, order = torch.sort(row.long() * V + col, stable=True)
    assert torch.equal(eid.long(), order) and torch.equal(g.col.long(), key % V)
    bounds = torch.arange(V + 1, device=dev)
    assert torch.equal(g.rowptr.long(), torch.searchsorted(key // V, bounds))
    gt = hgnn.hgnn_transpose(g)
    c, t = torch.sort(g.col.long(), stable=True)
    assert torch.equal(gt.eid.long(), t) and torch.equal(gt.col.long(), (key // V)[t]) and torch.equal(gt.rowptr.long(), torch.searchsorted(c, bounds))


# up to 2048 words in one launch, up to 8192 in another form of it, up to eight tiles of those merged where a pass is not enough
@pytest.mark.parametrize("E", [1, 63, 1025, 2047, 2048, 2049, 8191, 8193, 16384, 16385, 32768, 32769, 65536, 65537])
@pytest.mark.parametrize("V", [1, 300, 513, 70000, 1 << 20])
def test_sort_few_words(hgnn, dev, V, E):
    print(f"setup few words V={V} E={E}", flush=True)
    r = np.random.default_rng(V + E)
    row, col = (r.integers(0, V, E).astype(np.int32) for _ in range(2))
    row[E // 2:E // 2 + E // 5] = V - 1
    col[: E // 8] = col[0]
    row[E // 3:E // 3 + 9], col[E // 3:E // 3 + 9] = V // 2, V // 3  # one edge several times
    check_lists(hgnn, dev, V, row, col)


# long stretches of empty rows and columns, by the number of words to an offset: written where they are found, from 65537 offsets on but for
# windows of 1024; with few words all offsets by search, with many words to a window too
@pytest.mark.parametrize("V,E", [(23000, 3000), (24008, 3000), (24009, 3000), (65536, 9000), (65537, 9000), (66559, 9000), (66560, 9000), (66561, 9000),
                                 (1 << 20, 300000), (5000011, 3000), (5000011, 625001), (5000011, 625002), (100000, 1600000), (100001, 1600000)])
def test_long_gaps(hgnn, dev, V, E):
    print(f"setup gaps V={V} E={E}", flush=True)
    r = np.random.default_rng(V)
    some = [0, 1, 1022, 1023, 1024, 1025, 2047, 2048, 3071, 5000, 20959, V - 1025, V - 1024, V - 2, V - 1]
    for ids in ([V // 2], [0], [V - 1], [1023], [1024], some, some[1:-1])[: 7 if E < 10000 else 1 if E < 1000000 else 6]:
        row = np.array(ids, dtype=np.int32)[r.integers(0, len(ids), E)]
        check_lists(hgnn, dev, V, row, r.permutation(row))


def test_time_of_a_long_gap(hgnn, dev):
    """All edges at one vertex of many: the offsets of the others are written by many workgroups (one took six times as long as a uniform list)."""
    V, E = 1 << 25, 4000000
    best = {}
    for what in ("uniform", "one"):
        r = np.random.default_rng(1)
        row, col = (up(r.integers(0, V, E).astype(np.int32), dev) for _ in range(2))
        if what == "one":
            row.fill_(V // 2)
        best[what] = 1e9
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            hgnn.hgnn_coo_to_csr(row, col, V, V, want_eid=False)
            best[what] = min(best[what], time.perf_counter() - t)
    assert best["one"] <= 3 * best["uniform"], best


def test_time_of_few_words(hgnn, dev):
    """Few words over many vertices: a few launches and no loop over the stretches between them (twice as long as this many)."""
    V, E = 100000, 1000
    r = np.random.default_rng(1)
    row, col = (up(r.integers(0, V, E).astype(np.int32), dev) for _ in range(2))
    best = {}
    for v in (V, 1 << 16):
        best[v] = 1e9
        for _ in range(30):
            torch.cuda.synchronize()
            t = time.perf_counter()
            hgnn.hgnn_coo_to_csr(row % v, col % v, v, v)
            best[v] = min(best[v], time.perf_counter() - t)
    assert best[V] < 80e-6, best


@pytest.mark.parametrize("E", [1, 8193, 700000])
def test_ids_out_of_range(hgnn, dev, E):
    V = 1000
    r = np.random.default_rng(E)
    for which, bad in ((0, -1), (0, V), (1, -5), (1, 1 << 30)):
        ids = [r.integers(0, V, E).astype(np.int32) for _ in range(2)]
        ids[which][E - 1] = bad
        with pytest.raises(hgnn.HgnnError) as e:
            hgnn.hgnn_coo_to_csr(up(ids[0], dev), up(ids[1], dev), V, V)
        assert "outside" in str(e.value)
        ids[which][E - 1] = 0
        check_lists(hgnn, dev, V, ids[0], ids[1])


def test_plan_lists(hgnn, dev):
    """Rows shorter and longer than every threshold of a plan, empty rows between them."""
    r = np.random.default_rng(3)
    deg = np.concatenate([r.integers(0, 40, 3000), [31, 32, 33, 2047, 2048, 2049, 4096, 4097, 9000], np.zeros(1500, int), [1, 300, 5000]])
    V = deg.size
    row = np.repeat(np.arange(V, dtype=np.int32), deg)
    col = r.integers(0, V, row.size).astype(np.int32)
    g, gt = check_lists(hgnn, dev, V, row, col)
    for S in (64, 256, 1000):
        p = hgnn.hgnn_plan_create(g, S, 64, 1)
        x = hgnn.hgnn_plan_export(p)
        rowptr = down(g.rowptr).astype(np.int64)
        b, e = rowptr[:-1], rowptr[1:]
        split = np.flatnonzero((e > b) & (b // S != (e - 1) // S))
        assert np.array_equal(x["split_row"], split)
        assert np.array_equal(x["split_seg_lo"], b[split] // S) and np.array_equal(x["split_seg_hi"], (e[split] - 1) // S)


@pytest.mark.parametrize("rule", range(8))
def test_validation_rules(hgnn, dev, rule):
    V, E = 3000, 20000
    r = np.random.default_rng(rule)
    rowptr = np.sort(np.concatenate([[0, E], r.integers(0, E + 1, V - 1)])).astype(np.int32)
    col = np.concatenate([np.sort(r.integers(0, V, n)) for n in np.diff(rowptr)]).astype(np.int32)
    row, eid = np.repeat(np.arange(V), np.diff(rowptr)).astype(np.int32), r.permutation(E).astype(np.int32)
    k = int(rowptr[np.argmax(np.diff(rowptr))])  # inside the longest row
    if rule == 1:
        rowptr[0] = 1
    elif rule == 2:
        rowptr[-1] = E - 1
    elif rule == 3:
        rowptr[V // 2] = rowptr[V // 2 + 1] + 1
    elif rule == 4:
        col[k] = V
    elif rule == 5:
        eid[k] = -1
    elif rule == 6:
        row[k] += 1
    elif rule == 7:
        col[k], col[k + 1] = V - 1, 0
    g = hgnn.Csr(up(rowptr, dev), up(col, dev), row=up(row, dev), eid=up(eid, dev))
    words = [None, "rowptr[0]", "rowptr[nrows]", "decreases", "column id", "edge id", "COO row id", "ascending"]
    for call in (lambda: hgnn.hgnn_csr_validate(g), lambda: hgnn.hgnn_plan_create(g, 256, 8, 1)):
        if rule == 0:
            call()
            continue
        with pytest.raises(hgnn.HgnnError) as err:
            call()
        assert err.value.status == hgnn.HGNN_EINVAL and words[rule] in str(err.value)


def test_kept_memory(hgnn, dev):
    """Plans made and destroyed by several threads on streams of their own get memory of earlier ones and stay correct."""
    V, E = 2000, 30000
    r = np.random.default_rng(9)
    lists = [(up(r.integers(0, V, E).astype(np.int32), dev), up(r.integers(0, V, E).astype(np.int32), dev)) for _ in range(3)]
    X = torch.randn((V, 64), device=dev).half()
    want = []
    for row, col in lists:
        A = torch.zeros((V, V), device=dev)
        A.index_put_((row.long(), col.long()), torch.ones(E, device=dev), accumulate=True)
        want.append(A @ X.float())
    torch.cuda.synchronize()
    wrong = []

    def work(i):
        torch.cuda.set_device(dev)
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for k in range(6):
                row, col = lists[(i + k) % 3]
                g = hgnn.hgnn_coo_to_csr(row, col, V, V, want_eid=False)[0]
                p = hgnn.hgnn_plan_create(g, 64, 64, 1)
                Y = torch.empty_like(X)
                hgnn.hgnn_spmm_discretized(p, g, None, 1, X, Y)
                del p
                s.synchronize()
                if (Y.float() - want[(i + k) % 3]).abs().max() > 0.05:
                    wrong.append((i, k))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
    hgnn.hgnn_release_cached_memory()
    hgnn.hgnn_release_cached_memory()
    work(0)
    assert not wrong


@pytest.mark.parametrize("wide", [False, True])  # one sort key of all fields, or two arrays
@pytest.mark.parametrize("what", ["ends early", "ends late", "begins late", "falls", "negative", "all past the end"])
def test_transpose_of_a_malformed_offset_array(hgnn, dev, what, wide):
    """Transposition may come before validation: it stays inside its arrays whatever the offsets are.  The order of the columns
    does not depend on them."""
    print(f"transpose {what} wide={wide}", flush=True)
    V, E = ((1 << 24) + 1, (1 << 15) + 1) if wide else (700, 5000)
    r = np.random.default_rng(E)
    rowptr = np.sort(r.integers(0, E + 1, V + 1)).astype(np.int32)
    rowptr[0], rowptr[-1] = 0, E
    col = r.integers(0, V, E).astype(np.int32)
    if what == "ends early":
        rowptr = np.minimum(rowptr, E - 4500)
    elif what == "ends late":
        rowptr[-1] = E + 100000
    elif what == "begins late":
        rowptr = np.maximum(rowptr, 3000)
    elif what == "falls":
        rowptr[V // 3], rowptr[V // 2] = E, 0
    elif what == "negative":
        rowptr[V // 4:V // 2] = -(1 << 31)
    elif what == "all past the end":
        rowptr[:] = (1 << 31) - 1
    pad = 64
    out = [torch.full((n + 2 * pad,), -7, dtype=torch.int32, device=dev) for n in (V + 1, E, E)]
    g = hgnn.Csr(up(rowptr, dev), up(col, dev))
    from paper_2411_01109_amd import binding
    st = hgnn.load().hgnn_transpose(g.ref, *(o[pad:].data_ptr() for o in out), binding._stream(None))
    assert st == hgnn.HGNN_OK
    for o in out:
        assert (o[:pad] == -7).all() and (o[-pad:] == -7).all()
    t = np.argsort(col, kind="stable")
    assert np.array_equal(down(out[2][pad:-pad]), t)
    assert np.array_equal(down(out[0][pad:-pad]), np.searchsorted(col[t], np.arange(V + 1)))
    with pytest.raises(hgnn.HgnnError):
        hgnn.hgnn_csr_validate(g)


@pytest.mark.parametrize("ncols,mapped", [(100003, False), (100003, True), (233001, True)])
def test_export_of_automatic_blocks(hgnn, dev, ncols, mapped):
    """The plan keeps the finer cut alone where every pass walks it; the exported blocks are those of the coarse cut, whose borders
    the finer one need not have."""
    V, S = 5000, 256
    r = np.random.default_rng(ncols)
    rowptr = np.concatenate([[0], np.cumsum(r.integers(200, 900, V))]).astype(np.int32)
    E = int(rowptr[-1])
    row = np.repeat(np.arange(V), np.diff(rowptr))
    col = r.integers(0, ncols, E)
    col = col[np.lexsort((col, row))].astype(np.int32)
    eid = r.permutation(E).astype(np.int32) if mapped else None
    g = hgnn.Csr(up(rowptr, dev), up(col, dev), ncols=ncols, eid=None if eid is None else up(eid, dev))
    p = hgnn.hgnn_plan_create(g, S, 64, 1, col_blocks=0)
    nb = hgnn.hgnn_plan_col_blocks(p)
    assert nb >= 2 and hgnn.hgnn_plan_col_blocks_fine(p) == 2 * nb
    width = -(-ncols // nb)
    for b in range(nb):
        x = hgnn.hgnn_plan_block_export(p, b)
        at = np.flatnonzero((col >= b * width) & (col < (b + 1) * width))
        assert np.array_equal(x["col"], col[at]) and np.array_equal(x["eid"], eid[at] if mapped else at)
        rp = np.concatenate([[0], np.cumsum(np.bincount(row[at], minlength=V))])
        assert np.array_equal(x["rowptr"], rp)
        first = np.arange(0, at.size, S)
        assert np.array_equal(x["seg_row_lo"], row[at][first])
        assert np.array_equal(x["seg_row_hi"], row[at][np.minimum(first + S, at.size) - 1])
    with pytest.raises(hgnn.HgnnError):
        hgnn.hgnn_plan_block_export(p, nb)
    hgnn.hgnn_plan_destroy(p)
