"""GPU parity of the dense side of a layer (projection on the matrix cores, its transposed product and weight
gradient, the GAT feature gradient) against the CPU fp64 oracle, and of a whole GAT layer chained through them."""
import numpy as np
import pytest
import torch

import oracle
from parity import compare, down, f16, rand_graph, up

pytestmark = pytest.mark.gpu


def padded(a, ld, dev, fill=0.0):
    """Device copy of a inside rows of pitch ld; returns (view of the data, whole buffer)."""
    buf = torch.full((a.shape[0], ld), fill, dtype=torch.float16, device=dev)
    buf[:, :a.shape[1]] = up(a, dev)
    return buf[:, :a.shape[1]], buf


def check_f32(name, got, ref, sabs, rel=2e-5):
    err = np.abs(got.astype(np.float64) - ref)
    bound = rel * sabs + 1e-30
    assert np.all(err <= bound), f"{name}: worst error {err.max():.3e} against bound {bound[np.argmax(err - bound)]:.3e}"


LINEAR_CASES = [  # n, K, F, transposed weight, extra pitch of X, extra pitch of Y
    (1000, 64, 64, False, 0, 0), (333, 8, 8, False, 8, 0), (1, 16, 40, False, 0, 8), (4097, 128, 128, False, 0, 0),
    (700, 608, 64, False, 0, 0), (300, 1024, 256, False, 8, 8), (5000, 64, 7, False, 0, 1), (129, 72, 36, False, 0, 4),
    (1000, 64, 64, True, 0, 0), (257, 40, 96, True, 8, 0), (300, 1024, 200, True, 0, 0), (127, 24, 2, True, 0, 6),
    (2000, 64, 300, False, 0, 4),
]


@pytest.mark.parametrize("n,K,F,trans,px,py", LINEAR_CASES)
def test_linear_shapes(hgnn, dev, n, K, F, trans, px, py):
    print(f"linear n={n} K={K} F={F} trans={trans} px={px} py={py}", flush=True)
    r = np.random.default_rng(n + 3 * K + 7 * F)
    X = f16(r.standard_normal((n, K)))
    W = f16(r.standard_normal((F, K) if trans else (K, F)) / np.sqrt(K))
    ref, sabs = oracle.linear(X, W, trans=trans, want_sabs=True)
    Xd, _ = padded(X, K + px, dev)
    ldy = (F + py + 7) // 8 * 8
    Ybuf = torch.full((n, ldy), 7.0, dtype=torch.float16, device=dev)
    Wd = up(W, dev)
    hgnn.hgnn_linear(Xd, Wd, Ybuf[:, :F], trans_w=trans)
    got = down(Ybuf)
    compare("linear", got[:, :F], ref, sabs)
    assert np.all(got[:, F:] == 7.0), "columns beyond F were touched"
    # a weight with a pitch of its own gives the same bits
    Wp = torch.zeros((W.shape[0], W.shape[1] + 5), dtype=torch.float16, device=dev)
    Wp[:, :W.shape[1]] = Wd
    Y2 = torch.full((n, ldy), 7.0, dtype=torch.float16, device=dev)
    hgnn.hgnn_linear(Xd, Wp[:, :W.shape[1]], Y2[:, :F], trans_w=trans)
    assert np.array_equal(down(Y2).view(np.uint16), got.view(np.uint16))


# rows per wave (from 32768 / 65536 rows on with K <= 64 / 32), features split over workgroups, columns in chunks
@pytest.mark.parametrize("n,K,F,trans", [(65537, 32, 40, False), (65551, 24, 8, True), (32769, 64, 72, True), (40001, 40, 42, False),
                                         (333, 608, 300, False), (97, 608, 300, True), (65, 1304, 200, False), (130, 2504, 40, True),
                                         (31, 5000, 8, False), (16385, 128, 128, False)])
def test_linear_dispatch_edges(hgnn, dev, n, K, F, trans):
    test_linear_shapes(hgnn, dev, n, K, F, trans, 0, 0)


# few rows with many columns: tiles of 16 rows per workgroup and waves that share a tile's columns change with the rows
@pytest.mark.parametrize("n,K,F,trans", [(1, 128, 2, False), (15, 136, 16, True), (17, 1280, 64, False), (31, 1288, 64, False),
                                         (8191, 608, 42, False), (8193, 504, 64, True), (12289, 256, 128, False), (16400, 504, 32, False),
                                         (20480, 960, 8, True), (20481, 640, 40, False), (32767, 136, 128, True), (32768, 648, 24, False),
                                         (32769, 128, 64, False)])
def test_linear_shared_columns(hgnn, dev, n, K, F, trans):
    test_linear_shapes(hgnn, dev, n, K, F, trans, 0, 0)


# whole and partial 16-byte pieces of the weight, twice as many waves per workgroup (8192 tiles of rows), twice as many workgroups as fit (few columns,
# many features); what lies beside and behind the operands must not be looked at
@pytest.mark.parametrize("trans", [False, True])
@pytest.mark.parametrize("n,K,F", [(3, 8, 8), (250, 72, 40), (33000, 40, 52), (131090, 72, 8), (110001, 8, 608), (20000, 168, 100), (70, 2504, 24)])
def test_linear_stays_inside(hgnn, dev, n, K, F, trans):
    print(f"linear inside n={n} K={K} F={F} trans={trans}", flush=True)
    r = np.random.default_rng(n + K + F + trans)
    X = f16(r.standard_normal((n, K)))
    X[n // 2, K // 2] = np.inf
    W = f16(r.standard_normal((F, K) if trans else (K, F)) / np.sqrt(K))
    Xb = torch.full((n + 64, K + 8), float("nan"), dtype=torch.float16, device=dev)
    Wb = torch.full((W.shape[0] + 8, (W.shape[1] + 7) // 8 * 8 + 8), float("nan"), dtype=torch.float16, device=dev)
    Xb[:n, :K], Wb[:W.shape[0], :W.shape[1]] = up(X, dev), up(W, dev)
    Yb = torch.full((n + 1, (F + 7) // 8 * 8), 7.0, dtype=torch.float16, device=dev)
    hgnn.hgnn_linear(Xb[:n, :K], Wb[:W.shape[0], :W.shape[1]], Yb[:n, :F], trans_w=trans)
    got = down(Yb)
    assert np.all(got[n] == 7.0) and np.all(got[:, F:] == 7.0)
    finite = np.arange(n) != n // 2
    assert not np.isfinite(got[n // 2, :F]).any()
    ref, sabs = oracle.linear(X[finite], W, trans=trans, want_sabs=True)
    compare("linear", got[:n][finite][:, :F], ref, sabs)


def test_linear_identity_and_zero_rows(hgnn, dev):
    n, K = 777, 96
    r = np.random.default_rng(5)
    X = f16(r.standard_normal((n, K)))
    Xd = up(X, dev)
    Y = torch.empty((n, K), dtype=torch.float16, device=dev)
    hgnn.hgnn_linear(Xd, torch.eye(K, dtype=torch.float16, device=dev), Y)
    assert np.array_equal(down(Y).view(np.uint16), X.view(np.uint16))
    # n = 0 is a no-op; bad shapes are refused on the host
    hgnn.hgnn_linear(Xd[:0], torch.eye(K, dtype=torch.float16, device=dev), Y[:0])
    with pytest.raises(hgnn.HgnnError) as e:
        hgnn.hgnn_linear(Xd[:, :20], torch.zeros((20, 8), dtype=torch.float16, device=dev), Y[:, :8])
    assert e.value.status == hgnn.HGNN_EUNSUPPORTED  # K % 8 != 0
    with pytest.raises(hgnn.HgnnError) as e:
        hgnn.hgnn_linear(Xd, torch.zeros((K, 8), dtype=torch.float16, device=dev), Y[:, :8], F=16)
    assert e.value.status == hgnn.HGNN_EINVAL  # weight pitch smaller than F


WGRAD_CASES = [(1000, 64, 64), (17, 8, 8), (50000, 64, 64), (3000, 128, 72), (100, 200, 136), (16385, 16, 256), (5, 64, 64)]


@pytest.mark.parametrize("n,K,F", WGRAD_CASES)
def test_linear_wgrad_shapes(hgnn, dev, n, K, F):
    print(f"wgrad n={n} K={K} F={F}", flush=True)
    r = np.random.default_rng(n + K + F)
    X, dY = f16(r.standard_normal((n, K))), f16(r.standard_normal((n, F)))
    ref, sabs = oracle.linear_wgrad(X, dY, want_sabs=True)
    Xd, _ = padded(X, K + 8, dev)
    dYd, _ = padded(dY, F + 16, dev)
    ws = torch.empty(hgnn.hgnn_linear_wgrad_workspace(K, F), dtype=torch.uint8, device=dev)
    dWbuf = torch.full((K, F + 3), 7.0, dtype=torch.float32, device=dev)
    hgnn.hgnn_linear_wgrad(Xd, dYd, dWbuf[:, :F], ws)
    got = down(dWbuf)
    check_f32("wgrad", got[:, :F], ref, sabs)
    assert np.all(got[:, F:] == 7.0)
    # the same bits on a second run (fixed summation order), with a dirty workspace
    ws.fill_(0xff)
    dW2 = torch.empty((K, F), dtype=torch.float32, device=dev)
    hgnn.hgnn_linear_wgrad(Xd, dYd, dW2, ws)
    assert np.array_equal(down(dW2).view(np.uint32), got[:, :F].view(np.uint32))


# one or two waves across either side of dW, partial last blocks, fewer rows than a step
@pytest.mark.parametrize("n,K,F", [(31, 72, 64), (33, 64, 72), (4097, 128, 128), (129, 136, 8), (65, 608, 64), (20000, 104, 256)])
def test_linear_wgrad_dispatch_edges(hgnn, dev, n, K, F):
    test_linear_wgrad_shapes(hgnn, dev, n, K, F)


# the one-launch form for few rows: its last row and the next, steps of 32 rows missing for some waves, partial 16-blocks
@pytest.mark.parametrize("n,K,F", [(1, 8, 8), (32, 40, 24), (511, 64, 64), (513, 56, 48), (1999, 104, 72), (2048, 128, 64),
                                   (2049, 64, 64), (2048, 640, 128), (2048, 640, 136)])
def test_linear_wgrad_few_rows(hgnn, dev, n, K, F):
    test_linear_wgrad_shapes(hgnn, dev, n, K, F)


# the most rows of one launch and one more, for every size of dW that has a limit of its own
@pytest.mark.parametrize("n", [0, 1])
@pytest.mark.parametrize("most,K,F", [(2400, 64, 16), (1700, 64, 64), (3000, 128, 128), (4096, 256, 128), (2560, 256, 256)])
def test_linear_wgrad_one_launch_or_two(hgnn, dev, most, K, F, n):
    test_linear_wgrad_shapes(hgnn, dev, most + n, K, F)


# the number of partial results and the share of a slice that adds them: one step, few and many of a workgroup, whole rounds
# of workgroups, sides that end inside a tile or block, several blocks; last lines: dW of 128 x 128 and more behind few rows
@pytest.mark.parametrize("n,K,F", [(2433, 8, 8), (2500, 24, 40), (9000, 8, 72), (9000, 72, 8), (26000, 64, 48), (60000, 16, 16), (33333, 104, 64),
                                   (30001, 128, 120), (20000, 136, 8), (9001, 504, 40), (7000, 264, 136), (3001, 608, 200),
                                   (2000, 128, 128), (3001, 128, 128), (2500, 128, 256), (4097, 128, 256), (3001, 256, 256)])
def test_linear_wgrad_partials(hgnn, dev, n, K, F):
    test_linear_wgrad_shapes(hgnn, dev, n, K, F)


# steps of a workgroup that are added up in runs, for one and two waves across either side: some, many, the last run shorter
@pytest.mark.parametrize("n,K,F", [(450000, 8, 8), (300001, 40, 24), (20000, 64, 200), (5000, 504, 64), (7001, 264, 40), (3500, 256, 256), (90001, 72, 72)])
def test_linear_wgrad_runs(hgnn, dev, n, K, F):
    test_linear_wgrad_shapes(hgnn, dev, n, K, F)


@pytest.mark.parametrize("n,K,F,runs,partials", [(233000, 608, 64, 5, 96), (500000, 128, 128, 4, 512), (600000, 608, 128, 25, 96)])
def test_linear_wgrad_error_of_long_sums(hgnn, dev, n, K, F, runs, partials):
    """The error against 64 bits over many rows.  The k-th of r equal additions rounds to 2^-24 / sqrt(3) of its sum in the mean, whose square is k / r of
    the result's, so a chain leaves 2^-24 / sqrt(3) * sqrt(r / 2).  A product of 32 rows rounds some four times, eight of them follow each other; then
    the runs, a sixteenth of the partial results, and 16 sums of those.  One chain over all rows of a workgroup had 2.4 to 6.2e-7."""
    gen = torch.Generator(device=dev).manual_seed(n)
    X, dY = (torch.randn((n, c), generator=gen, device=dev, dtype=torch.float16) for c in (K, F))
    dW = torch.empty((K, F), dtype=torch.float32, device=dev)
    hgnn.hgnn_linear_wgrad(X, dY, dW, torch.empty(hgnn.hgnn_linear_wgrad_workspace(K, F), dtype=torch.uint8, device=dev))
    ref = sum(X[i:i + 50000].double().T.contiguous() @ dY[i:i + 50000].double() for i in range(0, n, 50000))
    rel = float((dW.double() - ref).norm() / ref.norm())
    print(f"wgrad n={n} K={K} F={F}: relative error {rel:.2e}", flush=True)
    assert rel <= 2.0 ** -24 / 3 ** 0.5 * (4 * 8 / 2 + runs / 2 + partials / 16 / 2 + 16 / 2) ** 0.5


def test_linear_wgrad_errors(hgnn, dev):
    X = torch.zeros((64, 64), dtype=torch.float16, device=dev)
    dW = torch.zeros((64, 64), dtype=torch.float32, device=dev)
    small = torch.empty(1024, dtype=torch.uint8, device=dev)
    with pytest.raises(hgnn.HgnnError) as e:
        hgnn.hgnn_linear_wgrad(X, X, dW, small)
    assert e.value.status == hgnn.HGNN_EINVAL and "workspace" in str(e.value)
    # no rows: the gradient is zero
    ws = torch.empty(hgnn.hgnn_linear_wgrad_workspace(64, 64), dtype=torch.uint8, device=dev)
    dW.fill_(5.0)
    hgnn.hgnn_linear_wgrad(X[:0], X[:0], dW, ws)
    assert np.all(down(dW) == 0)


@pytest.mark.parametrize("n,H,D", [(1000, 1, 64), (333, 4, 16), (5000, 3, 8), (64, 8, 64), (40000, 1, 8), (257, 2, 128)])
def test_gat_feature_grad_shapes(hgnn, dev, n, H, D):
    print(f"feature grad n={n} H={H} D={D}", flush=True)
    F = H * D
    r = np.random.default_rng(n + H + D)
    dV, hfeat = f16(r.standard_normal((n, F))), f16(r.standard_normal((n, F)))
    d_el, d_er = f16(0.3 * r.standard_normal((n, H))), f16(0.3 * r.standard_normal((n, H)))
    a_l, a_r = f16(0.5 * r.standard_normal(F)), f16(0.5 * r.standard_normal(F))
    dh_ref, dal_ref, dar_ref, sl, sr = oracle.gat_feature_grad(dV, d_el, d_er, a_l, a_r, hfeat, H)
    mag = (np.abs(dV.astype(np.float64)) + np.abs(np.repeat(d_el.astype(np.float64), D, 1) * a_l.astype(np.float64)) +
           np.abs(np.repeat(d_er.astype(np.float64), D, 1) * a_r.astype(np.float64)))
    dVd, _ = padded(dV, F + 8, dev)
    hd, _ = padded(hfeat, F + 16, dev)
    dhbuf = torch.full((n, F + 8), 7.0, dtype=torch.float16, device=dev)
    da_l = torch.full((F,), 7.0, dtype=torch.float32, device=dev)
    da_r = torch.full((F,), 7.0, dtype=torch.float32, device=dev)
    ws = torch.empty(hgnn.hgnn_gat_feature_grad_workspace(H, D), dtype=torch.uint8, device=dev)
    ws.fill_(0xff)
    hgnn.hgnn_gat_feature_grad(H, D, dVd, up(d_el, dev), up(d_er, dev), up(a_l, dev), up(a_r, dev), hd, dhbuf[:, :F],
                               da_l, da_r, ws)
    got = down(dhbuf)
    compare("dh", got[:, :F], dh_ref, mag)
    assert np.all(got[:, F:] == 7.0)
    check_f32("da_l", down(da_l), dal_ref, sl)
    check_f32("da_r", down(da_r), dar_ref, sr)


def test_gat_layer_forward_and_backward_chain(hgnn, dev):
    """h = X W; out = GAT aggregation of (h, h); then every gradient of L = <dOut, out>.  The oracle chain rounds to
    fp16 where the device stores fp16 (h, dV, d_el, d_er, dh) and nowhere else."""
    V, K, H, D = 1500, 40, 2, 16
    F = H * D
    rowptr, col = rand_graph(V, V, 9, 123, hubs=((3, 2500), (900, 400)), empties=(0, 77))
    r = np.random.default_rng(9)
    X = f16(r.standard_normal((V, K)))
    W = f16(r.standard_normal((K, F)) / np.sqrt(K))
    a_l, a_r = f16(0.3 * r.standard_normal(F)), f16(0.3 * r.standard_normal(F))
    dOut = f16(r.standard_normal((V, F)))
    # ---- oracle chain
    h64, h_sabs = oracle.linear(X, W, want_sabs=True)
    h16 = h64.astype(np.float16)
    out_ref, lse_ref, out_sabs = oracle.gat_forward(rowptr, col, h16, h16, a_l, a_r, H)
    dV_ref, del_ref, der_ref = oracle.gat_backward(rowptr, col, h16, h16, a_l, a_r, dOut, H)
    dh_ref, dal_ref, dar_ref, sl, sr = oracle.gat_feature_grad(dV_ref.astype(np.float16), del_ref.astype(np.float16),
                                                               der_ref.astype(np.float16), a_l, a_r, h16, H)
    dh16 = dh_ref.astype(np.float16)
    dX_ref, dX_sabs = oracle.linear(dh16, W, trans=True, want_sabs=True)
    dW_ref, dW_sabs = oracle.linear_wgrad(X, dh16, want_sabs=True)
    # ---- device chain
    g = hgnn.Csr(up(rowptr, dev), up(col, dev))
    p = hgnn.hgnn_plan_create(g, 128, F, H)
    gt = hgnn.hgnn_transpose(g)
    pt = hgnn.hgnn_plan_create(gt, 128, F, H)
    Xd, Wd, ald, ard, dOutd = up(X, dev), up(W, dev), up(a_l, dev), up(a_r, dev), up(dOut, dev)
    half = lambda *s: torch.empty(s, dtype=torch.float16, device=dev)
    h, out, dV, d_el, d_er, dh, dX = half(V, F), half(V, F), half(V, F), half(V, H), half(V, H), half(V, F), half(V, K)
    lse = torch.empty((V, H), dtype=torch.float32, device=dev)
    dW = torch.empty((K, F), dtype=torch.float32, device=dev)
    da_l, da_r = torch.empty(F, dtype=torch.float32, device=dev), torch.empty(F, dtype=torch.float32, device=dev)
    ws = torch.empty(max(hgnn.hgnn_linear_wgrad_workspace(K, F), hgnn.hgnn_gat_feature_grad_workspace(H, D)),
                     dtype=torch.uint8, device=dev)
    hgnn.hgnn_linear(Xd, Wd, h)
    hgnn.hgnn_gat_forward_fused(g, p, H, D, h, h, ald, ard, out, lse)
    hgnn.hgnn_gat_backward_fused(g, p, gt, pt, H, D, h, h, ald, ard, out, lse, dOutd, dV, d_el, d_er)
    hgnn.hgnn_gat_feature_grad(H, D, dV, d_el, d_er, ald, ard, h, dh, da_l, da_r, ws)
    hgnn.hgnn_linear(dh, Wd, dX, trans_w=True)
    hgnn.hgnn_linear_wgrad(Xd, dh, dW, ws)
    compare("layer h", down(h), h64, h_sabs)
    compare("layer out", down(out), out_ref, out_sabs)
    # gradients: the device's own fp16 intermediates differ from the oracle's by a rounding each, which the
    # cancelling sums behind d_el / d_er amplify; rel-L2 bands as for the fused backward on its own
    rel = lambda a, b: np.linalg.norm(a.astype(np.float64) - b) / np.linalg.norm(b)
    assert rel(down(dh), dh_ref) < 5e-3
    assert rel(down(dX), dX_ref) < 5e-3
    assert rel(down(dW), dW_ref) < 5e-3
    assert rel(down(da_l), dal_ref) < 2e-2 and rel(down(da_r), dar_ref) < 2e-2
    hgnn.hgnn_plan_destroy(p)
    hgnn.hgnn_plan_destroy(pt)


def test_dense_at_dense_degree_size(hgnn, dev):
    """The projection and the weight gradient at the vertex count and width of the dense-degree workload
    (233 000 x 64 -> 64): sampled rows of Y, the whole of dW."""
    n, K, F = 233000, 64, 64
    r = np.random.default_rng(2024)
    X = f16(r.standard_normal((n, K)))
    W = f16(r.standard_normal((K, F)) / 8)
    G = f16(r.standard_normal((n, F)))
    Xd, Gd, Wd = up(X, dev), up(G, dev), up(W, dev)
    Y = torch.empty((n, F), dtype=torch.float16, device=dev)
    hgnn.hgnn_linear(Xd, Wd, Y)
    rows = np.unique(np.concatenate([r.integers(0, n, 4000), [0, 127, 128, n - 129, n - 1]]))
    ref, sabs = oracle.linear(X[rows], W, want_sabs=True)
    compare("linear full", down(Y)[rows], ref, sabs)
    ws = torch.empty(hgnn.hgnn_linear_wgrad_workspace(K, F), dtype=torch.uint8, device=dev)
    dW = torch.empty((K, F), dtype=torch.float32, device=dev)
    hgnn.hgnn_linear_wgrad(Xd, Gd, dW, ws)
    dref, dsabs = oracle.linear_wgrad(X, G, want_sabs=True)
    check_f32("wgrad full", down(dW), dref, dsabs)


@pytest.mark.parametrize("K,KW,F", [(104, 100, 256), (48, 42, 128), (104, 97, 8), (640, 601, 200)])
def test_linear_weight_of_fewer_rows(hgnn, dev, K, KW, F):
    """X padded to K columns, W of KW rows: what lies behind W in memory is not read."""
    n = 700
    r = np.random.default_rng(K + F)
    Xh = np.zeros((n, K), dtype=np.float16)
    Xh[:, :KW] = f16(r.standard_normal((n, KW)))
    Wh = f16(r.standard_normal((KW, F)))
    buf = torch.full((K + 8, F), float("nan"), dtype=torch.float16, device=dev)
    buf[:KW] = up(Wh, dev)
    Y = torch.empty((n, F), dtype=torch.float16, device=dev)
    hgnn.hgnn_linear(up(Xh, dev), buf[:KW], Y)
    ref, sabs = oracle.linear(np.ascontiguousarray(Xh[:, :KW]), Wh, want_sabs=True)
    compare("linear, W of fewer rows", down(Y), ref, sabs)


# W that begins at any element, lines of any pitch, the last piece of a line whole, ragged or all there is (fewer than eight features), columns in chunks,
# columns shared by waves, fewer rows than columns of X; NaN between the lines and around them
@pytest.mark.parametrize("n,K,KW,F,trans,ldw,first", [
    (100, 64, 64, 8, False, 9, 1), (100, 64, 64, 9, False, 9, 0), (300, 64, 64, 42, False, 48, 0), (300, 64, 64, 42, False, 43, 3), (33, 40, 40, 15, False, 16, 8),
    (300, 24, 24, 7, False, 8, 0), (300, 72, 70, 1, False, 3, 5), (300, 72, 65, 3, False, 8, 0), (1000, 504, 504, 47, False, 47, 2), (400, 128, 121, 100, False, 104, 0),
    (2000, 608, 608, 300, False, 301, 1), (90, 2504, 2500, 41, False, 48, 0), (90, 2504, 2504, 41, False, 41, 7), (40, 1304, 1304, 130, False, 131, 1),
    (300, 64, 64, 42, True, 67, 0), (300, 24, 24, 5, True, 25, 3), (1000, 504, 504, 100, True, 505, 1), (90, 2504, 2504, 41, True, 2507, 5)])
def test_linear_weight_from_any_element(hgnn, dev, n, K, KW, F, trans, ldw, first):
    print(f"linear any n={n} K={K} KW={KW} F={F} trans={trans} ldw={ldw} first={first}", flush=True)
    r = np.random.default_rng(n + K + F + ldw)
    X = f16(r.standard_normal((n, K)))
    X[:, KW:] = 0
    W = f16(r.standard_normal((F, K) if trans else (KW, F)) / np.sqrt(K))
    flat = torch.full((first + W.shape[0] * ldw + 64,), float("nan"), dtype=torch.float16, device=dev)
    Wd = flat.as_strided(W.shape, (ldw, 1), first)
    Wd.copy_(up(W, dev))
    Y = torch.full((n + 1, (F + 7) // 8 * 8), 7.0, dtype=torch.float16, device=dev)
    hgnn.hgnn_linear(up(X, dev), Wd, Y[:n, :F], trans_w=trans)
    got = down(Y)
    assert np.all(got[n] == 7.0) and np.all(got[:, F:] == 7.0)
    ref, sabs = oracle.linear(np.ascontiguousarray(X[:, :KW]), W, trans=trans, want_sabs=True)
    compare("linear", got[:n, :F], ref, sabs)
    pad = torch.zeros((W.shape[0], (W.shape[1] + 7) // 8 * 8), dtype=torch.float16, device=dev)  # the same from aligned lines: the same bits
    pad[:, :W.shape[1]] = up(W, dev)
    Y2 = torch.full_like(Y, 7.0)
    hgnn.hgnn_linear(up(X, dev), pad[:, :W.shape[1]], Y2[:n, :F], trans_w=trans)
    assert np.array_equal(down(Y2).view(np.uint16), got.view(np.uint16))


# W^T of up to 32 columns: 16 features of four pieces at a time; one to twenty of them for one to sixteen waves
@pytest.mark.parametrize("n,K,F", [(40, 8, 1), (300, 32, 17), (4100, 24, 33), (20000, 16, 128), (70, 8, 256), (500, 32, 602), (70000, 8, 100)])
def test_linear_transposed_weight_of_few_columns(hgnn, dev, n, K, F):
    test_linear_stays_inside(hgnn, dev, n, K, F, True)


@pytest.mark.parametrize("n,K,F,ldw,trans", [(4096, 64, 42, 48, False), (4096, 64, 42, 42, False), (3000, 2504, 41, 48, False), (4096, 64, 41, 67, True),
                                             (60000, 608, 52, 56, False)])
def test_linear_ragged_weight_costs_as_much_as_a_whole_one(hgnn, dev, n, K, F, ldw, trans):
    """A weight with a ragged end or lines that begin anywhere takes no time of another order: at most 1.5 times that of the same with the features
    filled up (read by elements it was 1.8 to 2.6 times)."""
    X = torch.randn((n, K), device=dev).half()
    up8 = (F + 7) // 8 * 8
    Y = torch.empty((n, up8), dtype=torch.float16, device=dev)

    def time_of(W, f):
        hgnn.hgnn_linear(X, W, Y[:, :f], trans_w=trans)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for _ in range(20):
                hgnn.hgnn_linear(X, W, Y[:, :f], trans_w=trans)
        best = float("inf")
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            g.replay()
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    rows, cols = (F, K) if trans else (K, F)
    ragged = torch.randn((rows, ldw), device=dev).half()[:, :cols]
    whole = torch.randn((up8, K) if trans else (K, up8), device=dev).half()
    assert time_of(ragged, F) <= 1.5 * time_of(whole, up8)
