"""The work that a user of hgnn has it do, as cases that can be timed and compared: whole graph layers through the public entry
points (projection, aggregation and every gradient), the attention layer as separate calls on edge tensors, inference, the SpMM
without a plan, and the set-up of a graph from an edge list.  Sizes are those of the repository's five configurations, and generic
odd ones; graphs are uniform (one self-loop per vertex), R-MAT (power law) or with log-normal row lengths (dense degree)."""
import math

import torch

import paper_2411_01109_amd as hgnn

SLOPE = 0.2
HALF = torch.float16


def listed():
    return [
        # the smallest training step: a GCN layer on a small citation-sized graph, where the launches and the host path count
        {"name": "gcn_tiny", "kind": "gcn", "graph": "uniform", "V": 4096, "E": 36864, "K": 64, "F": 64, "norm": "values"},
        # a GCN's last layer: class scores (42 wide in rows of 48 halves), odd vertex count, norms from the degrees
        {"name": "gcn_classes", "kind": "gcn", "graph": "rmat", "V": 100003, "E": 1300001, "K": 64, "F": 42, "norm": "degrees"},
        # a large sparse GCN: a product graph whose feature table is beyond every cache, normalised weights kept as edge values
        {"name": "gcn_large", "kind": "gcn", "graph": "rmat", "V": 2400000, "E": 62000000, "K": 128, "F": 128, "norm": "values"},
        # GIN in its overflow-safe form on a power-law graph: (1 + eps) x + lambda mean, then the first layer of its MLP
        {"name": "gin_rmat", "kind": "gin", "graph": "rmat", "V": 131072, "E": 2097152, "K": 128, "F": 128},
        # the same on a social graph of high degree (hundreds of neighbours a vertex)
        {"name": "gin_dense", "kind": "gin", "graph": "lognormal", "V": 233000, "E": 114000000, "K": 64, "F": 64},
        # a GAT layer of four heads, trained with the single-pass aggregation
        {"name": "gat_rmat", "kind": "gat", "graph": "rmat", "V": 262144, "E": 5505024, "K": 64, "H": 4, "D": 16, "train": True},
        # a GAT's first layer on the high-degree graph: wide input features (602, padded to 608), one head of 64
        {"name": "gat_dense", "kind": "gat", "graph": "lognormal", "V": 233000, "E": 114000000, "K": 608, "H": 1, "D": 64, "train": True},
        # inference of a GAT layer with eight heads of eight on a graph of odd size: forward only
        {"name": "gat_infer", "kind": "gat", "graph": "uniform", "V": 19717, "E": 108365, "K": 504, "H": 8, "D": 8, "train": False},
        # the attention layer as separate calls, the scores and weights kept as edge tensors: what a framework's autograd does
        {"name": "calls_rmat", "kind": "calls", "graph": "rmat", "V": 262144, "E": 5505024, "H": 4, "D": 16},
        {"name": "calls_dense", "kind": "calls", "graph": "lognormal", "V": 233000, "E": 114000000, "H": 1, "D": 64},
        # the SpMM without a plan, forward and backward through the transposed graph's edge-id map
        {"name": "spmm_plain", "kind": "plain", "graph": "rmat", "V": 1200001, "E": 31000001, "F": 64},
        # a graph's set-up from an edge list, both directions with their plans: paid once for a static graph, per batch for sampled ones
        {"name": "setup", "kind": "setup", "graph": "rmat", "V": 262144, "E": 5505024, "F": 64},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: vertices and mean degree over their logarithms, widths from the ones in use (ragged ones among them);
    non-zeros x width stays below half of the largest listed case's."""
    kind = rng.choice(("gcn", "gin", "gat", "calls", "plain", "setup"))
    c = {"kind": kind, "graph": rng.choice(("uniform", "rmat", "rmat", "lognormal"))}
    c["V"] = _log(rng, 2000, 2400000)
    if kind in ("gat", "calls"):
        c["H"], c["D"] = rng.choice(((1, 64), (1, 32), (1, 128), (4, 16), (8, 8), (2, 32), (4, 32)))
        F = c["H"] * c["D"]
    else:
        F = c["F"] = rng.choice((16, 32, 42, 48, 64, 64, 100, 128, 128, 256))
    if kind in ("gcn", "gin", "gat"):
        c["K"] = rng.choice((32, 64, 104, 128, 256, 504, 608))
        c["V"] = min(c["V"], 300000000 // max(c["K"], F))
    if kind == "gin":
        c["K"] = min(c["K"], 256)
    if kind == "gcn":
        c["norm"] = rng.choice(("values", "degrees"))
    if kind == "gat":
        c["train"] = rng.random() < 0.67
    deg = math.exp(rng.uniform(math.log(4), math.log(500)))
    most = 5500000 if kind == "setup" else min(3500000000 // F, 60000000)
    c["V"] = min(c["V"], most // 3)
    c["E"] = int(max(min(c["V"] * deg, most), 2 * c["V"] + 1))
    return c


# ---------------------------------------------------------------------------------------------------- inputs
def _edges(c, gen, dev):
    """-> (row, col) of c's edge list: int32, in no order."""
    V, E = c["V"], c["E"]
    loops = c["graph"] == "uniform" or c["kind"] in ("gat", "calls")
    n = E - V if loops else E
    if c["graph"] == "uniform":
        row = torch.randint(0, V, (n,), generator=gen, device=dev, dtype=torch.int32)
        col = torch.randint(0, V, (n,), generator=gen, device=dev, dtype=torch.int32)
    elif c["graph"] == "rmat":  # quadrants 0.57 / 0.19 / 0.19 / 0.05, ids relabelled so that hubs are anywhere
        scale = max((V - 1).bit_length(), 1)
        row = torch.zeros(n, dtype=torch.int32, device=dev)
        col = torch.zeros(n, dtype=torch.int32, device=dev)
        for _ in range(scale):
            r = torch.rand(n, generator=gen, device=dev)
            low = r >= 0.76
            row.mul_(2).add_(low)
            col.mul_(2).add_(torch.where(low, r >= 0.95, r >= 0.57))
            del r, low
        name = torch.randperm(V, generator=gen, device=dev, dtype=torch.int32)
        row = name[((row.long() * V) >> scale)]
        col = name[((col.long() * V) >> scale)]
    else:  # log-normal row lengths, sigma 1, uniform columns
        ends = torch.randn(V, generator=gen, device=dev, dtype=torch.float64).exp_().cumsum(0)
        ends = (ends * (n / ends[-1])).round_().long()
        ends[-1] = n
        deg = torch.diff(ends, prepend=ends.new_zeros(1))
        row = torch.repeat_interleave(torch.arange(V, dtype=torch.int32, device=dev), deg, output_size=n)
        col = torch.randint(0, V, (n,), generator=gen, device=dev, dtype=torch.int32)
    if loops:
        ids = torch.arange(V, dtype=torch.int32, device=dev)
        row, col = torch.cat([row, ids]), torch.cat([col, ids])
    return row, col


def _pad(n):
    return (n + 7) // 8 * 8


def _normal(gen, dev, rows, cols, sd=1.0):
    """fp16 normals in rows of a pitch that is a multiple of 8 halves, the padding zero."""
    t = torch.zeros((rows, _pad(cols)), dtype=HALF, device=dev)
    t[:, :cols] = (torch.randn((rows, cols), generator=gen, device=dev) * sd).to(HALF)
    return t


def _zeros(dev, rows, cols, dtype=HALF):
    return torch.zeros((rows, _pad(cols)), dtype=dtype, device=dev)


class _State:
    pass


def prepare(case, seed):
    c, s = case, _State()
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    s.kind = kind = c["kind"]
    V, E = s.V, s.E = c["V"], c["E"]
    s.H, s.D = c.get("H", 1), c.get("D", 0)
    F = s.F = c.get("F") or s.H * s.D
    s.row, s.col = _edges(c, gen, dev)
    if kind == "setup":
        return s
    g = s.g = hgnn.hgnn_coo_to_csr(s.row, s.col, V, V, want_eid=False)[0]
    del s.row, s.col
    s.train = kind != "gat" or c["train"]
    gt = s.gt = hgnn.hgnn_transpose(g) if s.train else None
    if kind != "plain":
        s.plan = hgnn.hgnn_plan_create(g, 256, _pad(F), s.H, col_blocks=0)
        s.plan_t = hgnn.hgnn_plan_create(gt, 256, _pad(F), s.H, col_blocks=0) if s.train else None
    deg = lambda x: torch.diff(x.rowptr).clamp_(min=1).to(torch.float32)  # noqa: E731
    if kind in ("gcn", "plain"):
        rs, cs = deg(g).rsqrt_(), deg(gt).rsqrt_()
        if c.get("norm") == "degrees":
            s.rs, s.cs = rs, cs
        else:
            s.w = (torch.repeat_interleave(rs, torch.diff(g.rowptr), output_size=E) * cs[g.col.long()]).to(HALF).reshape(E, 1)
            if kind == "gcn":  # constant weights: brought into the transposed graph's order once
                s.w_t = torch.empty_like(s.w)
                hgnn.hgnn_edge_to_transposed(gt, 1, s.w, s.w_t)
                s.gt_plain = hgnn.Csr(gt.rowptr, gt.col, ncols=V)
    if kind == "gin":
        s.lam = 0.1
        s.lam_over_deg = 0.1 / deg(g)
    # a column scale goes onto the table first where rows are long enough for that to pay
    long_rows = E / V >= 24 and (kind == "gin" or c.get("norm") == "degrees")
    s.scaled = _zeros(dev, V, F) if long_rows else None
    if kind in ("gcn", "gin", "gat"):
        K = s.K = c["K"]
        wide, deep = (K, F) if kind != "gin" else (F, K)
        s.W = _normal(gen, dev, wide, deep, wide ** -0.5)
        s.X = _normal(gen, dev, V, wide)
        s.Y = _zeros(dev, V, deep)
        if kind != "gat":
            s.dY = _normal(gen, dev, V, deep)
        s.h = _zeros(dev, V, F)
        if s.train:
            s.dh = _zeros(dev, V, F)
            s.dX = _zeros(dev, V, wide)
            s.dW = torch.empty((_pad(wide), _pad(deep)), dtype=torch.float32, device=dev)
            n = hgnn.hgnn_linear_wgrad_workspace(_pad(wide), _pad(deep))
            if kind == "gat":
                n = max(n, hgnn.hgnn_gat_feature_grad_workspace(s.H, s.D))
            s.ws = torch.empty(n, dtype=torch.uint8, device=dev)
    if kind in ("gat", "calls"):
        s.a_l, s.a_r = _normal(gen, dev, 1, F, 0.1).reshape(-1), _normal(gen, dev, 1, F, 0.1).reshape(-1)
        s.d_el, s.d_er = (torch.empty((V, s.H), dtype=HALF, device=dev) for _ in range(2))
    if kind == "gat":
        s.lse, s.csum = (torch.empty((V, s.H), dtype=torch.float32, device=dev) for _ in range(2))
        if s.train:
            s.dY = _normal(gen, dev, V, F)
            s.masked, s.dV = _zeros(dev, V, F), _zeros(dev, V, F)
            s.da_l, s.da_r = (torch.empty(F, dtype=torch.float32, device=dev) for _ in range(2))
    if kind == "calls":
        s.h, s.dY = _normal(gen, dev, V, F), _normal(gen, dev, V, F)
        s.Y, s.dV = _zeros(dev, V, F), _zeros(dev, V, F)
        s.e, s.alpha, s.dalpha, s.ds = (torch.empty((E, s.H), dtype=HALF, device=dev) for _ in range(4))
        s.sliced = s.H == 1 and hgnn.hgnn_plan_num_slices(s.plan) > 0
    if kind == "plain":
        s.X, s.dY = _normal(gen, dev, V, F), _normal(gen, dev, V, F)
        s.Y, s.dX = _zeros(dev, V, F), _zeros(dev, V, F)
        n = hgnn.hgnn_spmm_workspace(V, V, E, F)
        s.ws = torch.empty(n, dtype=torch.uint8, device=dev) if n else None
    return s


# ---------------------------------------------------------------------------------------------------- one pass
def _gcn(s):
    """Y = A_w (X W); dh = A_w^T dY, dW = X^T dh, dX = dh W^T."""
    hgnn.hgnn_linear(s.X, s.W, s.h)
    if hasattr(s, "w"):
        hgnn.hgnn_spmm_discretized(s.plan, s.g, s.w, 1, s.h, s.Y, F=s.F)
        hgnn.hgnn_spmm_discretized(s.plan_t, s.gt_plain, s.w_t, 1, s.dY, s.dh, F=s.F)
    else:
        hgnn.hgnn_spmm_discretized_fused(s.plan, s.g, None, 1, s.h, s.Y, row_scale=s.rs, col_scale=s.cs, F=s.F, scaled_x=s.scaled)
        hgnn.hgnn_spmm_discretized_fused(s.plan_t, s.gt, None, 1, s.dY, s.dh, row_scale=s.cs, col_scale=s.rs, F=s.F, scaled_x=s.scaled)
    hgnn.hgnn_linear_wgrad(s.X, s.dh, s.dW, s.ws)
    hgnn.hgnn_linear(s.dh, s.W, s.dX, trans_w=True)
    return {"Y": s.Y, "dW": s.dW, "dX": s.dX}


def _gin(s):
    """h = (1 + eps) X + lambda mean(X), Y = h W; dh = dY W^T, dW = h^T dY, dX = the aggregation's transpose of dh."""
    hgnn.hgnn_spmm_discretized_fused(s.plan, s.g, None, 1, s.X, s.h, op=hgnn.HGNN_MEAN, self_feat=s.X, self_coef=1.0, agg_coef=s.lam, F=s.F)
    hgnn.hgnn_linear(s.h, s.W, s.Y)
    hgnn.hgnn_linear_wgrad(s.h, s.dY, s.dW, s.ws)
    hgnn.hgnn_linear(s.dY, s.W, s.dh, trans_w=True)
    hgnn.hgnn_spmm_discretized_fused(s.plan_t, s.gt, None, 1, s.dh, s.dX, col_scale=s.lam_over_deg, self_feat=s.dh, self_coef=1.0,
                                     F=s.F, scaled_x=s.scaled)
    return {"Y": s.Y, "dW": s.dW, "dX": s.dX}


def _gat(s):
    """The attention layer with the single-pass aggregation; trained: with every gradient."""
    hgnn.hgnn_linear(s.X, s.W, s.h)
    if not s.train:
        hgnn.hgnn_gat_forward_fused(s.g, s.plan, s.H, s.D, s.h, s.h, s.a_l, s.a_r, s.Y, neg_slope=SLOPE)
        return s.Y
    hgnn.hgnn_gat_forward_fused_save(s.g, s.plan, s.H, s.D, s.h, s.h, s.a_l, s.a_r, s.Y, s.lse, s.masked, s.csum, neg_slope=SLOPE)
    hgnn.hgnn_gat_backward_fused_saved(s.g, s.plan, s.gt, s.plan_t, s.H, s.D, s.h, s.h, s.a_l, s.a_r, s.Y, s.lse, s.masked, s.csum,
                                       s.dY, s.dV, s.d_el, s.d_er, neg_slope=SLOPE)
    hgnn.hgnn_gat_feature_grad(s.H, s.D, s.dV, s.d_el, s.d_er, s.a_l, s.a_r, s.h, s.dh, s.da_l, s.da_r, s.ws)
    hgnn.hgnn_linear_wgrad(s.X, s.dh, s.dW, s.ws)
    hgnn.hgnn_linear(s.dh, s.W, s.dX, trans_w=True)
    return {"Y": s.Y, "dW": s.dW, "dX": s.dX, "da_l": s.da_l, "da_r": s.da_r}


def _calls(s):
    """Score, softmax and weighted sum; then the weighted transpose, the dot products, and the softmax and score gradients."""
    H, D = s.H, s.D
    hgnn.hgnn_sddmm(s.g, s.plan, hgnn.HGNN_SDDMM_GAT_SCORE, H, D, s.h, s.h, s.e, s.a_l, s.a_r, SLOPE)
    hgnn.hgnn_edge_softmax(s.g, s.plan, H, s.e, s.alpha)
    hgnn.hgnn_spmm_discretized(s.plan, s.g, s.alpha, H, s.h, s.Y)
    hgnn.hgnn_spmm_discretized(s.plan_t, s.gt, s.alpha, H, s.dY, s.dV)
    hgnn.hgnn_sddmm(s.g, s.plan, hgnn.HGNN_SDDMM_DOT, H, D, s.dY, s.h, s.dalpha)
    hgnn.hgnn_edge_softmax_bwd(s.g, s.plan, H, s.alpha, s.dalpha, s.ds, e=s.e, neg_slope=SLOPE)
    hgnn.hgnn_edge_rowsum(s.g, s.plan, H, s.ds, s.d_el)
    if s.sliced:
        hgnn.hgnn_edge_colsum(s.g, s.plan, H, s.ds, s.d_er)
    else:
        hgnn.hgnn_edge_rowsum(s.gt, s.plan_t, H, s.ds, s.d_er)
    return {"e": s.e, "alpha": s.alpha, "Y": s.Y, "dV": s.dV, "dalpha": s.dalpha, "ds": s.ds, "d_er": s.d_er}


def _plain(s):
    hgnn.hgnn_spmm(s.g, s.w, 1, s.X, s.Y, F=s.F, workspace=s.ws)
    hgnn.hgnn_spmm(s.gt, s.w, 1, s.dY, s.dX, F=s.F, workspace=s.ws)
    return {"Y": s.Y, "dX": s.dX}


def _setup(s):
    g, eid = hgnn.hgnn_coo_to_csr(s.row, s.col, s.V, s.V)
    gt = hgnn.hgnn_transpose(g)
    plan = hgnn.hgnn_plan_create(g, 256, _pad(s.F), 1, col_blocks=0)
    plan_t = hgnn.hgnn_plan_create(gt, 256, _pad(s.F), 1, col_blocks=0)
    segments = hgnn.hgnn_plan_num_segments(plan), hgnn.hgnn_plan_num_split_rows(plan), hgnn.hgnn_plan_num_split_rows(plan_t)
    return {"rowptr": g.rowptr, "col": g.col, "eid": eid, "rowptr_t": gt.rowptr, "col_t": gt.col, "eid_t": gt.eid, "segments": segments}


_PASS = {"gcn": _gcn, "gin": _gin, "gat": _gat, "calls": _calls, "plain": _plain, "setup": _setup}


def run(state):
    return _PASS[state.kind](state)


# ---------------------------------------------------------------------------------------------------- what it takes
def work(case):
    """Every input read once, every output written once; intermediates of a layer are not counted."""
    c, kind = case, case["kind"]
    V, E, H = c["V"], c["E"], c.get("H", 1)
    F, K = c.get("F") or H * c["D"], c.get("K", 0)
    graph = 4 * E + 4 * (V + 1)
    if kind == "setup":
        return {"bytes": 8 * E + 5 * 4 * E + 2 * 4 * (V + 1), "flops": 0}
    if kind == "plain":
        return {"bytes": 2 * graph + 4 * E + 2 * E + 4 * 2 * V * F, "flops": 4 * E * F}
    if kind == "calls":  # features and gradient in, two vertex results, four edge tensors
        return {"bytes": 2 * graph + 4 * E + 4 * 2 * V * F + 4 * 2 * E * H + 2 * V * H, "flops": 6 * E * F}
    dense = 2 * V * K * F
    if kind == "gat" and not c["train"]:
        return {"bytes": graph + 2 * V * K + 2 * K * F + 2 * V * F, "flops": dense + 2 * E * F}
    wide, deep = (K, F) if kind != "gin" else (F, K)
    nbytes = 2 * graph + 2 * 2 * V * wide + 2 * 2 * V * deep + (2 + 4) * wide * deep
    if c.get("norm") == "values":
        nbytes += 2 * 2 * E
    if c.get("norm") == "degrees" or kind == "gin":
        nbytes += 2 * 4 * V
    return {"bytes": nbytes, "flops": 3 * dense + (4 if kind != "gat" else 8) * E * F}


def tolerance(case):
    """fp16 in memory, fp32 sums: a rounding or two per value of an output, two or three where layer steps follow each other.  The
    gradients of the attention vectors are sums of softmax gradients, which cancel inside a row, so more of them shows."""
    if case["kind"] == "setup":
        return "exact"
    return {"rel": 1e-2 if case["kind"] == "gat" else 2e-3, "max": 0.1}
