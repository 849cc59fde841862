"""The work a user of this library has it do, as timed cases: whole training epochs (eager, recorded as a HIP graph, two-stream
with a host tier), single layers with their backward pass, inference, bare aggregation, and the joint cache's own calls.

Every case is built from the seed alone (graph, features, weights, cached rows) through the public binding; graphs are
power-law partitions like those of ``paper_2508_13716_amd/synth.py``, drawn on the GPU so that making them is quick.  Shapes
follow the five named configurations (at full or reduced vertex count, degrees and widths kept) or are generic, ragged sizes
between them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2508_13716_amd import binding as B
from paper_2508_13716_amd import synth


def _case(name, what, kind="gcn", n_loc=0, n_halo=0, nnz=0, dims="", dtype="f32", tier=1.0, mode="staged", loss="ce", lr=0.0,
          sym=False, zipf=0.0, n_req=0):
    c = dict(what=what, kind=kind, n_loc=n_loc, n_halo=n_halo, nnz=nnz, dims=dims, dtype=dtype, tier=tier, mode=mode, loss=loss,
             lr=lr, sym=sym, zipf=zipf, n_req=n_req)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest evaluation graph, trained epoch by epoch with the in-epoch SGD step: bound by launches and latency
        _case("epoch_tiny", "epoch", n_loc=4096, n_halo=4096, nnz=40_000, dims="128-64-8", lr=0.01),
        # a small ragged partition whose epoch the program has recorded as a HIP graph and replays
        _case("epoch_small_recorded", "recorded", kind="sage", n_loc=9_973, n_halo=3_331, nnz=150_000, dims="100-64-7"),
        # one of four partitions of a dense-degree graph (the headline configuration, full size): half of the halo rows in the
        # pinned-host tier, transferred one epoch ahead on the side stream
        _case("epoch_dense", "epoch", n_loc=60_000, n_halo=120_000, nnz=30_000_000, dims="602-256-41", tier=0.5, mode="pipelined"),
        # sparse large partition, three-layer GraphSAGE at half the configuration's vertex count, every halo row on the GPU (what
        # the capacity rule grants on this card)
        _case("epoch_sage", "epoch", kind="sage", n_loc=306_000, n_halo=350_000, nnz=8_000_000, dims="100-256-256-47"),
        # an unpartitioned symmetric graph in bf16, three-layer GCN, no halo
        _case("epoch_whole_bf16", "epoch", n_loc=980_000, nnz=50_000_000, dims="128-256-256-47", dtype="bf16", sym=True),
        # cache stress: Zipf halo accesses, a tenth of the halo rows on the GPU, the rest staged from pinned memory
        _case("epoch_zipf_bf16", "epoch", n_loc=100_000, n_halo=200_000, nnz=4_000_000, dims="512-256-47", dtype="bf16", tier=0.1,
              zipf=1.1),
        # multi-label task on a GIN operator (edge values), ragged widths, the loss read back every epoch
        _case("epoch_gin_multilabel", "epoch", kind="gin", n_loc=21_557, n_halo=8_011, nnz=420_000, dims="50-128-121", loss="bce"),
        # one GraphSAGE layer forward and backward inside a caller's own training loop, gradient of the halo rows included
        _case("layer_halo_grad", "layer", kind="sage", n_loc=70_001, n_halo=45_003, nnz=1_500_000, dims="100-256"),
        # inference over a partition: fill the halo rows, two layers forward
        _case("infer_bf16", "infer", n_loc=150_000, n_halo=300_000, nnz=6_000_000, dims="512-256-47", dtype="bf16"),
        # bare aggregation and its transpose, as an outside layer implementation calls them
        _case("aggregate_pair", "aggregate", n_loc=120_011, n_halo=80_009, nnz=3_000_000, dims="100"),
        # request-list gather by global id (hash lookup), Zipf requests, one row in ten of the table on the GPU
        _case("gather_requests", "requests", n_halo=1_000_000, dims="128", tier=0.1, zipf=1.1, n_req=500_000),
        # JACA's refresh of a layer: rewrite every cached row of both tiers, then fill the layer input
        _case("cache_refresh", "refresh", n_halo=120_000, dims="256", tier=0.5),
    ]


def draw(rng):
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    what = rng.choice(["epoch", "epoch", "epoch", "recorded", "layer", "infer", "aggregate", "requests", "refresh"])
    dtype = rng.choice(["f32", "f32", "bf16"])
    if what in ("requests", "refresh"):
        n_halo = log(2_000, 400_000)
        return _case(None, what, n_halo=n_halo, dims=str(rng.choice([47, 64, 100, 128, 256, 602])), dtype=dtype,
                     tier=rng.choice([0.1, 0.3, 0.5, 1.0]), zipf=1.1 if what == "requests" else 0.0,
                     n_req=log(1_000, 500_000) if what == "requests" else 0)
    kind = rng.choice(["gcn", "gcn", "sage", "sage", "gin"])
    n_loc = log(1_000, 20_000) if what == "recorded" else log(1_000, 250_000)
    deg = log(4, 60)
    nnz = min(n_loc * deg, 6_000_000)
    if n_loc <= 50_000 and rng.random() < 0.2:
        nnz = min(n_loc * log(60, 400), 6_000_000)
    sym = kind == "gcn" and rng.random() < 0.25
    n_halo = 0 if sym or what == "recorded" and rng.random() < 0.5 else min(int(n_loc * rng.uniform(0.2, 2.0)), nnz // 3)
    f0, hid, cls = log(16, 602), rng.choice([32, 64, 100, 128, 200, 256]), log(2, 121)
    if what == "aggregate":
        dims = str(log(7, 300))
    elif what == "layer":
        dims = "%d-%d" % (min(f0, 300), hid)
    else:
        dims = "-".join(str(d) for d in ([f0, hid, cls] if rng.random() < 0.6 else [f0, hid, hid, cls]))
    epoch = what in ("epoch", "recorded")
    tier = rng.choice([0.5, 1.0, 1.0, 1.0]) if what == "epoch" and n_halo else 1.0
    return _case(None, what, kind=kind, n_loc=n_loc, n_halo=n_halo, nnz=nnz, dims=dims, dtype=dtype, tier=tier,
                 mode=rng.choice(["staged", "pipelined"]), loss="bce" if what == "epoch" and rng.random() < 0.25 else "ce",
                 lr=0.01 if epoch and dtype == "f32" and rng.random() < 0.5 else 0.0, sym=sym,
                 zipf=1.1 if n_halo and rng.random() < 0.2 else 0.0)


# ------------------------------------------------------------------------------------------------ inputs
def _dims(case):
    return [int(d) for d in case["dims"].split("-")]


def _ranks(gen, n, m, alpha, i0):
    """m ranks in [0, n) with density (rank + i0)^-alpha (inverse distribution function)."""
    u = torch.rand(m, generator=gen, device="cuda", dtype=torch.float64)
    e = 1.0 - alpha
    lo, hi = i0 ** e, (n + i0) ** e
    return ((lo + u * (hi - lo)).pow_(1.0 / e) - i0).long().clamp_(0, n - 1)


def _offset(n, alpha, share):
    """i0 for which rank 0 gets about `share` of the draws."""
    e = 1.0 - alpha
    top = lambda i0: ((1 + i0) ** e - i0 ** e) / ((n + i0) ** e - i0 ** e)  # noqa: E731
    lo, hi = 1e-3, float(max(n, 2))
    for _ in range(50):
        mid = math.sqrt(lo * hi)
        lo, hi = (mid, hi) if top(mid) > share else (lo, mid)
    return math.sqrt(lo * hi)


def _edges(case, gen):
    """CSR of a power-law partition (exponent 2.1, hubs scattered, duplicates removed), on the host; in-partition references of
    every halo vertex."""
    n_loc, n_halo, nnz = case["n_loc"], case["n_halo"], case["nnz"]
    n_cols, alpha = n_loc + n_halo, 1.0 / 1.1
    i0 = _offset(n_loc, alpha, max(8.0, min(n_loc / 4, 40.0 * nnz / n_loc, 30_000.0)) / nnz)
    perm = lambda n: torch.randperm(n, generator=gen, device="cuda")  # noqa: E731
    loops = torch.arange(n_loc, device="cuda")
    dst_of = perm(n_loc)
    if case["sym"]:
        u, v = (dst_of[_ranks(gen, n_loc, nnz // 2, alpha, i0)] for _ in range(2))
        keep = u != v
        u, v = u[keep], v[keep]
        rows, cols = [u, v], [v, u]
    else:
        n_he = max(nnz // 2, n_halo) if n_halo else 0
        u, v = dst_of[_ranks(gen, n_loc, nnz - n_he, alpha, i0)], perm(n_loc)[_ranks(gen, n_loc, nnz - n_he, alpha, i0)]
        keep = u != v
        rows, cols = [u[keep]], [v[keep]]
        if n_halo:      # every halo vertex is the source of an edge; the others follow the law (or Zipf)
            rows.append(dst_of[_ranks(gen, n_loc, n_he, alpha, i0)])
            more = (_ranks(gen, n_halo, n_he - n_halo, case["zipf"], 1.0) if case["zipf"] else
                    _ranks(gen, n_halo, n_he - n_halo, alpha, _offset(n_halo, alpha, max(8.0, 40.0 * n_he / n_halo) / n_he)))
            cols.append(n_loc + torch.cat([torch.arange(n_halo, device="cuda"), perm(n_halo)[more]]))
    if case["kind"] == "gcn":
        rows.append(loops)
        cols.append(loops)
    key = torch.unique(torch.cat(rows) * n_cols + torch.cat(cols))
    row = key // n_cols
    col = (key - row * n_cols).int()
    rowptr = torch.zeros(n_loc + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(row, minlength=n_loc), 0, out=rowptr[1:])
    refs = torch.bincount(col[col >= n_loc].long() - n_loc, minlength=n_halo).cpu().numpy() if n_halo else np.zeros(0, np.int64)
    return rowptr.cpu().numpy(), col.cpu().numpy(), refs


def _graph(case, gen):
    rowptr, col, refs = _edges(case, gen)
    n_loc, n_halo = case["n_loc"], case["n_halo"]
    if case["kind"] == "gin":
        rowptr, col, val = B.gin_operator(n_loc, n_halo, rowptr, col, 0.1)
        return B.Graph(n_loc, n_halo, rowptr, col, None, None, val, 0), refs
    r, c = B.norm_scales(B.NORM_MEAN if case["kind"] == "sage" else B.NORM_SYM, n_loc, n_halo, rowptr, 2 * refs)
    return B.Graph(n_loc, n_halo, rowptr, col, r, c, None, B.GRAPH_SYMMETRIC if case["sym"] else 0), refs


def _cache(case, gen, refs, dims, dt, map_kind=B.MAP_DIRECT):
    """Both tiers filled with rows ~N(0,1)."""
    n = case["n_halo"]
    gid = torch.randperm(n, generator=gen, device="cuda").cpu().numpy().astype(np.int64) * 7919 + 1_000_003
    c = B.Cache(gid, np.ascontiguousarray(refs, np.int64), int(round(case["tier"] * n)), dims, B.BF16 if dt is torch.bfloat16 else B.F32,
                map_kind)
    ids = torch.arange(n, device="cuda")
    for l, d in enumerate(dims):
        B.cache_update(c, l, ids, n, torch.randn(n, d, generator=gen, device="cuda").to(dt), d, 0)
    torch.cuda.synchronize()
    c.set_miss_mode({"staged": B.MISS_STAGED, "pipelined": B.MISS_PIPELINED}[case["mode"]])
    return c, gid


def _matrix(gen, rows, width, dt):
    """Feature rows ~N(0,1), each row starting on a cache line."""
    ld = synth.pad_to(width, 128 // dt.itemsize)
    x = torch.zeros(rows, ld, dtype=dt, device="cuda")
    x[:, :width] = torch.randn(rows, width, generator=gen, device="cuda").to(dt)
    return x, ld


_main, _side = [], []


def _streams():
    """The two streams a program runs this library on."""
    if not _main:
        _main.append(torch.cuda.Stream())
        _side.append(torch.cuda.Stream())
    return _main[0], _side[0]


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    dims, dt = _dims(case), torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    code = B.BF16 if dt is torch.bfloat16 else B.F32
    main, side = _streams()
    s = dict(what=case["what"], main=main, side=side, code=code, n_halo=case["n_halo"])
    if case["what"] == "requests":
        n = case["n_halo"]
        refs = torch.randint(1, 1 << 20, (n,), generator=gen, device="cuda")
        s["cache"], gid = _cache(case, gen, refs.cpu().numpy(), dims, dt, B.MAP_HASH)
        by_rank = torch.from_numpy(gid).cuda()[torch.argsort(refs, descending=True, stable=True)]
        s.update(width=dims[0], ids=by_rank[_ranks(gen, n, case["n_req"], case["zipf"], 1.0)],
                 out=torch.zeros(case["n_req"], dims[0], dtype=dt, device="cuda"))
    elif case["what"] == "refresh":
        n = case["n_halo"]
        s["cache"], _ = _cache(case, gen, torch.randint(1, 1000, (n,), generator=gen, device="cuda").cpu().numpy(), dims, dt)
        rows, ld = _matrix(gen, n, dims[0], dt)
        s.update(width=dims[0], ids=torch.randperm(n, generator=gen, device="cuda"), rows=rows, ld=ld,
                 out=torch.zeros(n, ld, dtype=dt, device="cuda"), stage=torch.empty(s["cache"].staging_bytes, dtype=torch.uint8, device="cuda"))
    else:
        s["graph"], refs = _graph(case, gen)
        {"aggregate": _prepare_aggregate}.get(case["what"], _prepare_model)(case, gen, s, refs, dims, dt)
    torch.cuda.synchronize()
    return s


def _prepare_aggregate(case, gen, s, refs, dims, dt):
    g, f = s["graph"], dims[0]
    s["x"], ld = _matrix(gen, g.n_cols, f, dt)
    s["dy"], _ = _matrix(gen, g.n_loc, f, dt)
    s.update(f=f, ld=ld, y=torch.zeros(g.n_loc, ld, dtype=dt, device="cuda"), dx=torch.zeros(g.n_cols, ld, dtype=dt, device="cuda"))
    s["ws_bytes"] = B.spmm_workspace_bytes(g, f, s["code"])
    s["ws"] = torch.empty(max(s["ws_bytes"], 256), dtype=torch.uint8, device="cuda")


def _prepare_model(case, gen, s, refs, dims, dt):
    g, code, n_loc, L = s["graph"], s["code"], case["n_loc"], len(dims) - 1
    sage, what = case["kind"] == "sage", case["what"]
    s["x"], s["ld"] = _matrix(gen, g.n_cols, dims[0], dt)
    s["cache"] = _cache(case, gen, refs, dims[:L], dt)[0] if g.n_halo and what != "layer" else None
    weight = lambda i: ((torch.rand(dims[i], dims[i + 1], generator=gen, device="cuda") * 2 - 1) * math.sqrt(6.0 / (dims[i] + dims[i + 1]))).to(dt)  # noqa: E731
    grad = lambda i: torch.zeros(dims[i], dims[i + 1], device="cuda")  # noqa: E731
    s["w"] = [weight(i) for i in range(L)]
    s["w_self"] = [weight(i) for i in range(L)] if sage else None
    s["b"] = [0.01 * torch.randn(d, generator=gen, device="cuda") for d in dims[1:]]
    s["dw"] = [grad(i) for i in range(L)]
    s["dw_self"] = [grad(i) for i in range(L)] if sage else None
    s["db"] = [torch.zeros(d, device="cuda") for d in dims[1:]]
    layers = [B.make_layer(B.SAGE_MEAN if sage else B.GCN, dims[i], dims[i + 1],
                           B.ACT_NONE if i == L - 1 and what != "layer" else B.ACT_RELU, code, s["w"][i], s["w_self"][i] if sage else None,
                           s["b"][i], out_f32=int(i == L - 1 and code == B.BF16 and what != "layer")) for i in range(L)]
    s["layers"] = layers
    empty = lambda n: torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")  # noqa: E731
    if what in ("layer", "infer"):
        for i, l in enumerate(layers):
            l.order = B.layer_order(g, l, what == "layer" or i > 0)
        s["saved"] = empty(max(B.layer_saved_bytes(g, l) for l in layers))
        s["ws_bytes"] = max(B.layer_workspace_bytes(g, l) for l in layers)
        s["ws"] = empty(s["ws_bytes"])
        rows = [n_loc if i == L - 1 else g.n_cols for i in range(L)]
        s["h"] = [torch.zeros(n, synth.pad_to(d, 128 // dt.itemsize), dtype=torch.float32 if l.out_f32 else dt, device="cuda")
                  for n, d, l in zip(rows, dims[1:], layers)]
        if what == "layer":
            s["dh0"] = _matrix(gen, n_loc, dims[1], dt)[0] / n_loc
            s["dh"], s["dx"] = torch.zeros_like(s["dh0"]), torch.zeros_like(s["x"])
        return
    s["labels"] = torch.randint(0, dims[-1], (n_loc,), generator=gen, device="cuda", dtype=torch.int32)
    s["targets"] = (torch.rand(n_loc, dims[-1], generator=gen, device="cuda") < 0.3).byte() if case["loss"] == "bce" else None
    s["mask"] = (torch.rand(n_loc, generator=gen, device="cuda") < 0.6).byte()
    s["logits"] = torch.zeros(n_loc, dims[-1], device="cuda")
    s["lr"] = case["lr"]
    s["ws_bytes"] = B.epoch_workspace_bytes(g, s["cache"], layers)
    s["ws"] = empty(s["ws_bytes"])
    if what == "recorded":
        s["loss"] = torch.zeros(1, device="cuda")
        torch.cuda.synchronize()
        s["recorded"] = B.EpochGraph(g, s["cache"], layers, s["x"], s["ld"], s["labels"], s["mask"], 0.0, s["logits"], s["dw"],
                                     s["dw_self"], s["db"], s["lr"], s["loss"], s["ws"], s["ws_bytes"], s["main"])


# ------------------------------------------------------------------------------------------------ one pass
def run(s):
    return {"epoch": _run_epoch, "recorded": _run_recorded, "layer": _run_layer, "infer": _run_infer, "aggregate": _run_aggregate,
            "requests": _run_requests, "refresh": _run_refresh}[s["what"]](s)


def _model_outputs(s, **more):
    out = dict(more, dw=s["dw"], dw_self=s["dw_self"], db=s["db"])
    if s.get("lr"):
        out.update(w=s["w"], w_self=s["w_self"], b=s["b"])
    return out


def _run_epoch(s):
    loss, _ = B.epoch(s["graph"], s["cache"], s["layers"], s["x"], s["ld"], s["labels"], s["mask"], 0.0, s["logits"], s["dw"],
                      s["dw_self"], s["db"], s["lr"], s["ws"], s["ws_bytes"], s["main"], s["side"] if s["n_halo"] else None,
                      want_loss=s["targets"] is not None, targets=s["targets"],
                      ldt=0 if s["targets"] is None else s["targets"].shape[1])
    return _model_outputs(s, logits=s["logits"], loss=loss)


def _run_recorded(s):
    s["recorded"].launch(s["main"])
    return _model_outputs(s, logits=s["logits"], loss=s["loss"])


def _run_layer(s):
    g, l, x, h = s["graph"], s["layers"][0], s["x"], s["h"][0]
    with torch.cuda.stream(s["main"]):
        B.layer_fwd(g, l, x, s["ld"], h, h.shape[1], s["saved"], s["ws"], s["ws_bytes"], s["main"])
        s["dh"].copy_(s["dh0"])      # the gradient that the caller's next layer hands back (the call overwrites it)
        B.layer_bwd(g, l, x, s["ld"], h, h.shape[1], s["saved"], s["dh"], s["dh"].shape[1], s["dw"][0],
                    s["dw_self"][0] if s["dw_self"] else None, s["db"][0], s["dx"], s["ld"], True, s["ws"], s["ws_bytes"], s["main"])
    return _model_outputs(s, h=h, dx=s["dx"])


def _run_infer(s):
    g, x, ld = s["graph"], s["x"], s["ld"]
    for i, l in enumerate(s["layers"]):
        if g.n_halo:
            B.halo_gather(s["cache"], i, None, g.n_halo, x[g.n_loc:], ld, stream=s["main"])
        h = s["h"][i]
        B.layer_fwd(g, l, x, ld, h, h.shape[1], s["saved"], s["ws"], s["ws_bytes"], s["main"])
        x, ld = h, h.shape[1]
    return s["h"]


def _run_aggregate(s):
    g, ld = s["graph"], s["ld"]
    B.spmm_fwd(g, s["x"], ld, s["y"], ld, s["f"], s["code"], s["main"], s["ws"], s["ws_bytes"])
    B.spmm_bwd(g, s["dy"], ld, s["dx"], ld, s["f"], s["code"], s["main"], s["ws"], s["ws_bytes"])
    return {"y": s["y"], "dx": s["dx"]}


def _run_requests(s):
    B.halo_gather(s["cache"], 0, s["ids"], s["ids"].numel(), s["out"], s["width"], by_gid=True, stream=s["main"])
    return s["out"]


def _run_refresh(s):
    c, n = s["cache"], s["n_halo"]
    B.cache_update(c, 0, s["ids"], n, s["rows"], s["ld"], 1, stream=s["main"])
    B.halo_gather(c, 0, None, n, s["out"], s["ld"], stream=s["main"], side_stream=s["side"], staging=s["stage"])
    return s["out"]


# ------------------------------------------------------------------------------------------------ what a pass cannot do without
def work(case):
    d, es, n_loc, n_halo = _dims(case), 2 if case["dtype"] == "bf16" else 4, case["n_loc"], case["n_halo"]
    what = case["what"]
    if what == "requests":
        return {"bytes": case["n_req"] * (8 + 2 * d[0] * es), "flops": 0}
    if what == "refresh":      # rows read, cached row written, cached row read, layer input written
        return {"bytes": n_halo * (8 + 4 * d[0] * es), "flops": 0}
    nnz, n = case["nnz"] + (n_loc if case["kind"] in ("gcn", "gin") else 0), n_loc + n_halo
    index = nnz * (8 if case["kind"] == "gin" else 4) + (n_loc + n) * 8
    if what == "aggregate":
        return {"bytes": 2 * index + 2 * (n + n_loc) * d[0] * es, "flops": 4 * nnz * d[0]}
    sage = 2 if case["kind"] == "sage" else 1
    L, weights = len(d) - 1, sum(a * b for a, b in zip(d, d[1:])) * sage
    halo = n_halo * sum(d[:L]) * es * (0 if what == "layer" else 1)
    fwd = sum(2 * n_loc * a * b * sage + 2 * nnz * min(a, b) for a, b in zip(d, d[1:]))
    if what == "infer":
        return {"bytes": index + n_loc * d[0] * es + halo + weights * es + n_loc * d[-1] * 4, "flops": fwd}
    if what == "layer":
        return {"bytes": 2 * index + 2 * n * d[0] * es + 2 * n_loc * d[1] * es + weights * (es + 4),
                "flops": 3 * fwd - 2 * nnz * min(d)}
    bwd = 2 * fwd - 2 * n_loc * d[0] * d[1] * sage - 2 * nnz * sum(min(a, b) for a, b in zip(d, d[1:])) - 2 * nnz * min(d[:2])
    return {"bytes": 2 * index + n_loc * d[0] * es + halo + weights * (es + 4) + n_loc * (d[-1] * 4 + 5), "flops": fwd + bwd}


def tolerance(case):
    """Four times what was measured between the two associations of every layer and the two forms of the fp32 product, at most
    what the comparison allows.  Forward passes and bare aggregation are float32 sums in another order (5e-7).  Where a ReLU is
    differentiated, a pre-activation within rounding of zero may fall on either side, and one such element moves a weight gradient
    that is a sum of cancelling terms by up to 3e-4 (8e-4, and a whole row of the input gradient, where the output gradient is
    white noise).  bf16: one rounding per stored intermediate, through three layers and back (2e-3 forward, 3e-2 for gradients)."""
    if case["what"] in ("requests", "refresh"):
        return "exact"
    if case["what"] in ("infer", "aggregate"):
        return {"rel": 5e-6, "max": 2e-4} if case["dtype"] == "f32" else {"rel": 1e-2, "max": 0.1}
    if case["dtype"] == "bf16":
        return {"rel": 3e-2, "max": 0.9 if case["what"] == "layer" else 0.5}
    return {"rel": 3e-3, "max": 0.9} if case["what"] == "layer" else {"rel": 1.2e-3, "max": 0.06}
