"""Layer and epoch parity of the HIP library against the CPU oracle (needs an MI355X)."""
import numpy as np
import pytest

from paper_2508_13716_amd import synth
from tests.gpu_compare import TOL, compare_epoch, say, teacher_forced_layers

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env(orc):
    import torch
    from paper_2508_13716_amd import binding as B, harness as H
    from tests import oracle_side as O
    assert torch.cuda.is_available()
    B.lib()
    return dict(torch=torch, B=B, H=H, O=O, orc=orc)


@pytest.mark.parametrize("orders", ["auto", "agg", "xform"])
@pytest.mark.parametrize("miss_mode", [0, 1, 2])
def test_epoch_config1_matches_oracle(env, orders, miss_mode):
    B, H, O = env["B"], env["H"], env["O"]
    import copy
    cfg = copy.deepcopy(synth.CONFIGS["C1"])
    cfg.cache_frac = 0.4 if miss_mode else 1.0        # config 1 proper caches every halo row on the GPU
    prob = H.make_problem(cfg, mask_frac=0.5)
    ords = None if orders == "auto" else [B.AGG_FIRST if orders == "agg" else B.XFORM_FIRST] * 2
    dp = H.DeviceProblem(prob, orders=ords, miss_mode=miss_mode)
    ref = O.oracle_epoch(prob)
    for rep in range(3 if miss_mode == 2 else 2):       # later runs: buffers (and prefetched rows) are reused
        loss, _ = dp.run_epoch()
        compare_epoch(env, prob, dp, ref, loss, TOL["f32"], f"C1 {orders} miss_mode={miss_mode} rep={rep}")
    if miss_mode == 1:
        teacher_forced_layers(env, prob, dp, O.oracle_epoch(prob, halo_grad=True), TOL["f32"], f"C1 {orders}", need_halo=True)
    dp.close()


@pytest.mark.parametrize("cache_frac", [0.0, 1.0])
def test_epoch_pipelined_with_one_tier_empty(env, cache_frac):
    """Pipelined mode scatters the GPU tier's rows and the staged host rows of a layer in one launch; with either tier
    empty the same call must serve the other one alone."""
    H, O, B = env["H"], env["O"], env["B"]
    import copy
    cfg = copy.deepcopy(synth.CONFIGS["C1"])
    cfg.cache_frac = cache_frac
    prob = H.make_problem(cfg, mask_frac=0.5)
    assert prob.cap_gpu == (0 if cache_frac == 0.0 else prob.part.n_halo)
    dp = H.DeviceProblem(prob, miss_mode=B.MISS_PIPELINED)
    ref = O.oracle_epoch(prob)
    for rep in range(3):
        say(f"pipelined epoch, cache_frac={cache_frac} rep={rep}")
        loss, _ = dp.run_epoch()
        compare_epoch(env, prob, dp, ref, loss, TOL["f32"], f"C1 pipelined cache_frac={cache_frac} rep={rep}")
    dp.close()


@pytest.mark.parametrize("name,scale", [("C2", 0.02), ("C3", 0.01), ("C4", 0.002), ("C5", 0.004), ("C3-bf16", 0.01),
                                        ("C4-f32", 0.002)])
def test_epoch_scaled_configs_match_oracle(env, name, scale):
    """The named workloads at a fraction of their size (same average degree and widths), plus the two crossings the named
    ones leave out: the GraphSAGE model with bf16 storage and the three-layer GCN on the symmetric graph in fp32."""
    B, H, O = env["B"], env["H"], env["O"]
    cfg = synth.CONFIGS[name.split("-")[0]].scaled(scale)
    if "-" in name:
        cfg.dtype = name.split("-")[1]
        cfg.name = f"{cfg.name}-{cfg.dtype}"
    prob = H.make_problem(cfg, mask_frac=0.5)
    say(f"{cfg.name}: n_loc={prob.part.n_loc} n_halo={prob.part.n_halo} nnz={prob.part.nnz} dims={cfg.dims} {cfg.dtype}")
    dp = H.DeviceProblem(prob)
    say(f"orders={dp.resolved_orders()}")
    ref = O.oracle_epoch(prob)
    loss, times = dp.run_epoch(want_times=True)
    compare_epoch(env, prob, dp, ref, loss, TOL[cfg.dtype], cfg.name)
    assert times["total_ms"] > 0 and times["aggregation_ms"] > 0 and len(times["records"]) >= 2 * dp.L
    # without a side stream the result is the same
    dp2 = H.DeviceProblem(prob, use_side_stream=False, orders=[B.XFORM_FIRST if l % 2 else B.AGG_FIRST for l in range(dp.L)])
    loss2, _ = dp2.run_epoch()
    compare_epoch(env, prob, dp2, ref, loss2, TOL[cfg.dtype], cfg.name + " single-stream, mixed orders")
    teacher_forced_layers(env, prob, dp, ref, TOL[cfg.dtype], cfg.name)
    teacher_forced_layers(env, prob, dp2, ref, TOL[cfg.dtype], cfg.name + " mixed orders")
    dp.close()
    dp2.close()


@pytest.mark.parametrize("kind,dtype,loss", [("gcn", "f32", "ce"), ("sage", "f32", "bce"), ("gin", "f32", "ce"), ("sage", "bf16", "ce"),
                                             ("gcn", "bf16", "bce")])
@pytest.mark.parametrize("dims,n_loc", [([40, 33, 48, 1], 500), ([24, 64, 130, 7], 20000), ([16, 50, 256], 3000), ([16, 50, 257], 3000)])
def test_epoch_fused_gradients(env, kind, dtype, loss, dims, n_loc):
    """What the gradient path forms on the way: the last bias gradient in the loss kernel (up to 256 classes; 257 take a pass
    of their own), the other ones in the weight gradients' products, sigma' where an input gradient is written (aggregation and
    product epilogues: both associations of every layer), the mask counted inside the loss kernel or before it (16384 rows).
    The tolerances are those of every epoch test: the fusion changes orders of summation, not what is rounded."""
    B, H, O = env["B"], env["H"], env["O"]
    cfg = synth.Config(f"fuse-{kind}-{dtype}", kind, n_loc, n_loc // 3, 8 * n_loc, dims, dtype, 1.0, max_deg=300,
                       seed=synth.BASE_SEED * 10 + 9, extra={"loss": loss, "gin_eps": 0.1})
    prob = H.make_problem(cfg, mask_frac=0.5)
    if kind == "gin":       # sums over up to 300 neighbours: keep the activations O(1)
        for p in prob.model:
            p.W *= np.float32(0.125)
    L = len(dims) - 1
    ref = O.oracle_epoch(prob)
    for orders in (None, [B.AGG_FIRST] * L, [B.XFORM_FIRST] * L):
        dp = H.DeviceProblem(prob, orders=orders)
        got, _ = dp.run_epoch()
        compare_epoch(env, prob, dp, ref, got, TOL[dtype], f"{cfg.name} {dims} {loss} orders={orders}")
        dp.close()


def test_epoch_pipelined_host_tier_sees_refilled_tables(env):
    """Pipelined mode copies the host tier for the next epoch while the current one runs.  Every epoch must
    still consume exactly the tables last loaded: after capgnn_cache_fill the prefetched rows are dropped."""
    B, H, O = env["B"], env["H"], env["O"]
    cfg = synth.CONFIGS["C3"].scaled(0.01)
    prob = H.make_problem(cfg, mask_frac=0.5)
    dp = H.DeviceProblem(prob, miss_mode=B.MISS_PIPELINED)
    ref = O.oracle_epoch(prob)
    for rep in range(3):
        loss, times = dp.run_epoch(want_times=(rep == 1))
        compare_epoch(env, prob, dp, ref, loss, TOL["f32"], f"pipelined rep={rep}")
    for l in (1, 0):
        prob.tables[l] = synth.make_features(prob.part.n_halo, cfg.dims[l], seed=991, stream=70 + l, dtype=cfg.dtype)
        dp.cache.fill(l, prob.tables[l])
    ref2 = O.oracle_epoch(prob)
    assert O.normwise(ref2["logits"], ref["logits"]) > 1e-2          # the new tables do change the result
    for rep in range(2):
        loss, _ = dp.run_epoch()
        compare_epoch(env, prob, dp, ref2, loss, TOL["f32"], f"pipelined after refill rep={rep}")
    dp.close()


@pytest.mark.parametrize("miss_mode", [1, 2])
def test_epoch_after_vertex_update_and_staleness_bound(env, miss_mode):
    """Cached halo rows are overwritten between epochs (capgnn_cache_update).  The next epoch must consume
    exactly the updated tables (also when the previous epoch had already prefetched the old ones), and when
    the update moves the last layer's halo rows by at most eps the logits move by at most the staleness
    bound of Lemma 2, eta^2 beta^2 eps (and by the sharper row-wise bound its chain of inequalities gives)."""
    torch, B, H, O = env["torch"], env["B"], env["H"], env["O"]
    cfg = synth.CONFIGS["C2"].scaled(0.02)
    prob = H.make_problem(cfg, mask_frac=0.5)
    part = prob.part
    dp = H.DeviceProblem(prob, miss_mode=miss_mode)
    ref = O.oracle_epoch(prob)
    for rep in range(2):
        loss, _ = dp.run_epoch()
    compare_epoch(env, prob, dp, ref, loss, TOL["f32"], f"before update (miss_mode {miss_mode})")
    logits_before = dp.results()["logits"].astype(np.float64)
    # stale rows: the last layer's halo inputs move by at most eps
    eps, l = 1e-2, dp.L - 1
    rng = np.random.default_rng(3)
    ids = rng.permutation(part.n_halo)[: part.n_halo // 2].astype(np.int64)
    new_rows = (prob.tables[l][ids] + rng.uniform(-eps, eps, (len(ids), cfg.dims[l]))).astype(np.float32)
    moved = float(np.abs(new_rows.astype(np.float64) - prob.tables[l][ids]).max())
    rows_d = H.np_to_dev(new_rows)
    torch.cuda.synchronize()
    B.cache_update(dp.cache, l, torch.from_numpy(ids).cuda(), len(ids), rows_d, cfg.dims[l], 7, stream=dp.stream)
    prob.tables[l][ids] = new_rows
    ref2 = O.oracle_epoch(prob)
    loss2, times2 = dp.run_epoch(want_times=True)
    compare_epoch(env, prob, dp, ref2, loss2, TOL["f32"], f"after update (miss_mode {miss_mode})")
    if miss_mode == B.MISS_PIPELINED:
        # the copy prefetched before the update was patched, not dropped: per layer the only host-tier transfer of
        # this epoch is the prefetch for the next one
        moves = [r["layer"] for r in times2["records"] if r["kind"] == "gather_miss"]
        assert sorted(moves) == list(range(dp.L)), moves
        loss3, _ = dp.run_epoch()                    # consumes the copy fetched after the update
        compare_epoch(env, prob, dp, ref2, loss3, TOL["f32"], "second epoch after update (pipelined)")
    delta = float(np.abs(dp.results()["logits"].astype(np.float64) - logits_before).max())
    W = prob.model[l].W.astype(np.float64)
    eta = max(part.n_cols, W.shape[0], W.shape[1])
    beta = max(1.0, float(np.abs(ref["hidden"][l - 1]).max()), float(np.abs(prob.tables[l]).max()), float(np.abs(W).max()))
    og = O.oracle_graph(part, cfg.kind)
    halo_rowsum = np.array([og.r[i] * og.c[part.col[part.rowptr[i]:part.rowptr[i + 1]]][part.col[part.rowptr[i]:part.rowptr[i + 1]] >= part.n_loc].sum()
                            for i in range(part.n_loc)])
    sharp = halo_rowsum.max() * W.shape[0] * np.abs(W).max() * moved
    say(f"stale rows moved by {moved:.3e}: logits moved by {delta:.3e}; row-wise bound {sharp:.3e}; Lemma 2 bound {eta ** 2 * beta ** 2 * moved:.3e}")
    assert 0 < delta <= sharp * (1 + 1e-3) + 1e-5 <= eta ** 2 * beta ** 2 * moved
    dp.close()


@pytest.mark.parametrize("graph", ["small", "blocked"])
@pytest.mark.parametrize("kind", ["gcn", "sage"])
@pytest.mark.parametrize("order", ["agg", "xform"])
@pytest.mark.parametrize("product", ["auto", "split"])
def test_layer_fwd_bwd_with_halo_gradient(env, kind, order, graph, product):
    """One layer, both association orders, with and without the halo part of the input gradient.  "blocked": a
    dense-degree partition whose operator gets the column-blocked copy in both directions, so the aggregations run the
    blocked kernels, on rows that the producing kernels have multiplied by the per-source weights (GCN) or with unit
    weights (mean aggregator).  "split": every fp32 product in its three-piece form, which these sizes would not pick by
    themselves; a GraphSAGE layer's two forward products then run as one launch over both weight matrices (the first
    reduction range, 50, ends inside a step)."""
    torch, B, H, O, orc = env["torch"], env["B"], env["H"], env["O"], env["orc"]
    if graph == "small":
        part = synth.make_partition("layer", 900, 700, 12000, seed=41, max_deg=2500, self_loops=(kind == "gcn"))
    else:
        part = synth.make_partition("layer-blk", 37000, 36000, 5200000, seed=43, max_deg=4000, halo_edge_frac=0.5,
                                    self_loops=(kind == "gcn"))
    fi, fo = 50, 36
    rng = np.random.default_rng(7)
    X = rng.standard_normal((part.n_cols, fi)).astype(np.float32)
    W = (rng.standard_normal((fi, fo)) * 0.2).astype(np.float32)
    Ws = (rng.standard_normal((fi, fo)) * 0.2).astype(np.float32) if kind == "sage" else None
    b = rng.standard_normal(fo).astype(np.float32)
    dH = rng.standard_normal((part.n_loc, fo)).astype(np.float32)
    og = O.oracle_graph(part, kind)
    ol = orc.Layer(kind, W.astype(np.float64), b.astype(np.float64), "relu", None if Ws is None else Ws.astype(np.float64))
    Href, saved = orc.layer_fwd(og, ol, X.astype(np.float64))
    bref = orc.layer_bwd(og, ol, X.astype(np.float64), saved, dH.astype(np.float64), need_dx=True)

    r, c = B.norm_scales(B.NORM_SYM if kind == "gcn" else B.NORM_MEAN, part.n_loc, part.n_halo, part.rowptr, part.halo_degree)
    g = B.Graph(part.n_loc, part.n_halo, part.rowptr, part.col, r, c)
    Wd, Wsd, bd = H.np_to_dev(W), (None if Ws is None else H.np_to_dev(Ws)), H.np_to_dev(b)
    ly = B.make_layer(B.GCN if kind == "gcn" else B.SAGE_MEAN, fi, fo, B.ACT_RELU, B.F32, Wd, Wsd, bd,
                      B.AGG_FIRST if order == "agg" else B.XFORM_FIRST,
                      f32_product=B.F32_PRODUCT_SPLIT if product == "split" else B.F32_PRODUCT_AUTO)
    ldx, ldh = 52, 36
    Xd = H.padded_matrix(X, ldx)
    Hd = torch.zeros((part.n_loc, ldh), device="cuda")
    saved_d = torch.empty(max(B.layer_saved_bytes(g, ly), 256), dtype=torch.uint8, device="cuda")
    wsb = B.layer_workspace_bytes(g, ly)
    ws = torch.empty(max(wsb, 256), dtype=torch.uint8, device="cuda")
    B.layer_fwd(g, ly, Xd, ldx, Hd, ldh, saved_d, ws, wsb)
    torch.cuda.synchronize()
    Hgot = Hd.cpu().numpy()
    assert O.normwise(Hgot, Href) <= TOL["f32"] and O.elementwise(Hgot, Href, by_row=True) <= TOL["f32"]
    # backward from the oracle's own forward output: its sign pattern is the oracle's sigma', so no decision can differ
    Hd = H.padded_matrix(Href.astype(np.float32), ldh)
    assert np.array_equal(Href.astype(np.float32) > 0, saved["Z"] > 0)
    for need_halo in (True, False):
        dHd = H.np_to_dev(dH)
        dW, dWs, db = torch.zeros_like(Wd), (None if Ws is None else torch.zeros_like(Wd)), torch.zeros_like(bd)
        rows = part.n_cols if need_halo else part.n_loc
        dX = torch.full((rows, ldx), 5.0, device="cuda")
        B.layer_bwd(g, ly, Xd, ldx, Hd, ldh, saved_d, dHd, fo, dW, dWs, db, dX, ldx, need_halo, ws, wsb)
        torch.cuda.synchronize()
        say(f"layer {kind} {order} need_halo={need_halo}")
        for name, a, want in (("dW", dW, bref["dW"]), ("db", db, bref["db"])) + ((("dWs", dWs, bref["dW_self"]),) if Ws is not None else ()):
            assert O.normwise(a.cpu().numpy(), want) <= TOL["f32"] and O.rowwise(a.cpu().numpy(), want) <= TOL["f32"], name
        got = dX.cpu().numpy()
        assert O.normwise(got[:, :fi], bref["dX"][:rows]) <= TOL["f32"]
        assert O.elementwise(got[:, :fi], bref["dX"][:rows], by_row=True) <= TOL["f32"]
        assert (got[:, fi:] == 5.0).all()
    g.close()


def test_epoch_sgd_step_and_no_halo(env):
    """Partition without halo vertices (cache is NULL) and the in-place W <- W - lr dW update."""
    torch, B, H, O = env["torch"], env["B"], env["H"], env["O"]
    cfg = synth.Config("nohalo", "gcn", 3000, 0, 30000, [40, 32, 5], "f32", 0.0, max_deg=400, symmetric=True, seed=77)
    prob = H.make_problem(cfg, mask_frac=0.7)
    dp = H.DeviceProblem(prob)
    ref = O.oracle_epoch(prob, lr=0.05)
    loss, _ = dp.run_epoch(lr=0.05)
    compare_epoch(env, prob, dp, ref, loss, TOL["f32"], "no-halo symmetric")
    torch.cuda.synchronize()
    for l in range(dp.L):
        assert O.normwise(H.dev_to_np(dp.W[l]), ref["new_W"][l]) <= TOL["f32"]
        assert O.normwise(H.dev_to_np(dp.bias[l]), ref["new_bias"][l]) <= TOL["f32"]
    dp.close()


def test_epoch_rejects_bad_arguments(env):
    torch, B, H = env["torch"], env["B"], env["H"]
    import copy
    cfg = copy.deepcopy(synth.CONFIGS["C1"]).scaled(0.1)
    prob = H.make_problem(cfg)
    dp = H.DeviceProblem(prob)
    with pytest.raises(B.CapgnnError) as e:       # workspace too small
        B.epoch(dp.graph, dp.cache, dp.layers, dp.X0, dp.ld0, dp.labels, dp.mask, 0.0, dp.logits, dp.dW, None,
                dp.dbias, 0.0, dp.ws, 1024, dp.stream, dp.side)
    assert e.value.code == B.ENOMEM
    with pytest.raises(B.CapgnnError) as e:       # halo vertices but no cache
        B.epoch(dp.graph, None, dp.layers, dp.X0, dp.ld0, dp.labels, dp.mask, 0.0, dp.logits, dp.dW, None,
                dp.dbias, 0.0, dp.ws, dp.ws_bytes, dp.stream, dp.side)
    assert e.value.code == B.EINVAL
    dp.close()


@pytest.mark.parametrize("case", ["C1", "C2-host-tier", "C1-sgd"])
def test_epoch_graph_replays_match_eager_epochs(env, case):
    """capgnn_epoch recorded as a HIP graph: every replay must give exactly what the eager epoch gives on the same buffer
    contents (same kernels, same order: bit for bit), also after the buffers' contents changed between replays (a cache
    update), with eager work and synchronisations between the replays, and with host-tier rows travelling inside the
    graph.  The first eager result is compared with the oracle."""
    torch, B, H, O = env["torch"], env["B"], env["H"], env["O"]
    if case == "C2-host-tier":
        cfg = synth.CONFIGS["C2"].scaled(0.02)
        prob = H.make_problem(cfg, mask_frac=0.5)
    else:
        cfg = synth.CONFIGS["C1"]
        prob = H.make_problem(cfg, mask_frac=0.5)
    lr = 0.05 if case == "C1-sgd" else 0.0
    part = prob.part
    # the eager side runs on one stream too (no side stream), as the recorded epoch does
    dp = H.DeviceProblem(prob, miss_mode=B.MISS_STAGED, use_side_stream=False)
    ref = O.oracle_epoch(prob)

    def snapshot():
        r = dp.results()
        return [r["logits"].copy()] + [a.copy() for a in r["dW"]] + [a.copy() for a in r["db"]]

    W0 = [w.clone() for w in dp.W]
    b0 = [b.clone() for b in dp.bias]

    def reset_weights():
        for w, w0 in zip(dp.W, W0):
            w.copy_(w0)
        for b, bb in zip(dp.bias, b0):
            b.copy_(bb)
        torch.cuda.synchronize()

    # eager: three epochs (with the SGD step they differ), a cache update before the third
    rng = np.random.default_rng(11)
    l_upd = dp.L - 1
    ids = rng.permutation(part.n_halo)[: max(part.n_halo // 3, 1)].astype(np.int64)
    new_rows = rng.standard_normal((len(ids), cfg.dims[l_upd])).astype(np.float32)
    ids_d, rows_d = torch.from_numpy(ids).cuda(), H.np_to_dev(new_rows)
    old_rows_d = H.np_to_dev(np.ascontiguousarray(prob.tables[l_upd][ids]))
    eager = []
    for it in range(3):
        if it == 2:
            B.cache_update(dp.cache, l_upd, ids_d, len(ids), rows_d, cfg.dims[l_upd], 5, stream=dp.stream)
        loss, _ = dp.run_epoch(lr=lr)
        eager.append((loss, snapshot()))
        if it == 0:
            compare_epoch(env, prob, dp, ref, loss, TOL["f32"], f"graph case {case}: eager epoch")
    # back to the start: weights, cache rows
    B.cache_update(dp.cache, l_upd, ids_d, len(ids), old_rows_d, cfg.dims[l_upd], 6, stream=dp.stream)
    reset_weights()
    for t in [dp.logits] + dp.dW + dp.dbias:
        t.zero_()
    torch.cuda.synchronize()

    eg, loss_dev = dp.capture_epoch(lr=lr)
    assert np.isnan(loss_dev.cpu().numpy()[0]) and not dp.logits.any()        # recording ran nothing
    scratch = torch.empty(1 << 20, device="cuda")
    for it in range(3):
        if it == 2:
            B.cache_update(dp.cache, l_upd, ids_d, len(ids), rows_d, cfg.dims[l_upd], 7, stream=dp.stream)
        eg.launch(dp.stream)
        torch.cuda.synchronize()
        got = snapshot()
        loss_g = float(loss_dev.cpu().numpy()[0])
        scratch.normal_()                        # the program's own eager work between the replays
        _ = float(scratch.sum().cpu())
        say(f"graph case {case}: replay {it}: loss {loss_g:.6f} (eager {eager[it][0]:.6f})")
        assert loss_g == eager[it][0], (it, loss_g, eager[it][0])
        for a, b in zip(got, eager[it][1]):
            assert np.array_equal(a, b), f"replay {it} differs from the eager epoch"
    if lr == 0.0:
        assert not np.array_equal(eager[2][1][0], eager[1][1][0])      # the update did change the result
    else:
        assert not np.array_equal(eager[1][1][0], eager[0][1][0])      # and so did the SGD step
    eg.close()
    with pytest.raises(B.CapgnnError):
        B.EpochGraph(dp.graph, dp.cache, dp.layers, dp.X0, dp.ld0, dp.labels, dp.mask, 0.0, dp.logits, dp.dW, None, dp.dbias,
                     0.0, None, dp.ws, dp.ws_bytes, None)             # the default stream cannot be captured
    # the stream is usable after the failed call, and after a successful capture
    loss, _ = dp.run_epoch(lr=0.0)
    assert np.isfinite(loss)
    dp.close()


@pytest.mark.parametrize("kind", ["gcn", "sage"])
def test_training_run_tracks_the_oracle(env, kind):
    """Twelve epochs with the in-place step W <- W - lr * dW (the update of the convergence theorem's proof): the loss of
    every epoch and the weights at the end must follow the oracle's own fp64 training run, which carries its weights in
    fp64 from step to step and takes nothing from the GPU.  The loss must also go down in the oracle's run: a sign error
    in the step would show there first."""
    torch, B, H, O, orc = env["torch"], env["B"], env["H"], env["O"], env["orc"]
    cfg = synth.Config(f"train-{kind}", kind, 2500, 1800, 40000, [48, 32, 7], "f32", 0.5, max_deg=600, seed=91)
    prob = H.make_problem(cfg, mask_frac=0.6)
    dp = H.DeviceProblem(prob, miss_mode=B.MISS_PIPELINED)
    lr, steps = 0.2, 12
    og = O.oracle_graph(prob.part, kind)
    layers = O.oracle_layers(prob)
    tables = [O.widen(t) for t in prob.tables]
    X0 = O.widen(prob.X0)
    ref_losses, gpu_losses = [], []
    for it in range(steps):
        ref = orc.epoch(og, layers, X0, tables, prob.labels, prob.mask, 0.0, lr)
        ref_losses.append(ref["loss"])
        for l, ly in enumerate(layers):
            ly.W = ref["new_W"][l]
            ly.bias = ref["new_bias"][l]
            if ly.W_self is not None:
                ly.W_self = ref["new_W_self"][l]
        loss, _ = dp.run_epoch(lr=lr)
        gpu_losses.append(loss)
    say(f"training {kind}: oracle loss {ref_losses[0]:.5f} -> {ref_losses[-1]:.5f}, GPU {gpu_losses[0]:.5f} -> {gpu_losses[-1]:.5f}")
    assert all(b < a for a, b in zip(ref_losses, ref_losses[1:])), ref_losses
    for a, b in zip(gpu_losses, ref_losses):
        assert abs(a - b) <= 1e-4 * max(1.0, abs(b)), (gpu_losses, ref_losses)
    torch.cuda.synchronize()
    for l, ly in enumerate(layers):
        assert O.normwise(H.dev_to_np(dp.W[l]), ly.W) <= 1e-3, l
        assert O.normwise(H.dev_to_np(dp.bias[l]), ly.bias) <= 1e-3, l
        if ly.W_self is not None:
            assert O.normwise(H.dev_to_np(dp.W_self[l]), ly.W_self) <= 1e-3, l
    dp.close()


@pytest.mark.parametrize("miss_mode", [1, 2])
def test_epoch_graph_with_side_stream_matches_eager_epochs(env, miss_mode):
    """The two-stream epoch recorded as a HIP graph (host-tier rows on the side stream; in pipelined mode every replay
    consumes what the run before it prefetched and prefetches for the next).  Replays must equal eager epochs bit for bit:
    on the static tables, after a cache update between replays (which patches the prefetched copy), and after a refill
    followed by one eager epoch that primes the prefetch again; recording a pipelined epoch that nothing has primed is an
    argument error, and eager epochs after the replays still see the right rows."""
    torch, B, H, O = env["torch"], env["B"], env["H"], env["O"]
    cfg = synth.CONFIGS["C2"].scaled(0.02)
    prob = H.make_problem(cfg, mask_frac=0.5)
    part = prob.part
    dp = H.DeviceProblem(prob, miss_mode=miss_mode)
    ref = O.oracle_epoch(prob)

    def snapshot():
        r = dp.results()
        return [r["logits"].copy()] + [a.copy() for a in r["dW"]] + [a.copy() for a in r["db"]]

    if miss_mode == B.MISS_PIPELINED:
        with pytest.raises(B.CapgnnError):
            dp.capture_epoch(two_streams=True)                   # nothing has prefetched the host tier yet
    loss0, _ = dp.run_epoch()
    compare_epoch(env, prob, dp, ref, loss0, TOL["f32"], f"two-stream graph (miss_mode {miss_mode}): eager epoch")
    base = snapshot()
    eg, loss_dev = dp.capture_epoch(two_streams=True)
    scratch = torch.empty(1 << 20, device="cuda")
    for it in range(3):
        eg.launch(dp.stream)
        torch.cuda.synchronize()
        scratch.normal_()
        _ = float(scratch.sum().cpu())
        assert float(loss_dev.cpu()[0]) == loss0
        for a, b in zip(snapshot(), base):
            assert np.array_equal(a, b), f"replay {it} differs from the eager epoch"
    # rows rewritten between replays, in both tiers
    rng = np.random.default_rng(17)
    l_upd = dp.L - 1
    ids = rng.permutation(part.n_halo)[: part.n_halo // 2].astype(np.int64)
    new_rows = rng.standard_normal((len(ids), cfg.dims[l_upd])).astype(np.float32)
    B.cache_update(dp.cache, l_upd, torch.from_numpy(ids).cuda(), len(ids), H.np_to_dev(new_rows), cfg.dims[l_upd], 3,
                   stream=dp.stream)
    prob.tables[l_upd][ids] = new_rows
    ref2 = O.oracle_epoch(prob)
    for it in range(2):
        eg.launch(dp.stream)
        torch.cuda.synchronize()
        compare_epoch(env, prob, dp, ref2, float(loss_dev.cpu()[0]), TOL["f32"], f"two-stream graph after update, replay {it}")
    upd = snapshot()
    loss_e, _ = dp.run_epoch()                                   # an eager epoch after the replays: same rows, same result
    for a, b in zip(snapshot(), upd):
        assert np.array_equal(a, b)
    # a refill drops the prefetched copy: one eager epoch primes it again, then the replays see the new table
    prob.tables[0] = synth.make_features(part.n_halo, cfg.dims[0], seed=5, stream=3, dtype=cfg.dtype)
    dp.cache.fill(0, prob.tables[0])
    ref3 = O.oracle_epoch(prob)
    loss3, _ = dp.run_epoch()
    compare_epoch(env, prob, dp, ref3, loss3, TOL["f32"], "two-stream graph: eager epoch after refill")
    want = snapshot()
    for it in range(2):
        eg.launch(dp.stream)
        torch.cuda.synchronize()
        for a, b in zip(snapshot(), want):
            assert np.array_equal(a, b), f"replay {it} after refill differs"
    eg.close()
    dp.close()


@pytest.mark.parametrize("kind,dtype", [("gcn", "f32"), ("gin", "f32"), ("gcn", "bf16")])
@pytest.mark.parametrize("n,classes,share", [(210_007, 17, 0.5), (110_003, 40, 0.0), (110_003, 47, 0.1), (110_003, 100, 0.8), (110_003, 130, 0.5),
                                             (110_003, 47, 0.9), (110_003, 47, 1.0)])
def test_epoch_gradient_rows_outside_the_loss_are_skipped(env, kind, dtype, n, classes, share):
    """A graph large enough for the last layer's transposed aggregation to skip the rows of dZ outside the training mask (one and
    several vectors per row, pieces of long rows, rows without entries, a mask that ends inside a word; above 85 % live rows every
    row is read).  dW of a linear one-layer model against X^T A^T dZ in float64 from the logits that the epoch itself returned:
    float32 sums of 34-entry rows and of n products of either sign (1e-5 of the norm), and for bf16 one more rounding of each
    element of A^T dZ (2^-9 at most)."""
    import scipy.sparse as sp
    torch, B = env["torch"], env["B"]
    rng = np.random.default_rng(7)
    deg = rng.integers(0, 69, n)
    deg[rng.integers(0, n, 5)] = 30_000
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    nnz = int(rowptr[-1])
    assert nnz >= 32 * n
    col = rng.integers(0, n, nnz).astype(np.int32)
    val = rng.uniform(0.5, 1.5, nnz).astype(np.float32) if kind == "gin" else None
    r, c = (None, None) if kind == "gin" else (rng.uniform(0.1, 0.3, n).astype(np.float32), rng.uniform(0.5, 1.5, n).astype(np.float32))
    g = B.Graph(n, 0, rowptr, col, r, c, val, 0)
    f_in, dt = 24, torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.randn(n, f_in, device="cuda").to(dt)
    w = (0.05 * torch.randn(f_in, classes, device="cuda")).to(dt)
    layer = B.make_layer(B.GCN, f_in, classes, B.ACT_NONE, B.BF16 if dtype == "bf16" else B.F32, w, None, None, B.XFORM_FIRST,
                         out_f32=int(dtype == "bf16"))
    labels = torch.randint(0, classes, (n,), device="cuda", dtype=torch.int32)
    mask = torch.from_numpy((rng.random(n) < share).astype(np.uint8)).cuda()
    logits, dw = torch.zeros(n, classes, device="cuda"), torch.zeros(f_in, classes, device="cuda")
    db = torch.zeros(classes, device="cuda")
    size = B.epoch_workspace_bytes(g, None, [layer])
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    for norm in (0.0, 1000.0):      # the normaliser counted, and given
        B.epoch(g, None, [layer], x, f_in, labels, mask, norm, logits, [dw], None, [db], 0.0, ws, size)
        torch.cuda.synchronize()
        z = logits.cpu().double()
        on = mask.cpu().double()
        dz = (torch.softmax(z, 1) - torch.nn.functional.one_hot(labels.cpu().long(), classes)) * on[:, None] / (norm or max(float(on.sum()), 1.0))
        a = sp.csr_matrix((np.ones(nnz) if val is None else val.astype(np.float64), col, rowptr), shape=(n, n))
        t = dz.numpy() if r is None else dz.numpy() * r[:, None].astype(np.float64)
        t = a.T @ t
        if c is not None:
            t *= c[:, None].astype(np.float64)
        ref = x.cpu().double().numpy().T @ t
        err = np.linalg.norm(dw.cpu().double().numpy() - ref) / max(np.linalg.norm(ref), 1e-30)
        say(f"rows skipped: {kind} {dtype} {n}x{classes} share {share} norm {norm}: {err:.2e}")
        assert err <= (1e-5 if dtype == "f32" else 2.0 ** -9) if share else not dw.any()


@pytest.mark.parametrize("n,hidden,classes", [(30_017, 100, 47), (30_016, 200, 47), (30_001, 200, 121), (66_001, 125, 47), (30_017, 130, 41), (30_017, 255, 100)])
def test_epoch_masked_sum_of_two_split_products(env, n, hidden, classes):
    """The input gradient of a transform-first GraphSAGE layer under the ReLU of the layer below, one launch over both weight matrices with the
    mask in its epilogue: with the weights in registers (one and two waves to a reduction, whole and ragged groups of columns) and in
    tiles.  Self loops only, so the lower layer's gradients are x^T (dZ (W + W_self)^T masked) and its column sums: each column against
    float64 with the epoch's own hidden layer and logits, 2e-6 of the largest (sums of up to 66000 terms in splits of 200 and a few float
    roundings before them; 2e-7 measured)."""
    torch, B = env["torch"], env["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + hidden)
    mk = lambda *s: torch.randn(*s, generator=gen, device="cuda")  # noqa: E731
    f_in = 24
    g = B.Graph(n, 0, np.arange(n + 1, dtype=np.int64), np.arange(n, dtype=np.int32), np.ones(n, np.float32), None)
    x, w, w_self = mk(n, f_in), [mk(f_in, hidden) / 5, mk(hidden, classes) / 10], [mk(f_in, hidden) / 5, mk(hidden, classes) / 10]
    b = [mk(hidden) / 5, mk(classes) / 5]
    layers = [B.make_layer(B.SAGE_MEAN, f_in, hidden, B.ACT_RELU, B.F32, w[0], w_self[0], b[0], B.AGG_FIRST, f32_product=B.F32_PRODUCT_SPLIT),
              B.make_layer(B.SAGE_MEAN, hidden, classes, B.ACT_NONE, B.F32, w[1], w_self[1], b[1], B.XFORM_FIRST, f32_product=B.F32_PRODUCT_SPLIT)]
    labels = torch.randint(0, classes, (n,), generator=gen, device="cuda", dtype=torch.int32)
    dw, ds, db = ([torch.zeros_like(t) for t in v] for v in (w, w_self, b))
    logits = torch.zeros(n, classes, device="cuda")
    ws = torch.empty(B.epoch_workspace_bytes(g, None, layers), dtype=torch.uint8, device="cuda")
    say(f"masked sum of two products {n} {hidden} {classes}")
    B.epoch(g, None, layers, x, f_in, labels, None, 0.0, logits, dw, ds, db, 0.0, ws, ws.numel())
    torch.cuda.synchronize()
    at, ld = B.epoch_activation(g, None, layers, 0, ws)
    at -= ws.data_ptr()
    h = ws[at:at + 4 * n * ld].view(torch.float32).view(n, ld)[:, :hidden]
    assert float((h.double() - (x.double() @ (w[0] + w_self[0]).double() + b[0].double()).clamp(min=0)).norm()) <= 1e-6 * float(h.double().norm())
    dz = torch.softmax(logits.double(), 1)
    dz[torch.arange(n, device="cuda"), labels.long()] -= 1
    dz0 = (dz / n) @ (w[1].double() + w_self[1].double()).T * (h > 0)
    for got, ref in ((dw[0], x.double().T @ dz0), (ds[0], x.double().T @ dz0), (db[0], dz0.sum(0))):
        e = float((got.double() - ref).abs().max() / ref.abs().max())
        say(f"   {e:.2e}")
        assert e <= 2e-6
    g.close()


@pytest.mark.parametrize("kind,dtype,lr", [("sage", "f32", 0.0), ("sage", "f32", 0.1), ("gcn", "f32", 0.0), ("gcn", "bf16", 0.0)])
def test_timed_epoch_keeps_every_stage_its_own_work(env, kind, dtype, lr):
    """The records of a timed epoch whose weight gradients are sums over parts: one loss record, forward and backward products for every
    layer; GraphSAGE, which needs no pass over a gradient alone, has an elementwise record where there is an update and no other.  Results are
    the same bits as those of an epoch without times, which leaves the sums to its end."""
    torch, B = env["torch"], env["B"]
    rng = np.random.default_rng(5)
    n, dims, L = 3001, (40, 32, 24, 7), 3
    dt, code = (torch.bfloat16, B.BF16) if dtype == "bf16" else (torch.float32, B.F32)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    mk = lambda *s: (torch.randn(*s, generator=gen, device="cuda") / 5).to(dt)  # noqa: E731
    g = B.Graph(n, 0, np.arange(0, 4 * n + 1, 4, dtype=np.int64), rng.integers(0, n, 4 * n).astype(np.int32), np.full(n, 0.25, np.float32), None)
    w, w_self = [mk(a, b) for a, b in zip(dims, dims[1:])], [mk(a, b) for a, b in zip(dims, dims[1:])]
    b = [torch.randn(d, generator=gen, device="cuda") for d in dims[1:]]
    x, labels = mk(n, dims[0]), torch.randint(0, dims[-1], (n,), generator=gen, device="cuda", dtype=torch.int32)
    order = B.AGG_FIRST if kind == "sage" else B.XFORM_FIRST
    sage = kind == "sage"
    start = [t.clone() for t in w + w_self + b]
    outs = []
    for timed in (False, True):
        say(f"timed epoch {kind} {dtype} lr={lr} timed={timed}")
        for t, s in zip(w + w_self + b, start): t.copy_(s)
        layers = [B.make_layer(B.SAGE_MEAN if sage else B.GCN, dims[l], dims[l + 1], B.ACT_RELU if l < L - 1 else B.ACT_NONE, code, w[l],
                               w_self[l] if sage else None, b[l], order, out_f32=int(l == L - 1 and dtype == "bf16")) for l in range(L)]
        ws = torch.empty(B.epoch_workspace_bytes(g, None, layers), dtype=torch.uint8, device="cuda")
        dw, ds = ([torch.zeros(a, c, device="cuda") for a, c in zip(dims, dims[1:])] for _ in range(2))
        db, logits = [torch.zeros(d, device="cuda") for d in dims[1:]], torch.zeros(n, dims[-1], device="cuda")
        loss, times = B.epoch(g, None, layers, x, dims[0], labels, None, 0.0, logits, dw, ds if sage else None, db, lr, ws, ws.numel(), want_times=timed)
        outs.append([*(t.clone() for t in dw + ds + db + w + w_self + b + [logits]), torch.tensor(loss)])
    kinds = [(r["kind"], r["layer"], r["backward"]) for r in times["records"]]
    assert kinds.count(("loss", L - 1, 0)) == 1
    assert all((k, l, bw) in kinds for l in range(L) for k, bw in (("gemm", 0), ("gemm", 1)))
    passes = [k for k in kinds if k[0] == "elementwise"]
    if sage: assert passes == ([("elementwise", 0, 1)] if lr else []) and (times["other_ms"] > 0) == bool(lr)
    assert all(torch.equal(p, q) for p, q in zip(*outs))


@pytest.mark.parametrize("kind,dtype", [("gcn", "f32"), ("sage", "f32"), ("gcn", "bf16"), ("sage", "bf16")])
@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("n,dims", [(37, (33, 64, 5)), (1003, (100, 32, 70)), (9001, (64, 128, 30, 7)), (33_001, (40, 31, 9))])
def test_small_products_of_a_layer_in_one_launch(env, kind, dtype, order, n, dims):
    """The small weight and input gradients of a layer run as one launch; an epoch that records its stages' times runs them one by one: the same
    parts, added up in another order (the gradients differ by fp32 rounding of sums of at most 512 parts, random: far below 2e-6).  The last
    size has reductions too long for the batch."""
    torch, B = env["torch"], env["B"]
    sage, bf = kind == "sage", dtype == "bf16"
    td, dt = (torch.bfloat16, B.BF16) if bf else (torch.float32, B.F32)
    rng = np.random.default_rng(n)
    deg = rng.integers(1, 5, n)
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    col = rng.integers(0, n, rowptr[-1]).astype(np.int32)
    g = B.Graph(n, 0, rowptr, col, (1.0 / deg).astype(np.float32), np.ones(n, np.float32))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    mk = lambda a, b: (torch.randn(a, b, generator=gen, device="cuda") / a ** 0.5).to(td)  # noqa: E731
    ld = -(-dims[0] // 8) * 8
    x = torch.zeros(n, ld, device="cuda", dtype=td)
    x[:, :dims[0]] = torch.randn(n, dims[0], generator=gen, device="cuda").to(td)
    L = len(dims) - 1
    w, ws_ = ([mk(a, b) for a, b in zip(dims, dims[1:])] for _ in range(2))
    b = [0.1 * torch.randn(d, generator=gen, device="cuda") for d in dims[1:]]
    labels = torch.randint(0, dims[-1], (n,), generator=gen, device="cuda", dtype=torch.int32)
    layers = [B.make_layer(B.SAGE_MEAN if sage else B.GCN, dims[i], dims[i + 1], B.ACT_NONE if i == L - 1 else B.ACT_RELU, dt, w[i], ws_[i] if sage else None,
                           b[i], order, out_f32=int(bf and i == L - 1)) for i in range(L)]
    wsb = B.epoch_workspace_bytes(g, None, layers)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    out = []
    for timed in (False, True):
        grads = [[torch.full((p, q), 7.0, device="cuda") for p, q in zip(dims, dims[1:])] for _ in range(2)] + [[torch.full((d,), 7.0, device="cuda") for d in dims[1:]]]
        logits = torch.zeros(n, dims[-1], device="cuda")
        print(f"small products in one launch {kind} {dtype} order={order} n={n} {dims} timed={timed}", flush=True)
        B.epoch(g, None, layers, x, ld, labels, None, 0.0, logits, grads[0], grads[1] if sage else None, grads[2], 0.0, ws, wsb, None, None, want_times=timed)
        torch.cuda.synchronize()
        out.append([t.double() for part in (grads if sage else [grads[0], grads[2]]) for t in part] + [logits.double()])
    for p, q in zip(*out):
        assert float((p - q).norm()) <= 2e-6 * float(q.norm())


@pytest.mark.parametrize("kind,dtype", [("gcn", "f32"), ("sage", "f32"), ("gcn", "bf16"), ("sage", "bf16")])
@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("n,dims", [(1003, (100, 32, 70)), (9001, (64, 128, 30, 7))])
def test_epoch_of_small_products_against_float64(env, kind, dtype, order, n, dims):
    """An untimed epoch, whose layers run their small products as one launch and whose loss reaches the host by the last kernel, and a timed one,
    whose loss is copied: losses alike, and both, with gradients and logits, as float64 has them as far as pre-activations within rounding
    of zero let them: one that changes sides moves a gradient by up to 1e-3 (fp32), bf16 roundings through three layers by up to 6e-2; a
    product taken for another is off by 1."""
    torch, B = env["torch"], env["B"]
    sage, bf, L = kind == "sage", dtype == "bf16", len(dims) - 1
    td, dt = (torch.bfloat16, B.BF16) if bf else (torch.float32, B.F32)
    rng = np.random.default_rng(n)
    deg = rng.integers(1, 5, n)
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    col = rng.integers(0, n, rowptr[-1]).astype(np.int32)
    g = B.Graph(n, 0, rowptr, col, (1.0 / deg).astype(np.float32), np.ones(n, np.float32))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    ld = -(-dims[0] // 8) * 8
    x = torch.zeros(n, ld, device="cuda", dtype=td)
    x[:, :dims[0]] = torch.randn(n, dims[0], generator=gen, device="cuda").to(td)
    w, w_self = ([(torch.randn(p, q, generator=gen, device="cuda") / p ** 0.5).to(td) for p, q in zip(dims, dims[1:])] for _ in range(2))
    b = [0.1 * torch.randn(d, generator=gen, device="cuda") for d in dims[1:]]
    labels = torch.randint(0, dims[-1], (n,), generator=gen, device="cuda", dtype=torch.int32)
    layers = [B.make_layer(B.SAGE_MEAN if sage else B.GCN, dims[i], dims[i + 1], B.ACT_NONE if i == L - 1 else B.ACT_RELU, dt, w[i],
                           w_self[i] if sage else None, b[i], order, out_f32=int(bf and i == L - 1)) for i in range(L)]
    size = B.epoch_workspace_bytes(g, None, layers)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    dst, src = torch.arange(n, device="cuda").repeat_interleave(torch.from_numpy(deg).cuda()), torch.from_numpy(col).cuda().long()
    leaf = [[t.detach().double().requires_grad_() for t in part] for part in (w, w_self, b)]
    h = x[:, :dims[0]].double()
    for i in range(L):
        m = torch.zeros_like(h).index_add(0, dst, h[src] / torch.from_numpy(deg).cuda()[dst].double()[:, None])
        z = m @ leaf[0][i] + leaf[2][i] + (h @ leaf[1][i] if sage else 0)
        h = z.clamp(min=0) if i < L - 1 else z
    ref_loss = torch.nn.functional.cross_entropy(z, labels.long())
    ref_loss.backward()
    ref = [t.grad for part in (leaf if sage else [leaf[0], leaf[2]]) for t in part] + [z.detach()]
    losses, bound = [], 6e-2 if bf else 1e-3
    for timed in (False, True):
        grads = [[torch.full((p, q), 7.0, device="cuda") for p, q in zip(dims, dims[1:])] for _ in range(2)] + [[torch.full((d,), 7.0, device="cuda") for d in dims[1:]]]
        logits = torch.zeros(n, dims[-1], device="cuda")
        say(f"epoch of small products against float64 {kind} {dtype} order={order} n={n} {dims} timed={timed}")
        losses.append(B.epoch(g, None, layers, x, ld, labels, None, 0.0, logits, grads[0], grads[1] if sage else None, grads[2], 0.0, ws, size, None, None,
                              want_times=timed)[0])
        torch.cuda.synchronize()
        got = [t for part in (grads if sage else [grads[0], grads[2]]) for t in part] + [logits]
        err = [float((p.double() - q).norm() / q.norm()) for p, q in zip(got, ref)]
        assert max(err) <= bound and abs(losses[-1] - float(ref_loss)) <= bound * float(ref_loss), (err, losses)
    assert abs(losses[0] - losses[1]) <= 2e-6 * losses[1]
    g.close()


def test_epochs_of_one_graph_in_many_threads_return_their_own_loss(env):
    """Twenty threads, each with a stream, workspace, labels and results of its own, run epochs of one graph at the same time: more than the graph has
    pinned lines for their losses, so some come by a copy.  Each epoch returns the loss of its own labels, the one that it returned alone."""
    import threading
    torch, B = env["torch"], env["B"]
    n, dims, T, reps = 20_011, (64, 32, 9), 20, 6
    rng = np.random.default_rng(5)
    deg = rng.integers(1, 9, n)
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    g = B.Graph(n, 0, rowptr, rng.integers(0, n, rowptr[-1]).astype(np.int32), (1.0 / deg).astype(np.float32), np.ones(n, np.float32))
    x = torch.randn(n, dims[0], device="cuda")
    w, b = [torch.randn(p, q, device="cuda") / p ** 0.5 for p, q in zip(dims, dims[1:])], [0.1 * torch.randn(q, device="cuda") for q in dims[1:]]
    layers = [B.make_layer(B.GCN, dims[i], dims[i + 1], B.ACT_NONE if i else B.ACT_RELU, B.F32, w[i], None, b[i]) for i in range(2)]
    size = B.epoch_workspace_bytes(g, None, layers)
    own = [dict(labels=torch.randint(0, 2 + t % 8, (n,), device="cuda", dtype=torch.int32), ws=torch.empty(size, dtype=torch.uint8, device="cuda"),
                dw=[torch.zeros_like(m) for m in w], db=[torch.zeros_like(m) for m in b], logits=torch.zeros(n, dims[-1], device="cuda"), st=torch.cuda.Stream())
           for t in range(T)]
    torch.cuda.synchronize()
    run = lambda o: B.epoch(g, None, layers, x, dims[0], o["labels"], None, 0.0, o["logits"], o["dw"], None, o["db"], 0.0, o["ws"], size, o["st"])[0]  # noqa: E731
    alone = []
    for t, o in enumerate(own):
        alone.append(run(o))
        ref = float(torch.nn.functional.cross_entropy(o["logits"].double(), o["labels"].long()))
        assert abs(alone[-1] - ref) <= 1e-5 * ref, (t, alone[-1], ref)       # a mean of 20 k terms, each a few fp32 roundings
        o["first"] = [m.clone() for m in o["dw"] + o["db"]]
    assert len(set(alone)) == T
    torch.cuda.synchronize()
    say(f"{T} threads, {reps} epochs each")
    got, start = [[] for _ in range(T)], threading.Barrier(T)

    def work(t):
        start.wait()
        for _ in range(reps): got[t].append(run(own[t]))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(T)]
    for t in threads: t.start()
    for t in threads: t.join()
    torch.cuda.synchronize()
    assert got == [[a] * reps for a in alone]
    assert all(torch.equal(p, q) for o in own for p, q in zip(o["dw"] + o["db"], o["first"]))
    assert run(own[0]) == alone[0]
    g.close()


@pytest.mark.parametrize("recorded", [False, True])
@pytest.mark.parametrize("L,shared", [(2, "none"), (3, "dw"), (3, "bias"), (16, "none"), (16, "dw")])
def test_epoch_end_adds_up_every_gradient(env, L, shared, recorded):
    """What an epoch leaves to its last launch: the loss, every gradient and the SGD step, with up to 16 GraphSAGE layers (more sums than
    one launch takes), and with gradient buffers that layers share, which hold the first layer's in the end, as the backward pass
    writes it last.  Three passes with eager work between them; each equals the separate layer calls' order of writes: the step is W - lr dW
    with the gradients as returned, bit for bit, and the gradients equal those of a run with buffers of their own."""
    torch, B = env["torch"], env["B"]
    rng = np.random.default_rng(L)
    n, D, lr = 700, 24, 0.5
    g = B.Graph(n, 0, np.arange(0, 3 * n + 1, 3, dtype=np.int64), rng.integers(0, n, 3 * n).astype(np.int32), np.full(n, 1 / 3, np.float32), None)
    mk = lambda *s: [torch.randn(*s, device="cuda") / 5 for _ in range(L)]  # noqa: E731
    w, w_self, b = mk(D, D), mk(D, D), mk(D)
    start = [t.clone() for t in w + w_self + b]
    layers = [B.make_layer(B.SAGE_MEAN, D, D, B.ACT_RELU if l < L - 1 else B.ACT_NONE, B.F32, w[l], w_self[l], b[l], B.AGG_FIRST) for l in range(L)]
    x = torch.randn(n, D, device="cuda")
    labels = torch.randint(0, D, (n,), device="cuda", dtype=torch.int32)
    size = B.epoch_workspace_bytes(g, None, layers)
    st = torch.cuda.Stream()

    def run(share):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        zero = lambda *s: [torch.full(s, 7.0, device="cuda") for _ in range(L)]  # noqa: E731
        dw, ds, db = zero(D, D), zero(D, D), zero(D)
        if share == "dw": dw = [dw[0]] * L
        if share == "bias": db = [db[0]] * L
        loss = torch.zeros(1, device="cuda")
        torch.cuda.synchronize()
        eg = B.EpochGraph(g, None, layers, x, D, labels, None, 0.0, None, dw, ds, db, lr, loss, ws, size, st) if recorded else None
        for it in range(3):
            say(f"epoch end L={L} shared={share} recorded={recorded} pass {it}")
            for t, s in zip(w + w_self + b, start): t.copy_(s)
            torch.cuda.synchronize()
            if recorded: eg.launch(st)
            else: loss.fill_(B.epoch(g, None, layers, x, D, labels, None, 0.0, None, dw, ds, db, lr, ws, size, stream=st, want_loss=True)[0])
            torch.cuda.synchronize()
            for t, s, d in zip(w + w_self + b, start, dw + ds + db):
                assert torch.equal(t, s - lr * d)
        assert np.isfinite(float(loss)) and float(loss) > 0
        return dw, ds, db, float(loss)

    own, got = run("none"), run(shared)
    assert got[3] == own[3] and torch.equal(got[0][0], own[0][0]) and torch.equal(got[2][0], own[2][0])
    assert all(torch.equal(p, q) for p, q in zip(got[1], own[1]))
    assert all(float(t.abs().max()) > 0 for t in own[0] + own[1] + own[2])


@pytest.mark.parametrize("recorded", [False, True])
@pytest.mark.parametrize("tie", ["layers", "self", "all", "bias", "overlap"])
def test_sgd_step_adds_every_gradient_of_a_shared_tensor(env, tie, recorded):
    """Layers that share a tensor (tied weights, W_self == W, one bias, a matrix that starts inside another one) get the updates of all
    of them, one after the other: W - lr (dW_0 + dW_1 + ..) in the order of the layers.  Each update of an element rounds its product
    and its difference at most: 2^-23 of the largest magnitude per update, a hundredth of what a lost update would leave out."""
    torch, B = env["torch"], env["B"]
    rng = np.random.default_rng(11)
    n, D, L, lr = 300, 256, 3, 30.0
    rowptr = np.arange(0, 4 * n + 1, 4, dtype=np.int64)
    g = B.Graph(n, 0, rowptr, rng.integers(0, n, 4 * n).astype(np.int32), np.full(n, 0.25, np.float32), None)
    buf = torch.from_numpy((rng.standard_normal((2 * L, D * D)) / 16).astype(np.float32)).cuda()
    bias = torch.from_numpy((rng.standard_normal((L, D)) / 16).astype(np.float32)).cuda()
    w_at = {"layers": [0] * L, "all": [0] * L, "overlap": [0, D * D // 2, D * D]}.get(tie, [l * D * D for l in range(L)])
    s_at = {"self": w_at, "all": w_at}.get(tie, [(L + l) * D * D for l in range(L)])
    b_at = [0] * L if tie in ("bias", "all") else list(range(L))
    flat = buf.view(-1)
    layers = [B.make_layer(B.SAGE_MEAN, D, D, B.ACT_RELU if l < L - 1 else B.ACT_NONE, B.F32, flat[w_at[l]:], flat[s_at[l]:], bias[b_at[l]], B.AGG_FIRST)
              for l in range(L)]
    x = torch.randn(n, D, device="cuda")
    labels = torch.randint(0, D, (n,), device="cuda", dtype=torch.int32)
    mk = lambda *s: [torch.zeros(*s, device="cuda") for _ in range(L)]  # noqa: E731
    dw, ds, db = mk(D, D), mk(D, D), mk(D)
    size = B.epoch_workspace_bytes(g, None, layers)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    st = torch.cuda.Stream()
    start = buf.clone(), bias.clone()
    flat_0, bias_0 = flat.double().cpu().numpy(), bias.double().cpu().numpy()
    torch.cuda.synchronize()
    if recorded:
        eg = B.EpochGraph(g, None, layers, x, D, labels, None, 0.0, None, dw, ds, db, lr, None, ws, size, st)
    for it in range(3):
        say(f"shared tensors {tie} recorded={recorded} step {it}")
        buf.copy_(start[0])
        bias.copy_(start[1])
        torch.cuda.synchronize()
        if recorded:
            eg.launch(st)
        else:
            B.epoch(g, None, layers, x, D, labels, None, 0.0, None, dw, ds, db, lr, ws, size, stream=st, want_loss=False)
        torch.cuda.synchronize()
        want_w, want_b = flat_0.copy(), bias_0.copy()
        least = np.inf
        for l in range(L):
            for at, d in ((w_at[l], dw[l]), (s_at[l], ds[l])):
                step = lr * d.double().cpu().numpy().ravel()
                want_w[at:at + D * D] -= step
                least = min(least, np.abs(step).max())
            step = lr * db[l].double().cpu().numpy()
            want_b[b_at[l]] -= step
            least = min(least, np.abs(step).max())
        bound = 2 * L * 2.0 ** -23 * max(np.abs(flat_0).max(), np.abs(want_w).max(), np.abs(bias_0).max(), np.abs(want_b).max())
        assert least > 100 * bound, "a lost update would not be seen"
        assert np.abs(flat.double().cpu().numpy() - want_w).max() <= bound
        assert np.abs(bias.double().cpu().numpy() - want_b).max() <= bound


@pytest.mark.parametrize("dtype,form,inner,width,n", [("f32", 0, 4096, 4096, 150_001), ("f32", 1, 2048, 2048, 150_001), ("f32", 2, 2048, 2048, 150_001),
                                                      ("f32", 0, 64, 64, 520_007), ("f32", 2, 64, 64, 520_007), ("f32", 1, 1024, 64, 40_001),
                                                      ("bf16", 0, 4096, 4096, 150_001), ("bf16", 0, 64, 64, 520_007), ("bf16", 0, 320, 320, 520_007),
                                                      ("bf16", 0, 640, 64, 120_001)])
def test_epoch_bias_gradient_of_many_equal_rows(env, dtype, form, inner, width, n):
    """The hidden layers' bias gradients are column sums that the weight gradients' products form on the way.  Every row of dZ is the
    same here (self loops, equal rows and labels) and its elements are known: the last weight matrix holds one power of two per row, so
    dZ of the layer below is an element of the loss gradient times that.  A running fp32 sum of n equal terms drifts by up to n 2^-25,
    all in one direction: wide layers have few reduction splits and would add thousands of terms in a row.  Bound: the loss gradient's
    element (exponential, sum, quotient and product, 8 roundings) plus 32 fp32 additions in a row (2^-20) plus two roundings of the
    partial and the whole sum: 2^-19; with bf16 storage the element is rounded to bf16 before, which is repeated here."""
    torch, B = env["torch"], env["B"]
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    code = B.BF16 if dtype == "bf16" else B.F32
    C, dims = 4, [8, inner, width, 4]
    g = B.Graph(n, 0, np.arange(n + 1, dtype=np.int64), np.arange(n, dtype=np.int32), None, None)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(width + n)
    x = (torch.rand(1, 8, generator=gen, device="cuda") + 0.5).to(dt).repeat(n, 1)
    at = torch.arange(width, device="cuda") % C
    power = torch.exp2(-(torch.arange(width, device="cuda") % 3).float())
    w = [(torch.rand(8, inner, generator=gen, device="cuda") / 8).to(dt), (torch.rand(inner, width, generator=gen, device="cuda") * (2.0 / inner)).to(dt),
         torch.zeros(width, C, device="cuda")]
    w[2][torch.arange(width, device="cuda"), at] = power * 2.0 ** (2 - width.bit_length())
    w[2] = w[2].to(dt)
    layers = [B.make_layer(B.GCN, dims[l], dims[l + 1], B.ACT_RELU if l < 2 else B.ACT_NONE, code, w[l], None, None, B.AGG_FIRST, out_f32=int(dtype == "bf16" and l == 2),
                           f32_product=form) for l in range(3)]
    labels = torch.ones(n, device="cuda", dtype=torch.int32)
    logits = torch.zeros(n, C, device="cuda")
    dw = [torch.zeros(dims[l], dims[l + 1], device="cuda") for l in range(3)]
    db = [torch.zeros(d, device="cuda") for d in dims[1:]]
    size = B.epoch_workspace_bytes(g, None, layers)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    say(f"bias gradient of equal rows {dtype} form={form} {inner} x {width}, {n} rows")
    B.epoch(g, None, layers, x, 8, labels, None, 0.0, logits, dw, None, db, 0.0, ws, size)
    torch.cuda.synchronize()
    assert torch.equal(logits, logits[:1].expand(n, C))
    z = logits[0].double()
    dz = (torch.softmax(z, 0) - torch.tensor([0.0, 1.0, 0.0, 0.0], device="cuda", dtype=torch.float64)) / n
    err = ((db[2].double() - n * dz).abs() / (n * dz).abs()).max().item()
    if dtype == "bf16":
        dz = dz.to(torch.bfloat16).double()
    ref = n * dz[at] * w[2][torch.arange(width, device="cuda"), at].double()
    got = db[1].double()
    rel = ((got - ref).abs() / ref.abs()).max().item()
    say(f"   largest relative error: last bias {err:.2e}, hidden bias {rel:.2e}")
    assert err <= 2.0 ** -19 and rel <= 2.0 ** -19
