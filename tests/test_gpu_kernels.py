"""Per-kernel parity of the HIP library against the CPU oracle (needs an MI355X).

fp32 results must agree within 1e-4, bf16 within 2e-2, in the norm-wise metric
max|gpu - ref| / max|ref| and, for the aggregations, also element by element:
|gpu - ref| <= tol (|ref| + rms of the element's own row), so that the rows of hub vertices cannot vouch
for short rows; cache lookup and gather must agree bit for bit.
"""
import numpy as np
import pytest

from paper_2508_13716_amd import synth

pytestmark = pytest.mark.gpu

TOL_F32 = 1e-4
TOL_BF16 = 2e-2


@pytest.fixture(scope="module")
def env(orc):
    import torch
    from paper_2508_13716_amd import binding as B, harness as H
    from tests import oracle_side as O
    assert torch.cuda.is_available()
    B.lib()
    return dict(torch=torch, B=B, H=H, O=O, orc=orc)


def say(msg):
    print(msg, flush=True)


def adversarial_graphs():
    rng = np.random.default_rng(17)
    gs = [synth.hand_partition(9, 6, [(int(rng.integers(0, 9)), int(rng.integers(0, 15))) for _ in range(40)] +
                               [(0, 1), (0, 1)], name="dups+empty"),
          synth.hand_partition(6, 5000, [(0, j) for j in range(6, 5006)] + [(2, 9), (5, 5)], name="one-5000-row"),
          synth.hand_partition(4, 3, [], name="no-edges"),
          synth.hand_partition(1, 0, [(0, 0)], name="single"),
          synth.make_partition("cl-small", 700, 500, 9000, seed=5, max_deg=300),
          synth.make_partition("cl-long", 300, 9000, 40000, seed=6, max_deg=9000, halo_edge_frac=0.9)]
    return gs


def run_spmm(env, part, F, ld, dtype, with_vals, seed, blocked=False, unit_weights=False):
    torch, B, H, O, orc = env["torch"], env["B"], env["H"], env["O"], env["orc"]
    rng = np.random.default_rng(seed)
    r = rng.uniform(0.5, 1.5, part.n_loc).astype(np.float32)
    c = rng.uniform(0.5, 1.5, part.n_cols).astype(np.float32)
    if unit_weights:       # every entry weighs 1 in both directions: the kernels read bare source rows
        r, c = np.ones_like(r), np.ones_like(c)
    v = rng.uniform(-1, 1, part.nnz).astype(np.float32) if with_vals else None
    X = rng.standard_normal((part.n_cols, F)).astype(np.float32)
    dY = rng.standard_normal((part.n_loc, F)).astype(np.float32)
    if dtype == "bf16":
        Xs, dYs = synth.f32_to_bf16_rne(X).reshape(X.shape), synth.f32_to_bf16_rne(dY).reshape(dY.shape)
    else:
        Xs, dYs = X, dY
    g = B.Graph(part.n_loc, part.n_halo, part.rowptr, part.col, r, c, v)
    dt = B.BF16 if dtype == "bf16" else B.F32
    Xd, dYd = H.padded_matrix(Xs, ld), H.padded_matrix(dYs, ld)
    # sentinel-filled outputs: whatever the kernel must not touch stays recognisable
    Yd = torch.full((part.n_loc, ld), 7.0, dtype=Xd.dtype, device="cuda")
    dXd = torch.full((part.n_cols, ld), 7.0, dtype=Xd.dtype, device="cuda")
    ws, wsb = None, 0
    if blocked:       # with scratch the column-blocked kernel runs, or very long rows are cut into pieces
        wsb = B.spmm_workspace_bytes(g, F, dt)
        assert wsb > 0, "graph or width qualifies neither for the column-blocked kernel nor for cut rows"
        ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    B.spmm_fwd(g, Xd, ld, Yd, ld, F, dt, ws=ws, ws_bytes=wsb)
    B.spmm_bwd(g, dYd, ld, dXd, ld, F, dt, ws=ws, ws_bytes=wsb)
    torch.cuda.synchronize()
    og = orc.Graph(part.n_loc, part.n_cols, part.rowptr, part.col, r.astype(np.float64), c.astype(np.float64),
                   None if v is None else v.astype(np.float64))
    Yref = orc.spmm_fwd(og, O.widen(Xs))
    dXref = orc.spmm_bwd(og, O.widen(dYs))
    Y, dX = O.widen(H.dev_to_np(Yd)), O.widen(H.dev_to_np(dXd))
    tol = TOL_BF16 if dtype == "bf16" else TOL_F32
    errs = (O.normwise(Y[:, :F], Yref), O.elementwise(Y[:, :F], Yref, by_row=True),
            O.normwise(dX[:, :F], dXref), O.elementwise(dX[:, :F], dXref, by_row=True))
    say(f"   fwd {errs[0]:.2e} norm-wise, {errs[1]:.2e} element-wise by row; transposed {errs[2]:.2e}, {errs[3]:.2e}")
    assert max(errs) <= tol, (part.name, F, ld, dtype, errs)
    assert (Y[:, F:] == 7.0).all() and (dX[:, F:] == 7.0).all(), "padding columns were written"
    g.close()


@pytest.mark.parametrize("gi", range(6))
def test_spmm_adversarial_graphs_f32(env, gi):
    part = adversarial_graphs()[gi]
    for F, ld in [(1, 1), (7, 7), (8, 8), (41, 44), (64, 64), (100, 100), (130, 132)]:
        say(f"spmm f32 {part.name} F={F} ld={ld}")
        run_spmm(env, part, F, ld, "f32", with_vals=(F % 2 == 1), seed=gi * 100 + F)


@pytest.mark.parametrize("F,ld", [(602, 602), (602, 608), (256, 256), (800, 800), (1000, 1001)])
def test_spmm_wide_rows_f32(env, F, ld):
    part = synth.make_partition("cl-wide", 500, 400, 8000, seed=8, max_deg=2500)
    say(f"spmm f32 wide F={F} ld={ld}")
    run_spmm(env, part, F, ld, "f32", with_vals=False, seed=F)


@pytest.mark.parametrize("F,ld", [(3, 3), (16, 16), (47, 48), (128, 128), (512, 512), (600, 600), (1500, 1504)])
def test_spmm_bf16(env, F, ld):
    for part in adversarial_graphs()[:2] + adversarial_graphs()[4:]:
        say(f"spmm bf16 {part.name} F={F} ld={ld}")
        run_spmm(env, part, F, ld, "bf16", with_vals=False, seed=F)


@pytest.mark.parametrize("shape", ["wide", "tall"])
def test_spmm_column_blocked(env, shape):
    """Dense-degree operators get a column-blocked copy (several source blocks, long (block,row) groups);
    with scratch the blocked kernel + its fixed-order reduction run.  'wide' blocks the forward product,
    'tall' the transposed one; ragged last block, empty groups, partial last slice, edge values."""
    if shape == "wide":
        part = synth.make_partition("blk-wide", 2500, 38000, 330000, seed=21, max_deg=9000, halo_edge_frac=0.9)
    else:
        part = synth.make_partition("blk-tall", 37000, 2000, 2600000, seed=22, max_deg=4000, halo_edge_frac=0.2)
    for F, ld, dtype, vals in [(32, 32, "f32", False), (41, 44, "f32", True), (256, 256, "f32", False),
                               (602, 604, "f32", False), (64, 64, "bf16", False), (200, 200, "bf16", True),
                               (256, 264, "bf16", False)]:
        say(f"spmm blocked {part.name} F={F} ld={ld} {dtype}")
        run_spmm(env, part, F, ld, dtype, vals, seed=F, blocked=True)


@pytest.mark.parametrize("shape", ["wide", "tall"])
def test_spmm_column_blocked_unit_weights(env, shape):
    """The same operators with every weight equal to 1 (no edge values, scales of 1): the blocked kernel then reads
    its entries as 2-byte row numbers inside the source block, exchanges no weights between lanes and adds instead of
    multiplying.  Widths span one partial slice, several slices and a ragged last slice, both storage types."""
    if shape == "wide":
        part = synth.make_partition("blk-wide-1", 2500, 38000, 330000, seed=31, max_deg=9000, halo_edge_frac=0.9)
    else:
        part = synth.make_partition("blk-tall-1", 37000, 2000, 2600000, seed=32, max_deg=4000, halo_edge_frac=0.2)
    for F, ld, dtype in [(32, 32, "f32"), (41, 44, "f32"), (256, 256, "f32"), (602, 604, "f32"), (64, 64, "bf16"),
                         (200, 200, "bf16")]:
        say(f"spmm blocked, unit weights {part.name} F={F} ld={ld} {dtype}")
        run_spmm(env, part, F, ld, dtype, False, seed=F, blocked=True, unit_weights=True)


def test_spmm_rows_cut_into_pieces(env):
    """Rows and columns far longer than one workgroup's share: with scratch they are cut into pieces whose
    partial sums are combined in a fixed order.  One row of 40000 entries, one exactly at the cutting
    threshold plus one, two halo columns referenced by 33000 rows (ragged last piece), the rest short."""
    rng = np.random.default_rng(5)
    n_loc, n_halo = 45000, 50
    n_cols = n_loc + n_halo
    rows = [rng.integers(0, n_cols, 40000), rng.integers(0, n_cols, 16385)]
    for i in range(2, n_loc):
        extra = [n_loc, n_loc + 1] if i < 33002 else []
        rows.append(np.array(list(rng.integers(0, n_cols, 3)) + extra))
    rowptr = np.zeros(n_loc + 1, np.int64)
    np.cumsum([len(r) for r in rows], out=rowptr[1:])
    col = np.concatenate(rows).astype(np.int32)
    part = synth.Partition("cut", n_loc, n_halo, rowptr, col, np.arange(n_halo, dtype=np.int64),
                           np.ones(n_halo, np.int64), np.ones(n_halo, np.int64), False, False)
    for F, ld, dtype, vals in [(32, 32, "f32", False), (41, 44, "f32", True), (256, 256, "bf16", False),
                               (100, 104, "bf16", True), (7, 7, "f32", False)]:
        say(f"spmm cut rows F={F} ld={ld} {dtype}")
        run_spmm(env, part, F, ld, dtype, vals, seed=F, blocked=True)


def test_spmm_exact_on_small_integers(env):
    """Integer features, unit scales: every partial sum is exactly representable, so fp32 and bf16
    results must equal the oracle exactly."""
    torch, B, H, O, orc = env["torch"], env["B"], env["H"], env["O"], env["orc"]
    part = synth.make_partition("ints", 400, 300, 3000, seed=9, max_deg=100)
    rng = np.random.default_rng(1)
    X = rng.integers(-2, 3, (part.n_cols, 24)).astype(np.float32)
    g = B.Graph(part.n_loc, part.n_halo, part.rowptr, part.col)
    og = orc.Graph(part.n_loc, part.n_cols, part.rowptr, part.col, np.ones(part.n_loc), np.ones(part.n_cols))
    ref = orc.spmm_fwd(og, X.astype(np.float64))
    assert np.abs(ref).max() <= 256
    for dt, Xs in ((B.F32, X), (B.BF16, synth.f32_to_bf16_rne(X).reshape(X.shape))):
        Xd = H.np_to_dev(Xs)
        Yd = torch.zeros((part.n_loc, 24), dtype=Xd.dtype, device="cuda")
        B.spmm_fwd(g, Xd, 24, Yd, 24, 24, dt)
        torch.cuda.synchronize()
        assert np.array_equal(O.widen(H.dev_to_np(Yd)), ref)
    g.close()


@pytest.mark.parametrize("scratch", [True, False])
@pytest.mark.parametrize("fill", [0, 45000])
def test_spmm_row_length_classes_exact(env, fill, scratch):
    """Row lengths on both sides of every limit of the work list: eight entries per trip of a lane group, 16 .. 128 entries
    for a group alone, pieces of 64 entries (small graph: its longest row ends after the launch but for the narrowest rows,
    which take one launch) or 512 (more than 2 M entries), cut from twice that length on.
    One width per lane-group size and one whose rows are not vectors; small integers, so every order of summation gives the
    same float and a bf16 result is that float rounded once: equality."""
    torch, B, H, O, orc = env["torch"], env["B"], env["H"], env["O"], env["orc"]
    rng = np.random.default_rng(3 + fill)
    lens = [0, 1, 2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 193, 255, 256, 257, 511, 513, 1023, 1024,
            1025, 1537, 5000] + [48] * fill
    n_loc, n_halo = len(lens), 700
    rowptr = np.zeros(n_loc + 1, np.int64)
    np.cumsum(lens, out=rowptr[1:])
    col = rng.integers(0, n_loc + n_halo, rowptr[-1]).astype(np.int32)
    val = rng.integers(-1, 2, rowptr[-1]).astype(np.float32)
    for F, ld, vals in [(5, 8, False), (30, 32, True), (60, 64, False), (41, 41, True)] + ([] if fill else [
            (100, 104, True), (250, 256, False), (400, 400, True), (1600, 1600, False)]):
        for dt in (B.F32, B.BF16):
            say(f"spmm row classes F={F} ld={ld} dtype={dt} fill={fill} scratch={scratch}")
            X = rng.integers(-2, 3, (n_loc + n_halo, F)).astype(np.float32)
            g = B.Graph(n_loc, n_halo, rowptr, col, None, None, val if vals else None)
            og = orc.Graph(n_loc, n_loc + n_halo, rowptr, col, np.ones(n_loc), np.ones(n_loc + n_halo),
                           val.astype(np.float64) if vals else None)
            Xd = H.padded_matrix(X if dt == B.F32 else synth.f32_to_bf16_rne(X).reshape(X.shape), ld)
            wsb = B.spmm_workspace_bytes(g, F, dt) if scratch else 0
            ws = torch.empty(wsb, dtype=torch.uint8, device="cuda") if wsb else None
            assert wsb > 0 or not scratch
            for back in (False, True):
                n_out = n_loc + n_halo if back else n_loc
                ref = (orc.spmm_bwd(og, X[:n_loc].astype(np.float64)) if back else orc.spmm_fwd(og, X.astype(np.float64)))
                Yd = torch.full((n_out, ld), 7.0, dtype=Xd.dtype, device="cuda")
                (B.spmm_bwd if back else B.spmm_fwd)(g, Xd, ld, Yd, ld, F, dt, ws=ws, ws_bytes=wsb)
                torch.cuda.synchronize()
                Y = O.widen(H.dev_to_np(Yd))
                want = ref if dt == B.F32 else synth.bf16_to_f32(synth.f32_to_bf16_rne(ref.astype(np.float32))).reshape(ref.shape)
                assert np.array_equal(Y[:, :F], want), (F, dt, back)
                assert (Y[:, F:] == 7.0).all(), "padding columns were written"
            g.close()


@pytest.mark.parametrize("n40,n70", [(179, 60), (180, 60), (10, 240), (10, 241)])
def test_spmm_middling_rows_of_a_small_graph_exact(env, n40, n70):
    """Rows below the cut that a small graph's one launch gives workgroups of their own, up to 256 with the cut rows (16 here): both
    classes at the limit, the lower one a row beyond it, only the upper one, neither.  Small integers: equality."""
    torch, B, H, O, orc = env["torch"], env["B"], env["H"], env["O"], env["orc"]
    rng = np.random.default_rng(n40 + n70)
    lens = rng.permutation([130] * 15 + [700] + [70] * n70 + [40] * n40 + [33, 31, 5, 0] + [9] * 300)
    n_loc, n_halo = len(lens), 100
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = rng.integers(0, n_loc + n_halo, rowptr[-1]).astype(np.int32)
    val = rng.integers(-1, 2, rowptr[-1]).astype(np.float32)
    for F, ld, vals in [(5, 8, False), (41, 41, True), (64, 64, False), (128, 128, True), (250, 256, False), (700, 700, True)]:
        X = rng.integers(-2, 3, (n_loc + n_halo, F)).astype(np.float32)
        og = orc.Graph(n_loc, n_loc + n_halo, rowptr, col, np.ones(n_loc), np.ones(n_loc + n_halo), val.astype(np.float64) if vals else None)
        ref = orc.spmm_fwd(og, X.astype(np.float64))
        for dt in (B.F32, B.BF16):
            say(f"spmm middling rows n40={n40} n70={n70} F={F} dtype={dt}")
            g = B.Graph(n_loc, n_halo, rowptr, col, None, None, val if vals else None)
            Xd = H.padded_matrix(X if dt == B.F32 else synth.f32_to_bf16_rne(X).reshape(X.shape), ld)
            wsb = B.spmm_workspace_bytes(g, F, dt)
            for ws in (torch.empty(wsb, dtype=torch.uint8, device="cuda"), None):
                Yd = torch.full((n_loc, ld), 7.0, dtype=Xd.dtype, device="cuda")
                B.spmm_fwd(g, Xd, ld, Yd, ld, F, dt, ws=ws, ws_bytes=wsb if ws is not None else 0)
                torch.cuda.synchronize()
                Y = O.widen(H.dev_to_np(Yd))
                want = ref if dt == B.F32 else synth.bf16_to_f32(synth.f32_to_bf16_rne(ref.astype(np.float32))).reshape(ref.shape)
                assert np.array_equal(Y[:, :F], want), (F, dt)
                assert (Y[:, F:] == 7.0).all()
            g.close()


@pytest.mark.parametrize("scratch", [True, False])
@pytest.mark.parametrize("hub,others", [(500_000, 350_000), (60_000, 90_000), (2_100, 6_000)])
def test_spmm_hub_of_a_small_graph_exact(env, hub, others, scratch):
    """Graphs below 2^20 entries whose longest row, and in the transposed product whose longest column, holds a large part of them: with
    scratch it is cut over many workgroups (pieces of 64, 128 and 256 entries) unless it ends with the launch anyway (the narrow rows
    here), without it one workgroup walks it.  Small integers, sums below 2^24: equality, and a bf16 result is the sum rounded once."""
    torch, B, H, O, orc = env["torch"], env["B"], env["H"], env["O"], env["orc"]
    rng = np.random.default_rng(hub)
    n_loc, n_halo = others // 6, 300
    n_cols = n_loc + n_halo
    rowptr = np.concatenate([[0, 2, 2 + hub], 2 + hub + 3 * np.arange(1, n_loc - 1)]).astype(np.int64)
    col = rng.integers(0, n_cols, rowptr[-1]).astype(np.int32)
    col[2 + hub::3] = n_loc + 7                   # the first entry of every short row
    val = rng.integers(-1, 2, rowptr[-1]).astype(np.float32)
    assert rowptr[-1] < 2 ** 20
    for F, ld, vals in [(5, 8, True), (41, 44, False), (64, 64, True), (260, 264, False)] + ([(700, 704, False), (41, 41, True)] if hub < 10_000 else []):
        for dt in (B.F32, B.BF16):
            say(f"spmm hub of {hub} entries, {rowptr[-1]} in all, F={F} ld={ld} dtype={dt} scratch={scratch}")
            X = rng.integers(-2, 3, (n_cols, F)).astype(np.float32)
            g = B.Graph(n_loc, n_halo, rowptr, col, None, None, val if vals else None)
            og = orc.Graph(n_loc, n_cols, rowptr, col, np.ones(n_loc), np.ones(n_cols), val.astype(np.float64) if vals else None)
            Xd = H.padded_matrix(X if dt == B.F32 else synth.f32_to_bf16_rne(X).reshape(X.shape), ld)
            wsb = B.spmm_workspace_bytes(g, F, dt) if scratch else 0
            ws = torch.empty(wsb, dtype=torch.uint8, device="cuda") if wsb else None
            assert wsb > 0 or not scratch
            for back in (False, True):
                ref = orc.spmm_bwd(og, X[:n_loc].astype(np.float64)) if back else orc.spmm_fwd(og, X.astype(np.float64))
                Yd = torch.full((n_cols if back else n_loc, ld), 7.0, dtype=Xd.dtype, device="cuda")
                (B.spmm_bwd if back else B.spmm_fwd)(g, Xd, ld, Yd, ld, F, dt, ws=ws, ws_bytes=wsb)
                torch.cuda.synchronize()
                Y = O.widen(H.dev_to_np(Yd))
                want = ref if dt == B.F32 else synth.bf16_to_f32(synth.f32_to_bf16_rne(ref.astype(np.float32))).reshape(ref.shape)
                assert np.array_equal(Y[:, :F], want), (F, dt, back)
                assert (Y[:, F:] == 7.0).all(), "padding columns were written"
            g.close()


def test_spmm_on_config1_graph(env):
    cfg = synth.CONFIGS["C1"]
    part = synth.partition_for(cfg)
    say("spmm C1")
    run_spmm(env, part, 128, 128, "f32", False, 1)
    run_spmm(env, part, 64, 64, "f32", False, 2)


def test_graph_create_rejects_malformed_input(env):
    B = env["B"]
    with pytest.raises(B.CapgnnError):
        B.Graph(2, 0, np.array([0, 1, 3]), np.array([0, 5, 1], np.int32))       # column out of range
    with pytest.raises(B.CapgnnError):
        B.Graph(2, 0, np.array([0, 2, 1]), np.array([0, 1], np.int32))          # rowptr decreases
    with pytest.raises(B.CapgnnError):
        B.Graph(2, 0, np.array([1, 2, 3]), np.array([0, 1, 1], np.int32))       # rowptr[0] != 0
    with pytest.raises(B.CapgnnError):                                          # claims symmetry, is not
        B.Graph(2, 0, np.array([0, 1, 1]), np.array([1], np.int32), flags=B.GRAPH_SYMMETRIC)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,cap", [(1, 1), (3, 0), (67, 30), (8191, 4000), (8193, 8193), (70_001, 35_003)])
def test_full_gather_row_counts_and_widths_bit_exact(env, n, cap, dtype):
    """Both launch forms of the full-batch gather (four rows per lane group where there are many rows of more than one load per lane,
    else one: the widest rows here are more than one load in either type), with one and two tiers, at widths
    whose rows are shorter than a vector, end in the middle of one, or are wider than a lane group; destinations that are and
    are not 16-byte aligned.  Bit copies: no tolerance."""
    torch, B = env["torch"], env["B"]
    dims = [1, 7, 50, 128, 301, 701]
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rng = np.random.default_rng(n)
    c = B.Cache(rng.permutation(n).astype(np.int64) + 17, rng.integers(1, 100, n).astype(np.int64), cap, dims, B.BF16 if dtype == "bf16" else B.F32)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    ids = torch.arange(n, device="cuda")
    stage = torch.empty(max(c.staging_bytes, 256), dtype=torch.uint8, device="cuda")
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    for l, d in enumerate(dims):
        rows = torch.randn(n, d, generator=gen, device="cuda").to(dt)
        B.cache_update(c, l, ids, n, rows, d, 0)
        for ld in (d, (d + 15) // 16 * 16 + 16):
            for two_streams in (False, True):
                say(f"full gather n={n} cap={cap} width={d} ld={ld} two_streams={two_streams}")
                out = torch.full((n + 1, ld), -3.0, dtype=dt, device="cuda")
                torch.cuda.synchronize()
                if two_streams:
                    B.halo_gather(c, l, None, n, out, ld, stream=main, side_stream=side, staging=stage)
                else:
                    B.halo_gather(c, l, None, n, out, ld, stream=main)
                torch.cuda.synchronize()
                assert torch.equal(out[:n, :d], rows)
                assert (out[n] == -3).all() and (out[:, d:] == -3).all()      # nothing beyond the rows is written


# ----------------------------------------------------------------------------- cache
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cap_frac", [0.0, 0.37, 1.0])
def test_cache_placement_lookup_gather_bit_exact(env, dtype, cap_frac):
    torch, B, H, O, orc = env["torch"], env["B"], env["H"], env["O"], env["orc"]
    part = synth.make_partition("cache", 300, 5000, 30000, seed=21, max_deg=200)
    n = part.n_halo
    cap = int(cap_frac * n)
    dims = [602, 47, 8]
    dt = B.BF16 if dtype == "bf16" else B.F32
    tables = [synth.make_features(n, d, seed=3, stream=30 + i, dtype=dtype) for i, d in enumerate(dims)]
    say(f"cache dtype={dtype} cap={cap}/{n}")
    c = B.Cache(part.halo_gid, part.halo_prio, cap, dims, dt, B.MAP_HASH)
    for l in range(3):
        c.fill(l, tables[l])
    # placement: tier membership equals the oracle's
    _, tier_ref = orc.placement(part.halo_gid, part.halo_prio, cap)
    tier, slot = c.query(np.arange(n))
    assert np.array_equal(tier, tier_ref)
    assert sorted(slot[tier == 0]) == list(range(cap)) and sorted(slot[tier == 1]) == list(range(n - cap))
    tier_g, slot_g = c.query(part.halo_gid, by_gid=True)
    assert np.array_equal(tier_g, tier) and np.array_equal(slot_g, slot)
    # device lookup, including absent keys
    rng = np.random.default_rng(4)
    absent = rng.integers(1 << 41, 1 << 42, 1000).astype(np.int64)
    ids = np.concatenate([part.halo_gid[rng.integers(0, n, 3000)], absent])
    ids_d = torch.from_numpy(ids).cuda()
    t_d = torch.empty(len(ids), dtype=torch.int8, device="cuda")
    s_d = torch.empty(len(ids), dtype=torch.int64, device="cuda")
    c.lookup(ids_d, t_d, s_d, by_gid=True)
    torch.cuda.synchronize()
    t_h, s_h = c.query(ids, by_gid=True, check=False)
    assert np.array_equal(t_d.cpu().numpy(), t_h) and np.array_equal(s_d.cpu().numpy(), s_h)
    assert (t_h[-1000:] == -1).all() and (t_h[:3000] >= 0).all()

    side = torch.cuda.Stream()
    main = torch.cuda.Stream()
    stg = torch.empty(max(c.staging_bytes, 256), dtype=torch.uint8, device="cuda")
    for l, d in enumerate(dims):
        per16 = 16 // (2 if dtype == "bf16" else 4)
        for ld in (d, synth.pad_to(d, per16)):
            ref_all, _ = orc.gather(tables[l], np.arange(n))
            for staging, sd in ((None, None), (None, side), (stg, side), (stg, None)):
                out = torch.full((n, ld), 3.0, dtype=H.np_to_dev(tables[l][:1]).dtype, device="cuda")
                rc, st = B.halo_gather(c, l, None, n, out, ld, stream=main, side_stream=sd, staging=staging, want_stats=True)
                got = H.dev_to_np(out)
                assert got[:, :d].tobytes() == ref_all.tobytes(), (l, ld, staging is not None, sd is not None)
                assert (O.widen(got[:, d:]) == 3.0).all()
                assert (st.hits, st.misses, st.absent) == (cap, n - cap, 0)
            # request list: duplicates, arbitrary order, by halo-local index and by global id, absent ids
            req = rng.integers(0, n, 7001).astype(np.int64)
            ref, _ = orc.gather(tables[l], req)
            for by_gid, sd in ((False, None), (True, side)):
                ids_h = part.halo_gid[req] if by_gid else req
                out = torch.full((len(req), ld), 3.0, dtype=H.np_to_dev(tables[l][:1]).dtype, device="cuda")
                rc, st = B.halo_gather(c, l, torch.from_numpy(ids_h).cuda(), len(req), out, ld, by_gid=by_gid,
                                       stream=main, side_stream=sd, want_stats=True)
                assert H.dev_to_np(out)[:, :d].tobytes() == ref.tobytes()
                assert st.hits == int((tier[req] == 0).sum()) and st.misses == int((tier[req] == 1).sum())
            bad = req.copy()
            bad[10], bad[500] = -5, n + 3
            ref, n_abs = orc.gather(tables[l], bad)
            out = torch.full((len(req), ld), 3.0, dtype=H.np_to_dev(tables[l][:1]).dtype, device="cuda")
            rc, st = B.halo_gather(c, l, torch.from_numpy(bad).cuda(), len(bad), out, ld, stream=main,
                                   want_stats=True, check=False)
            assert rc == B.ENOTFOUND and st.absent == n_abs == 2
            assert H.dev_to_np(out)[:, :d].tobytes() == ref.tobytes()
    c.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cap_frac", [0.0, 0.37, 1.0])
def test_cache_update_and_stale_list_bit_exact(env, dtype, cap_frac):
    """Vertex update (both tiers, repeated and absent ids, by index and by global id) and the
    bounded-staleness list against the oracle: every cached byte and every stamp afterwards."""
    torch, B, H, O, orc = env["torch"], env["B"], env["H"], env["O"], env["orc"]
    part = synth.make_partition("cache-upd", 300, 5000, 30000, seed=23, max_deg=200)
    n = part.n_halo
    cap = int(cap_frac * n)
    dims = [70, 256]
    dt = B.BF16 if dtype == "bf16" else B.F32
    tables = [synth.make_features(n, d, seed=5, stream=40 + i, dtype=dtype) for i, d in enumerate(dims)]
    stamps = [np.zeros(n, np.int64) for _ in dims]
    c = B.Cache(part.halo_gid, part.halo_prio, cap, dims, dt, B.MAP_HASH)
    for l in range(len(dims)):
        c.fill(l, tables[l])
    tier, _ = c.query(np.arange(n))
    rng = np.random.default_rng(6)
    main = torch.cuda.Stream()
    ids_out = torch.empty(n, dtype=torch.int64, device="cuda")
    for epoch in range(1, 6):
        for l, d in enumerate(dims):
            per16 = 16 // (2 if dtype == "bf16" else 4)
            ld = d if epoch % 2 else synth.pad_to(d, per16) + per16
            m = int(rng.integers(1, 3000))
            ids = rng.integers(-2, n + 2, m).astype(np.int64)                      # repeats and absent ids
            by_gid = bool(epoch % 2 == 0)
            ids_call = np.where((ids >= 0) & (ids < n), part.halo_gid[np.clip(ids, 0, n - 1)], (1 << 45) + ids) if by_gid else ids
            rows = synth.make_features(m, d, seed=100 + epoch, stream=50 + l, dtype=dtype)
            say(f"cache update dtype={dtype} cap={cap}/{n} epoch={epoch} layer={l} m={m} ld={ld} by_gid={by_gid}")
            rows_d = H.padded_matrix(rows, ld)
            torch.cuda.synchronize()
            st = B.cache_update(c, l, torch.from_numpy(ids_call).cuda(), m, rows_d, ld, epoch, by_gid=by_gid, stream=main,
                                want_stats=True)
            n_abs = orc.cache_update(tables[l], stamps[l], ids, rows, epoch)
            last = np.full(n, -1, np.int64)
            ok = (ids >= 0) & (ids < n)
            last[ids[ok]] = np.nonzero(ok)[0]                                      # one write per distinct vertex
            touched = np.nonzero(last >= 0)[0]
            assert st.absent == n_abs
            assert st.hits == int((tier[touched] == 0).sum()) and st.misses == int((tier[touched] == 1).sum())
            out = torch.full((n, ld), 3.0, dtype=rows_d.dtype, device="cuda")
            torch.cuda.synchronize()
            B.halo_gather(c, l, None, n, out, ld, stream=main)
            torch.cuda.synchronize()
            assert H.dev_to_np(out)[:, :d].tobytes() == tables[l].tobytes()
            for max_age in (0, 2):
                cnt, oldest = B.cache_stale(c, l, epoch, max_age, ids_out, stream=main)
                ref_ids, ref_old = orc.stale_ids(stamps[l], epoch, max_age)
                assert cnt == len(ref_ids) and oldest == ref_old
                assert np.array_equal(ids_out[:cnt].cpu().numpy(), ref_ids)
    # a refill starts the layer's history again
    c.fill(0, tables[0])
    cnt, oldest = B.cache_stale(c, 0, 5, 0, ids_out, stream=main)
    assert cnt == n and oldest == 0
    c.close()


def test_cache_edge_cases(env):
    torch, B = env["torch"], env["B"]
    with pytest.raises(B.CapgnnError):
        B.Cache(np.array([5, 5], np.int64), np.array([1, 2], np.int64), 1, [4], B.F32)     # duplicate gid
    c = B.Cache(np.zeros(0, np.int64), np.zeros(0, np.int64), 10, [4], B.F32)                # empty halo
    out = torch.zeros((1, 4), device="cuda")
    assert B.halo_gather(c, 0, None, 0, out, 4) == B.OK
    with pytest.raises(B.CapgnnError):
        B.halo_gather(c, 1, None, 0, out, 4)                                                 # no such layer
    c.close()


def test_zipf_request_stream_hit_rate(env):
    """Requests drawn Zipf(1.1) over halo vertices ranked by priority, top 10 % on the GPU:
    the measured hit fraction equals H_{k,s}/H_{N,s} up to sampling noise."""
    torch, B = env["torch"], env["B"]
    N, k, s = 200_000, 20_000, 1.1
    p = np.arange(1, N + 1, dtype=np.float64) ** -s
    p /= p.sum()
    rng = np.random.default_rng(5)
    gid = rng.permutation(N).astype(np.int64) * 3 + 11
    prio = (1e12 * p).astype(np.int64)
    c = B.Cache(gid, prio, k, [16], B.F32, B.MAP_HASH)
    c.fill(0, np.zeros((N, 16), np.float32))
    req = rng.choice(N, size=1_000_000, p=p)
    out = torch.empty((len(req), 16), device="cuda")
    rc, st = B.halo_gather(c, 0, torch.from_numpy(gid[req]).cuda(), len(req), out, 16, by_gid=True, want_stats=True)
    expect = float(np.sum(np.arange(1, k + 1, dtype=np.float64) ** -s) / np.sum(np.arange(1, N + 1, dtype=np.float64) ** -s))
    assert abs(st.hits / len(req) - expect) < 3e-3
    c.close()


# ----------------------------------------------------------------------------- dense products
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_gemm_vs_oracle(env, dtype, ta, tb):
    torch, B, H, O, orc = env["torch"], env["B"], env["H"], env["O"], env["orc"]
    rng = np.random.default_rng(ta * 2 + tb)
    dt = B.BF16 if dtype == "bf16" else B.F32
    tol = TOL_BF16 if dtype == "bf16" else TOL_F32
    for (M, N, K) in [(1, 1, 1), (130, 41, 602), (257, 256, 100), (1000, 47, 256), (64, 200, 33), (300, 8, 5000)]:
        say(f"gemm {dtype} ta={ta} tb={tb} M={M} N={N} K={K}")
        A = rng.standard_normal((K, M) if ta else (M, K)).astype(np.float32)
        Bm = rng.standard_normal((N, K) if tb else (K, N)).astype(np.float32)
        bias = rng.standard_normal(N).astype(np.float32)
        if dtype == "bf16":
            A, Bm = synth.f32_to_bf16_rne(A).reshape(A.shape), synth.f32_to_bf16_rne(Bm).reshape(Bm.shape)
        ref = orc.matmul(O.widen(A), O.widen(Bm), ta=bool(ta), tb=bool(tb))
        for pad in (0, 3):
            lda, ldb, ldc = A.shape[1] + pad, Bm.shape[1] + pad, N + pad
            Ad, Bd = H.padded_matrix(A, lda), H.padded_matrix(Bm, ldb)
            Ad[:, A.shape[1]:] = float("nan")            # whatever the padding holds must not reach the result
            Bd[:, Bm.shape[1]:] = float("nan")
            wsb = B.gemm_workspace_bytes(ta, M, N, K)
            ws = torch.empty(max(wsb, 256), dtype=torch.uint8, device="cuda")
            Cd = torch.full((M, ldc), 2.0, dtype=torch.float32, device="cuda")
            B.gemm(ta, tb, M, N, K, Ad, lda, Bd, ldb, Cd, ldc, dt, out_f32=1, ws=ws, ws_bytes=wsb)
            torch.cuda.synchronize()
            got = Cd.cpu().numpy()
            assert O.normwise(got[:, :N], ref) <= tol
            assert (got[:, N:] == 2.0).all()
            # epilogue: accumulate + bias + relu, output in the storage dtype
            Cd2 = torch.full((M, ldc), 0.5, dtype=Ad.dtype, device="cuda")
            B.gemm(ta, tb, M, N, K, Ad, lda, Bd, ldb, Cd2, ldc, dt, accumulate=1, bias=H.np_to_dev(bias), relu=1,
                   ws=ws, ws_bytes=wsb)
            torch.cuda.synchronize()
            ref2 = np.maximum(ref + 0.5 + bias[None, :], 0.0)
            assert O.normwise(O.widen(H.dev_to_np(Cd2))[:, :N], ref2) <= tol


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_gemm_bf16_matrix_core_path(env, ta, tb):
    """bf16 operands with 16-byte aligned rows take the bf16 MFMA kernel (weights of plain products are
    repacked, so their pitch may be anything).  Small-integer operands make every product and partial sum
    exactly representable: the result must equal the oracle exactly, which pins the operand lane layout;
    random operands are compared within the bf16 tolerance.  Sizes span several tiles and ragged tails."""
    torch, B, H, O, orc = env["torch"], env["B"], env["H"], env["O"], env["orc"]
    rng = np.random.default_rng(10 + ta * 2 + tb)
    for (M, N, K) in [(333, 47, 256), (130, 256, 40), (257, 130, 1000), (64, 64, 32), (500, 41, 4100)]:
        for ints in (True, False):
            say(f"gemm bf16 mfma ta={ta} tb={tb} M={M} N={N} K={K} ints={ints}")
            shapeA, shapeB = ((K, M) if ta else (M, K)), ((N, K) if tb else (K, N))
            if ints:
                A = rng.integers(-2, 3, shapeA).astype(np.float32)
                Bm = rng.integers(-2, 3, shapeB).astype(np.float32)
            else:
                A = rng.standard_normal(shapeA).astype(np.float32)
                Bm = rng.standard_normal(shapeB).astype(np.float32)
            A, Bm = synth.f32_to_bf16_rne(A).reshape(A.shape), synth.f32_to_bf16_rne(Bm).reshape(Bm.shape)
            ref = orc.matmul(O.widen(A), O.widen(Bm), ta=bool(ta), tb=bool(tb))
            lda = synth.pad_to(A.shape[1], 8)
            ldb = synth.pad_to(Bm.shape[1], 8) if ta else Bm.shape[1] + 1     # a weight's pitch is free
            ldc = N + 3
            Ad, Bd = H.padded_matrix(A, lda), H.padded_matrix(Bm, ldb)
            Ad[:, A.shape[1]:] = float("nan")            # a ragged last column group is read up to the pitch: the padding
            Bd[:, Bm.shape[1]:] = float("nan")            # must end up nowhere in the result
            wsb = B.gemm_workspace_bytes(ta, M, N, K)
            ws = torch.empty(max(wsb, 256), dtype=torch.uint8, device="cuda")
            Cd = torch.full((M, ldc), 2.0, dtype=torch.float32, device="cuda")
            B.gemm(ta, tb, M, N, K, Ad, lda, Bd, ldb, Cd, ldc, B.BF16, out_f32=1, ws=ws, ws_bytes=wsb)
            torch.cuda.synchronize()
            got = Cd.cpu().numpy()
            if ints:
                assert np.array_equal(got[:, :N].astype(np.float64), ref)
            else:
                assert O.normwise(got[:, :N], ref) <= TOL_BF16
            assert (got[:, N:] == 2.0).all()


@pytest.mark.parametrize("M,N,K", [(16, 32, 16383), (16, 32, 16384), (1, 1, 16391), (33, 5, 20001), (256, 31, 5000), (289, 31, 5000), (300, 7, 2049),
                                   (256, 32, 32768), (257, 32, 32768), (602, 3, 14001)])
def test_gemm_bf16_reductions_of_at_most_32_columns_exact(env, M, N, K):
    """Weight gradients on both sides of each line between the forms for one and for two waves per SIMD: the length of the chains, workgroups
    and compute units, the size of X; alone and added to what C holds.  Small integers: every sum is an integer below 2^24
    (9 * 32768 + 2), so each form gives it exactly, and gives the same on a second call."""
    torch, B, H = env["torch"], env["B"], env["H"]
    rng = np.random.default_rng(M + N + K)
    A = rng.integers(-3, 4, (K, M)).astype(np.float32)
    G = rng.integers(-3, 4, (K, N)).astype(np.float32)
    ref = A.T.astype(np.float64) @ G.astype(np.float64)
    st = lambda x: synth.f32_to_bf16_rne(x).reshape(x.shape)
    lda, ldg, ldc = synth.pad_to(M, 8), synth.pad_to(N, 8), N + 3
    Ad, Gd = H.padded_matrix(st(A), lda), H.padded_matrix(st(G), ldg)
    Ad[:, M:] = float("nan")
    Gd[:, N:] = float("nan")
    wsb = B.gemm_workspace_bytes(1, M, N, K)
    ws = torch.empty(max(wsb, 256), dtype=torch.uint8, device="cuda")
    for acc in (0, 1, 0):
        Cd = torch.full((M, ldc), 2.0, dtype=torch.float32, device="cuda")
        say(f"gemm bf16 reduction {M}x{N}x{K} accumulate={acc}")
        B.gemm(1, 0, M, N, K, Ad, lda, Gd, ldg, Cd, ldc, B.BF16, out_f32=1, accumulate=acc, ws=ws, ws_bytes=wsb)
        torch.cuda.synchronize()
        got = Cd.cpu().numpy()
        assert np.array_equal(got[:, :N].astype(np.float64), ref + 2.0 * acc)
        assert (got[:, N:] == 2.0).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_gemm_size_classes_exact(env, dtype, ta, tb):
    """Both sides of the limits between the product kernels: single elements, ragged 32- and 64-wide tiles, K around a unit, a
    batch and 128, 512 and 513 tiles of 32 rows, 768 and 769 tiles of 64 rows, vertex reductions with one and with many
    splits; rows that are and are not 16-byte aligned.  Small integers: every product and sum is an integer below 2^24
    (K * 9 at most), so each form of the product gives it exactly."""
    torch, B, H, O = env["torch"], env["B"], env["H"], env["O"]
    rng = np.random.default_rng(70 + 2 * ta + tb)
    sizes = [(1, 1, 1), (31, 33, 7), (32, 32, 8), (33, 64, 9), (65, 65, 31), (64, 63, 33), (97, 130, 127), (96, 128, 128), (40, 40, 129),
             (70, 256, 300)]
    sizes += [(130, 121, 2999), (64, 47, 5003), (8, 7, 20000), (257, 200, 1025), (602, 41, 6001), (602, 200, 3500), (320, 16, 5000)] if ta else [
        (16384, 64, 20), (16385, 64, 20), (49152, 64, 36), (49153, 64, 36), (3000, 300, 100)]
    for M, N, K in sizes:
        A = rng.integers(-3, 4, (K, M) if ta else (M, K)).astype(np.float32)
        Bm = rng.integers(-3, 4, (N, K) if tb else (K, N)).astype(np.float32)
        ref = (A.T if ta else A).astype(np.float64) @ (Bm.T if tb else Bm).astype(np.float64)
        st = (lambda x: synth.f32_to_bf16_rne(x).reshape(x.shape)) if dtype == "bf16" else (lambda x: x)
        dt = B.BF16 if dtype == "bf16" else B.F32
        for mult, forms in ((8, (0, 1, 2)), (1, (0,))):           # row pitches: whole vectors, or the bare width plus one
            lda = synth.pad_to(A.shape[1], mult) + (mult == 1)
            ldb = synth.pad_to(Bm.shape[1], mult) + (mult == 1)
            ldc = N + 3
            Ad, Bd = H.padded_matrix(st(A), lda), H.padded_matrix(st(Bm), ldb)
            Ad[:, A.shape[1]:] = float("nan")                     # what the padding holds never reaches C
            Bd[:, Bm.shape[1]:] = float("nan")
            for form in forms if dtype == "f32" else (0,):
                wsb = B.gemm_workspace_bytes(ta, M, N, K)
                ws = torch.empty(max(wsb, 256), dtype=torch.uint8, device="cuda")
                Cd = torch.full((M, ldc), 2.0, dtype=torch.float32, device="cuda")
                say(f"gemm classes {dtype} ta={ta} tb={tb} {M}x{N}x{K} lda={lda} form={form}")
                B.gemm(ta, tb, M, N, K, Ad, lda, Bd, ldb, Cd, ldc, dt, out_f32=1, ws=ws, ws_bytes=wsb, f32_product=form)
                torch.cuda.synchronize()
                got = Cd.cpu().numpy()
                assert np.array_equal(got[:, :N].astype(np.float64), ref), (M, N, K, form)
                assert (got[:, N:] == 2.0).all(), "padding columns were written"


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("tb", [0, 1])
def test_gemm_vertex_reduction_with_little_workspace(env, dtype, tb):
    """X^T G splits its reduction as far as the workspace goes: at most 31 steps of 16 need none, longer ones as many splits as have 16
    steps each; with no room at all those are CAPGNN_ENOMEM, C untouched.  Small integers: exact with any number of splits."""
    torch, B, H = env["torch"], env["B"], env["H"]
    rng = np.random.default_rng(tb)
    for M, N, K, form in [(64, 64, 256, 0), (33, 70, 300, 0), (100, 256, 511, 0), (8, 5, 511, 2), (64, 64, 20000, 0), (130, 121, 6000, 1), (64, 200, 2999, 2)]:
        A, Bm = rng.integers(-3, 4, (K, M)).astype(np.float32), rng.integers(-3, 4, (N, K) if tb else (K, N)).astype(np.float32)
        ref = A.T.astype(np.float64) @ (Bm.T if tb else Bm).astype(np.float64)
        bf = dtype == "bf16"
        st = (lambda x: synth.f32_to_bf16_rne(x).reshape(x.shape)) if bf else (lambda x: x)
        lda, ldb = synth.pad_to(M, 8) + 1, synth.pad_to(Bm.shape[1], 8) + 1         # unaligned bf16 rows: steps of 16
        Ad, Bd = H.padded_matrix(st(A), lda), H.padded_matrix(st(Bm), ldb)
        step = 32 if not bf and not tb and form == 2 else 16
        splits = min(1536 // (-(-M // 128) * -(-N // (64 if N <= 64 else 128))), K // (16 * step))
        need = splits * M * N * 4 if splits > 1 else 0
        for room in ([need, 0] if need else [0]):
            say(f"gemm X^T G {dtype} tb={tb} {M}x{N}x{K} form={form}: {room} bytes of workspace")
            ws = torch.empty(room, dtype=torch.uint8, device="cuda") if room else None
            Cd = torch.full((M, N), 2.0, device="cuda")
            call = lambda: B.gemm(1, tb, M, N, K, Ad, lda, Bd, ldb, Cd, N, B.BF16 if bf else B.F32, out_f32=1, ws=ws, ws_bytes=room, f32_product=form)  # noqa: E731
            if room < need:
                with pytest.raises(B.CapgnnError) as e:
                    call()
                assert e.value.code == B.ENOMEM
            else:
                call()
            torch.cuda.synchronize()
            got = Cd.cpu().numpy()
            assert (got == 2.0).all() if room < need else np.array_equal(got.astype(np.float64), ref), (M, N, K, room)


@pytest.mark.parametrize("M,N,K,parts", [(128, 256, 40_000, 32), (256, 256, 20_000, 16), (389, 16, 20_000, 39), (100, 41, 100_000, 121), (512, 200, 1000, 0)])
def test_gemm_bf16_aligned_vertex_reduction_with_little_workspace(env, M, N, K, parts):
    """X^T G of bf16 operands with aligned rows, which runs in registers with the workspace that the query names: with less, the small kernel's fewer
    splits, or the registers' at 16 steps of 32 each, down to the parts of the fewer of both; with four bytes less CAPGNN_ENOMEM, C
    untouched.  Small integers: exact with any number of splits."""
    torch, B = env["torch"], env["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M)
    lda, ldb = -(-M // 8) * 8, -(-N // 8) * 8
    A, G = (torch.randint(-3, 4, (K, w), generator=gen, device="cuda") for w in (lda, ldb))
    ref = A[:, :M].double().T @ G[:, :N].double()
    A, G = A.bfloat16(), G.bfloat16()
    fine = min(1536 // (-(-M // 128) * -(-N // (64 if N <= 64 else 128))), K // 512) * M * N * 4
    rooms = {parts * M * N * 4, (parts + 1) * M * N * 4, fine, B.gemm_workspace_bytes(1, M, N, K)}
    for room in sorted(rooms) + ([parts * M * N * 4 - 4, 0] if parts else []):
        say(f"gemm bf16 X^T G {M}x{N}x{K}: {room} bytes of workspace")
        ws = torch.empty(room, dtype=torch.uint8, device="cuda") if room else None
        Cd = torch.full((M, N), 2.0, device="cuda")
        call = lambda: B.gemm(1, 0, M, N, K, A, lda, G, ldb, Cd, N, B.BF16, out_f32=1, ws=ws, ws_bytes=room)  # noqa: E731
        if room < parts * M * N * 4:
            with pytest.raises(B.CapgnnError) as e:
                call()
            assert e.value.code == B.ENOMEM
        else:
            call()
        torch.cuda.synchronize()
        assert (Cd == 2.0).all() if room < parts * M * N * 4 else torch.equal(Cd.double(), ref), room


@pytest.mark.parametrize("ta,tb,M,N,K", [(0, 0, 164_001, 47, 40), (0, 1, 164_001, 64, 72), (0, 0, 82_100, 130, 24), (0, 1, 82_100, 200, 33), (1, 0, 513, 64, 131_100),
                                         (1, 1, 600, 41, 180_001), (1, 0, 300, 130, 38_400), (1, 1, 257, 250, 25_000)])
def test_gemm_bf16_full_size_tiles_exact(env, ta, tb, M, N, K):
    """The 128-row tiles of the bf16 kernel, 64 and 128 columns wide, at sizes that the 64-row tiles and the small kernel leave to them.
    Small integers (sums below 2^24): equality, which pins the operands' lane layout and the ragged edges."""
    torch, B = env["torch"], env["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M)
    mk = lambda r, c: torch.randint(-2, 3, (r, c), generator=gen, device="cuda")  # noqa: E731
    A, W = mk(*((K, M) if ta else (M, K))), mk(*((N, K) if tb else (K, N)))
    ref = (A.T if ta else A).double() @ (W.T if tb else W).double()
    pad = lambda x: torch.nn.functional.pad(x.bfloat16(), (0, -x.shape[1] % 8), value=float("nan")).contiguous()  # noqa: E731
    Ad, Wd = pad(A), pad(W)
    wsb = B.gemm_workspace_bytes(ta, M, N, K)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    for room in (wsb,) if ta else (wsb, 0):         # a plain product without one reads the weights as they are
        Cd = torch.full((M, N + 3), 2.0, device="cuda")
        say(f"gemm bf16 full-size tiles ta={ta} tb={tb} {M}x{N}x{K} workspace {room}")
        B.gemm(ta, tb, M, N, K, Ad, Ad.shape[1], Wd, Wd.shape[1], Cd, N + 3, B.BF16, out_f32=1, ws=ws if room else None, ws_bytes=room)
        torch.cuda.synchronize()
        assert torch.equal(Cd[:, :N].double(), ref) and (Cd[:, N:] == 2.0).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("M,N,K", [(1, 3, 64), (33, 32, 65), (97, 17, 111), (64, 33, 112), (31, 64, 127), (100, 130, 128), (65, 200, 144), (40, 64, 160), (129, 31, 191), (70, 47, 200),
                                   (500, 5, 255), (33, 65, 257), (96, 100, 384), (45, 256, 602)])
def test_gemm_small_plain_partial_batches_exact(env, dtype, tb, M, N, K):
    """Plain products of the small kernel whose waves have whole units, parts of a unit and none beside one another (K around units of 8 and 16 and
    the 128 and 256 of a batch of four waves); rows aligned and not; with the whole epilogue.  Small integers: equality."""
    torch, B = env["torch"], env["B"]
    td, dt = (torch.bfloat16, B.BF16) if dtype == "bf16" else (torch.float32, B.F32)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    mk = lambda r, c: torch.randint(-2, 3, (r, c), generator=gen, device="cuda").float()  # noqa: E731
    A, W, mask, bias = mk(M, K), mk(*((N, K) if tb else (K, N))), mk(M, N), mk(1, N)[0].contiguous()
    ref = A.double() @ (W.T if tb else W).double()
    for pad in (0, 1, 8):
        wide = lambda x: torch.nn.functional.pad(x, (0, (-x.shape[1] % 8 if pad == 8 else 0) + pad), value=float("nan")).to(td).contiguous()  # noqa: E731
        Ad, Wd, Md = wide(A), wide(W), wide(mask)
        wsb = B.gemm_workspace_bytes(0, M, N, K)
        ws = torch.empty(max(wsb, 1), dtype=torch.uint8, device="cuda")
        for full in (0, 1):
            say(f"gemm small plain {dtype} tb={tb} {M}x{N}x{K} pad={pad} epilogue={full}")
            Cd = torch.full((M, N + 3), 2.0, device="cuda")
            B.gemm(0, tb, M, N, K, Ad, Ad.shape[1], Wd, Wd.shape[1], Cd, N + 3, dt, out_f32=1, accumulate=full, bias=bias if full else None, relu=full,
                   relu_mask=Md if full and dtype == "f32" else None, ldm=Md.shape[1] if full and dtype == "f32" else 0, ws=ws, ws_bytes=wsb)
            torch.cuda.synchronize()
            want = (ref + 2.0 + bias).clamp(min=0) * ((mask > 0) if dtype == "f32" else 1) if full else ref
            assert torch.equal(Cd[:, :N].double(), want.double()) and (Cd[:, N:] == 2.0).all()


@pytest.mark.parametrize("M,N,K", [(512, 129, 1), (513, 200, 15), (602, 256, 17), (515, 131, 63), (512, 132, 65), (520, 250, 257), (601, 255, 1000), (100, 70, 21_001),
                                   (129, 65, 17_000), (40, 140, 30_011), (128, 256, 300_000), (97, 41, 70_001), (389, 2, 20_003), (130, 64, 50_000), (33, 129, 66_666)])
def test_gemm_bf16_vertex_reduction_in_registers_exact(env, M, N, K):
    """X^T G of bf16 operands with aligned rows at sizes that the small kernel leaves: tiles of 128 rows and of 64 and 128 columns whole and
    ragged, K around a step of 16, the four waves and the four steps of a turn, one split and many, last rows that end inside four columns; with
    the workspace that was asked for, with as little as the call accepts, and, there, with the whole epilogue, stored as float and as bf16.  Small
    integers (sums below 2^24, below 2^8 where they are stored as bf16): equality.  Padding is NaN; the last rows end with the allocation."""
    torch, B = env["torch"], env["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    A, G = (torch.randint(-3, 4, (K, w), generator=gen, device="cuda").float() for w in (M, N))
    ref = A.double().T @ G.double()
    bias = torch.randint(-9, 9, (N,), generator=gen, device="cuda").float()
    splits = min(1536 // (-(-M // 128) * -(-N // (64 if N <= 64 else 128))), K // 512)
    least = splits * M * N * 4 if splits > 1 else 0
    for pad in (0, 8):
        flat = lambda x: torch.cat([torch.nn.functional.pad(x[:-1], (0, -x.shape[1] % 8 + pad), value=float("nan")).reshape(-1), x[-1]]).bfloat16()  # noqa: E731
        Ad, Gd = flat(A), flat(G)
        lda, ldb = (-(-w // 8) * 8 + pad for w in (M, N))
        for room, full, f32 in ((B.gemm_workspace_bytes(1, M, N, K), 0, 1), (least, 0, 1), (least, 1, 1)) + (((least, 1, 0),) if K < 20 else ()):
            say(f"gemm bf16 X^T G in registers {M}x{N}x{K} pad={pad} workspace={room} epilogue={full} f32={f32}")
            ws = torch.empty(max(room, 1), dtype=torch.uint8, device="cuda")
            Cd = torch.full((M, N + 3), 2.0, device="cuda", dtype=torch.float32 if f32 else torch.bfloat16)
            B.gemm(1, 0, M, N, K, Ad, lda, Gd, ldb, Cd, N + 3, B.BF16, out_f32=f32, accumulate=full, bias=bias if full else None, relu=full, ws=ws,
                   ws_bytes=room)
            torch.cuda.synchronize()
            want = (ref + 2.0 + bias).clamp(min=0) if full else ref
            assert torch.equal(Cd[:, :N].double(), want) and (Cd[:, N:] == 2.0).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N", [(1, 1), (40, 32), (130, 47), (512, 129), (602, 256)])
def test_gemm_empty_reduction_is_the_epilogue_of_zeros(env, dtype, ta, tb, M, N):
    """K = 0, rows aligned and not, columns whole groups of four and not, every form of the fp32 product: zeros, with the epilogue where one is
    asked for.  Operands are rows of infinities around the empty matrices' addresses: none of them may be read."""
    torch, B = env["torch"], env["B"]
    td, dt = (torch.bfloat16, B.BF16) if dtype == "bf16" else (torch.float32, B.F32)
    bias, mask = torch.arange(N, device="cuda").float() - 3.0, torch.randint(-1, 2, (M, N), device="cuda").to(td)
    for pad in (8, 9):
        lda, ldb = -(-(M if ta else 1) // 8) * 8 + pad, -(-(N if not tb else 1) // 8) * 8 + pad
        A, W = (torch.full((4 * max(M, N) * ld + 8 * ld,), float("inf"), device="cuda").to(td)[4 * ld:] for ld in (lda, ldb))
        wsb = B.gemm_workspace_bytes(ta, M, N, 0)
        ws = torch.empty(max(wsb, 256), dtype=torch.uint8, device="cuda")
        for full, form, f32 in ((0, 0, 1), (1, 0, 1), (1, 0, 0)) + (((1, 1, 1), (1, 2, 1)) if dtype == "f32" else ()):
            say(f"gemm empty reduction {dtype} ta={ta} tb={tb} {M}x{N} pad={pad} epilogue={full} form={form} f32={f32}")
            Cd = torch.full((M, N + 3), 2.0, device="cuda", dtype=td if not f32 else torch.float32)
            B.gemm(ta, tb, M, N, 0, A, lda, W, ldb, Cd, N + 3, dt, out_f32=f32, accumulate=full, bias=bias if full else None, relu=full,
                   relu_mask=mask if full else None, ldm=N if full else 0, ws=ws, ws_bytes=wsb, f32_product=form)
            torch.cuda.synchronize()
            want = (2.0 + bias).clamp(min=0).expand(M, N) * (mask > 0) if full else torch.zeros(M, N, device="cuda")
            assert torch.equal(Cd[:, :N].double(), want.to(Cd.dtype).double()) and (Cd[:, N:] == 2.0).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("kind", ["gcn", "sage"])
@pytest.mark.parametrize("f_in,f_out", [(602, 47), (33, 130), (64, 64)])
def test_layer_gradients_of_a_partition_without_local_rows_are_zero(env, dtype, kind, f_in, f_out):
    """AGG_FIRST on a partition of halo rows alone: weight and bias gradients are empty sums."""
    torch, B = env["torch"], env["B"]
    td, dt = (torch.bfloat16, B.BF16) if dtype == "bf16" else (torch.float32, B.F32)
    sage = kind == "sage"
    g = B.Graph(0, 5, np.zeros(1, np.int64), np.zeros(0, np.int32), np.ones(0, np.float32), np.ones(5, np.float32))
    ldi, ldo = -(-f_in // 8) * 8, -(-f_out // 8) * 8
    big = lambda r, c: torch.full((r, c), float("inf"), device="cuda").to(td)  # noqa: E731
    x, h, dh, w, w_self, bias = big(5, ldi), big(4, ldo), big(4, ldo), big(f_in, f_out), big(f_in, f_out), torch.zeros(f_out, device="cuda")
    l = B.make_layer(B.SAGE_MEAN if sage else B.GCN, f_in, f_out, B.ACT_RELU, dt, w, w_self if sage else None, bias, B.AGG_FIRST)
    wsb = B.layer_workspace_bytes(g, l)
    saved, ws = big(8, ldi), torch.empty(max(wsb, 256), dtype=torch.uint8, device="cuda")
    dw, dws, db = torch.full((f_in, f_out), 7.0, device="cuda"), torch.full((f_in, f_out), 7.0, device="cuda"), torch.full((f_out,), 7.0, device="cuda")
    say(f"layer without local rows {kind} {dtype} {f_in}-{f_out}")
    B.layer_fwd(g, l, x, ldi, h, ldo, saved, ws, wsb)
    B.layer_bwd(g, l, x, ldi, h, ldo, saved, dh, ldo, dw, dws if sage else None, db, None, 0, 0, ws, wsb)
    torch.cuda.synchronize()
    assert not dw.any() and not db.any() and not (sage and dws.any())
    g.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,f_in,f_out", [(40_000, 100, 100), (70_001, 131, 200), (20_003, 520, 136), (66_000, 97, 64)])
def test_layer_pair_of_weight_gradients_in_registers_exact(env, dtype, n, f_in, f_out):
    """Both weight gradients of a GraphSAGE layer in one launch of the kernels that hold their results in registers (fp32 above 64 columns), and its
    bias gradient, one entry of weight one per row.  Small integers (sums below 2^24): equality."""
    torch, B = env["torch"], env["B"]
    td, dt = (torch.bfloat16, B.BF16) if dtype == "bf16" else (torch.float32, B.F32)
    rng = np.random.default_rng(n)
    col = rng.integers(0, n, n).astype(np.int32)
    g = B.Graph(n, 0, np.arange(0, n + 1, dtype=np.int64), col, np.ones(n, np.float32), np.ones(n, np.float32))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    ldi, ldo = -(-f_in // 8) * 8, -(-f_out // 8) * 8
    x, dh = (torch.nn.functional.pad(torch.randint(-3, 4, (n, w), generator=gen, device="cuda").to(td), (0, ld - w)) for w, ld in ((f_in, ldi), (f_out, ldo)))
    w, w_self = (torch.zeros(f_in, f_out, device="cuda", dtype=td) for _ in range(2))
    l = B.make_layer(B.SAGE_MEAN, f_in, f_out, B.ACT_NONE, dt, w, w_self, torch.zeros(f_out, device="cuda"), B.AGG_FIRST)
    saved = torch.empty(B.layer_saved_bytes(g, l), dtype=torch.uint8, device="cuda")
    wsb = B.layer_workspace_bytes(g, l)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    h = torch.zeros(n, ldo, device="cuda", dtype=td)
    dw, dws, db = torch.zeros(f_in, f_out, device="cuda"), torch.zeros(f_in, f_out, device="cuda"), torch.zeros(f_out, device="cuda")
    say(f"pair of weight gradients {dtype} {n} {f_in}->{f_out}")
    B.layer_fwd(g, l, x, ldi, h, ldo, saved, ws, wsb, None)
    B.layer_bwd(g, l, x, ldi, h, ldo, saved, dh.clone(), ldo, dw, dws, db, None, 0, False, ws, wsb, None)
    torch.cuda.synchronize()
    X, D = x[:, :f_in].double(), dh[:, :f_out].double()
    m = X[torch.from_numpy(col).long().cuda()]
    assert torch.equal(dw.double(), m.T @ D) and torch.equal(dws.double(), X.T @ D)
    assert torch.equal(db.double(), D.sum(0))


@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("M,N,K", [(16384, 128, 128), (16385, 65, 7), (16415, 100, 129), (20000, 130, 200), (16399, 256, 256), (50001, 257, 47),
                                   (16386, 300, 256), (17003, 200, 257), (16384, 72, 511), (16417, 256, 512), (16383, 256, 64), (16390, 256, 520),
                                   (30_000, 128, 128), (30_001, 72, 96), (25_009, 66, 100), (70_017, 160, 257), (60_031, 256, 256), (33_001, 250, 200), (49_185, 100, 129),
                                   (24_577, 65, 7), (16_417, 256, 16), (24_600, 72, 17), (16_400, 200, 32)])
def test_gemm_bf16_many_rows_exact(env, tb, M, N, K):
    """bf16 products of many rows whose result is stored as bf16 (weights held in registers from 16384 rows on): the last tile of
    rows whole, short and of one row, K around a unit and around 128, 256 and 512, N not a multiple of eight, of a wave's 32 and of a
    workgroup's columns; with and without bias, ReLU and mask.  Integers of at most 8 bits: equality.  Padding of every operand is NaN
    and C's own stays as it is."""
    torch, B = env["torch"], env["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    mk = lambda r, c: torch.randint(-1, 2, (r, c), generator=gen, device="cuda").float()  # noqa: E731
    A, W = mk(M, K), mk(*((N, K) if tb else (K, N))) * (torch.rand((N, K) if tb else (K, N), generator=gen, device="cuda") < 0.1)
    bias, mask = mk(1, N)[0].contiguous(), mk(M, N)
    pad = lambda x: torch.nn.functional.pad(x.bfloat16(), (0, -x.shape[1] % 8 + 8), value=float("nan")).contiguous()  # noqa: E731
    Ad, Wd, Md = pad(A), pad(W), pad(mask)
    plain = A @ (W.T if tb else W)
    assert float(plain.abs().max()) < 250
    wsb = B.gemm_workspace_bytes(0, M, N, K)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    ldc = (N + 7) // 8 * 8 + 8
    for use_bias, relu, use_mask in ((False, 0, False), (True, 1, False), (False, 0, True)):
        say(f"gemm bf16 many rows tb={tb} {M}x{N}x{K} bias={use_bias} relu={relu} mask={use_mask}")
        Cd = torch.full((M, ldc), 2.0, device="cuda", dtype=torch.bfloat16)
        B.gemm(0, tb, M, N, K, Ad, Ad.shape[1], Wd, Wd.shape[1], Cd, ldc, B.BF16, bias=bias if use_bias else None, relu=relu,
               relu_mask=Md if use_mask else None, ldm=Md.shape[1] if use_mask else 0, ws=ws, ws_bytes=wsb)
        torch.cuda.synchronize()
        ref = plain + bias if use_bias else plain
        ref = ref.clamp(min=0) if relu else ref
        ref = ref * (mask > 0) if use_mask else ref
        assert torch.equal(Cd[:, :N].float(), ref) and (Cd[:, N:] == 2.0).all()


@pytest.mark.parametrize("M,N,K,mask,streamed", [(20_000, 72, 64, 0, 0), (25_000, 72, 64, 0, 1), (30_000, 120, 248, 1, 1), (20_000, 120, 248, 1, 0), (50_000, 96, 320, 0, 0),
                                                 (50_000, 96, 448, 0, 1), (50_000, 66, 200, 0, 0), (25_000, 66, 100, 0, 1), (50_000, 100, 128, 1, 0), (16_384, 256, 160, 0, 1),
                                                 (16_384, 160, 160, 0, 0), (30_000, 160, 160, 0, 1), (50_000, 160, 160, 1, 0), (90_000, 160, 160, 1, 1), (40_000, 248, 248, 1, 0),
                                                 (60_000, 248, 248, 1, 1), (16_384, 504, 120, 1, 1), (50_000, 300, 64, 0, 0), (50_000, 250, 200, 0, 1), (50_000, 250, 200, 1, 0),
                                                 (16_383, 248, 200, 0, 0), (100_000, 64, 128, 0, 0),
                                                 (30_000, 65, 7, 0, 1), (30_000, 72, 16, 0, 1), (20_000, 256, 24, 0, 1), (20_000, 200, 32, 0, 1), (70_000, 128, 7, 1, 1)])
def test_gemm_bf16_many_rows_route(env, M, N, K, mask, streamed):
    """Which bf16 products of many rows keep their weights in registers and which run in tiles, from the image of the weights left in the
    workspace, at sizes where each is the faster one and with the workspace that was asked for; the result of either against float64 (one rounding, 2^-8 of a value at most, and
    sums in float: 2^-9 in the 2-norm)."""
    torch, B = env["torch"], env["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    pad = lambda x: torch.nn.functional.pad(x.bfloat16(), (0, -x.shape[1] % 8)).contiguous()  # noqa: E731
    A, W, Md = (pad(torch.randn(r, c, generator=gen, device="cuda")) for r, c in ((M, K), (K, N), (M, N)))
    wsb = B.gemm_workspace_bytes(0, M, N, K)
    ws = torch.full((wsb,), 0xA5, dtype=torch.uint8, device="cuda")
    C = torch.zeros(M, Md.shape[1], dtype=torch.bfloat16, device="cuda")
    say(f"gemm bf16 route {M}x{N}x{K} mask={mask}")
    B.gemm(0, 0, M, N, K, A, A.shape[1], W, W.shape[1], C, C.shape[1], B.BF16, relu_mask=Md if mask else None, ldm=Md.shape[1] if mask else 0, ws=ws, ws_bytes=wsb)
    torch.cuda.synchronize()
    units = 8 if K <= 128 else 16 if K <= 256 else 32
    tiled = N * -(-K // 8) * 16                                         # the weights as the tiles read them, at most
    image = -(-N // 128) * 128 * units * 32
    assert tiled < image <= wsb
    assert bool((ws[tiled:image] != 0xA5).any()) == bool(streamed)
    ref = A[:, :K].double() @ W[:, :N].double()
    ref = ref * (Md[:, :N] > 0) if mask else ref
    assert float((C[:, :N].double() - ref).norm()) <= 2.0 ** -9 * float(ref.norm())


@pytest.mark.parametrize("M,N,K", [(1, 1, 16384), (3, 7, 16385), (64, 16, 16387), (100, 17, 20003), (127, 32, 16447), (128, 33, 16449), (130, 41, 30001),
                                   (257, 48, 16400), (602, 49, 17000), (255, 64, 65537)])
def test_gemm_f32_narrow_vertex_reduction_exact(env, M, N, K):
    """X^T G in float with at most 64 columns over 16384 vertices and more: tiles of 16 columns and of 128 rows whole and ragged, K around
    batches and splits, rows aligned and not, accumulating and with bias and ReLU; with less than the workspace asked for, the splits of
    the staged kernel (one for every 16 steps of 16, and no more than fill the chip six times), and with room for two splits
    CAPGNN_ENOMEM, C untouched.  Small integers (sums below 2^24): equality.  Padding is NaN; the last rows end with the allocation."""
    torch, B = env["torch"], env["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    A, G = (torch.randint(-3, 4, (K, w), generator=gen, device="cuda").float() for w in (M, N))
    ref = A.double().T @ G.double()
    bias = torch.randint(-9, 9, (N,), generator=gen, device="cuda").float()
    wsb = B.gemm_workspace_bytes(1, M, N, K)
    for pad in (0, 1, 4):
        flat = lambda x: torch.cat([torch.nn.functional.pad(x[:-1], (0, pad), value=float("nan")).reshape(-1), x[-1]])  # noqa: E731
        Ad, Gd = flat(A), flat(G)
        least = min(1536 // -(-M // 128), K // 256) * M * N * 4
        for room, accumulate, relu in ((wsb, 0, 0), (wsb, 1, 1), (least, 0, 0), (2 * M * N * 4, 0, 0)):
            say(f"gemm narrow X^T G {M}x{N}x{K} pad={pad} workspace={room} accumulate={accumulate}")
            ws = torch.empty(room, dtype=torch.uint8, device="cuda")
            Cd = torch.full((M, N + 3), 2.0, device="cuda")
            call = lambda: B.gemm(1, 0, M, N, K, Ad, M + pad, Gd, N + pad, Cd, N + 3, B.F32, accumulate=accumulate, bias=bias if relu else None,  # noqa: E731
                                  relu=relu, ws=ws, ws_bytes=room)
            if room == 2 * M * N * 4:
                with pytest.raises(B.CapgnnError) as e:
                    call()
                torch.cuda.synchronize()
                assert e.value.code == B.ENOMEM and (Cd == 2.0).all()
                continue
            call()
            torch.cuda.synchronize()
            want = (ref + 2.0 + bias).clamp(min=0) if accumulate else ref
            assert torch.equal(Cd[:, :N].double(), want) and (Cd[:, N:] == 2.0).all()


@pytest.mark.parametrize("M,N,K", [(64, 41, 20_000), (128, 47, 250_000), (128, 24, 300_000), (256, 64, 40_000), (264, 20, 30_000), (300, 41, 200_000), (602, 64, 16_384)])
def test_gemm_f32_narrow_vertex_reduction_fills_the_chip_evenly(env, M, N, K):
    """With the workspace that was asked for, a narrow X^T G is cut into as many parts as make one workgroup per compute unit, or two where
    the parts are long, and no number between: counted in the parts left in the workspace.  Small integers: equality."""
    torch, B = env["torch"], env["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    A, G = (torch.randint(-3, 4, (K, w), generator=gen, device="cuda").float() for w in (M, N))
    wsb = B.gemm_workspace_bytes(1, M, N, K)
    ws = torch.full((wsb // 4,), float("nan"), device="cuda")
    C = torch.zeros(M, N, device="cuda")
    say(f"gemm narrow X^T G parts {M}x{N}x{K}")
    B.gemm(1, 0, M, N, K, A, M, G, N, C, N, B.F32, ws=ws, ws_bytes=wsb)
    torch.cuda.synchronize()
    tiles, per_cu = -(-M // 128), 2 if K * -(-M // 128) > 1 << 18 else 1
    most = 256 * per_cu // tiles
    assert int((~ws.isnan()).sum()) == M * N * (most // 8 * 8 if most > 8 else most)
    assert torch.equal(C.double(), A.double().T @ G.double())


@pytest.mark.parametrize("n,f_in,f_out", [(16384, 100, 41), (20001, 130, 64), (40000, 64, 8)])
def test_layer_narrow_weight_gradients_exact(env, n, f_in, f_out):
    """Both weight gradients and the bias gradient of a GraphSAGE layer with at most 64 outputs, over 16384 vertices and more, one entry
    of weight one per row.  Small integers: equality."""
    torch, B = env["torch"], env["B"]
    rng = np.random.default_rng(n)
    col = rng.integers(0, n, n).astype(np.int32)
    g = B.Graph(n, 0, np.arange(0, n + 1, dtype=np.int64), col, np.ones(n, np.float32), np.ones(n, np.float32))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    x, dh = (torch.randint(-3, 4, (n, w), generator=gen, device="cuda").float() for w in (f_in, f_out))
    w, w_self = (torch.zeros(f_in, f_out, device="cuda") for _ in range(2))
    l = B.make_layer(B.SAGE_MEAN, f_in, f_out, B.ACT_NONE, B.F32, w, w_self, torch.zeros(f_out, device="cuda"), B.AGG_FIRST)
    saved = torch.empty(B.layer_saved_bytes(g, l), dtype=torch.uint8, device="cuda")
    wsb = B.layer_workspace_bytes(g, l)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    h, dw, dws, db = torch.zeros(n, f_out, device="cuda"), torch.zeros_like(w), torch.zeros_like(w), torch.zeros(f_out, device="cuda")
    say(f"narrow weight gradients of a layer {n} {f_in}->{f_out}")
    B.layer_fwd(g, l, x, f_in, h, f_out, saved, ws, wsb, None)
    B.layer_bwd(g, l, x, f_in, h, f_out, saved, dh.clone(), f_out, dw, dws, db, None, 0, False, ws, wsb, None)
    torch.cuda.synchronize()
    m = x[torch.from_numpy(col).long().cuda()]
    assert torch.equal(dw.double(), m.double().T @ dh.double()) and torch.equal(dws.double(), x.double().T @ dh.double())
    assert torch.equal(db.double(), dh.double().sum(0))


@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("M,N,K", [(24609, 128, 128), (24608, 65, 7), (24640, 100, 129), (20000, 132, 200), (16399, 256, 256), (50001, 255, 47),
                                   (12288, 200, 256), (12321, 256, 255), (12352, 196, 128), (49183, 64, 256), (49153, 47, 130), (50000, 1, 200),
                                   (70_001, 121, 100), (70_016, 125, 128), (33_025, 255, 127), (20_011, 200, 161), (70_001, 100, 192), (45_057, 96, 129)])
def test_gemm_f32_many_rows_exact(env, tb, M, N, K):
    """fp32 products of many rows in three bf16 pieces (weights held in registers where 64 x 64 tiles do not fit the chip at once, up to
    256 columns and 256 k): the last tile of rows whole, short and of one row, K around a unit and around 128 and 256, N not a multiple of
    four and of a wave's 32; with and without bias, ReLU and mask.  Sums of integers that need two and three pieces but fit 24 bits: equality.  Padding of
    every operand is NaN and C's own stays as it is."""
    torch, B = env["torch"], env["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    mk = lambda r, c, m: torch.randint(-m, m + 1, (r, c), generator=gen, device="cuda").float()  # noqa: E731
    A = mk(M, K, 511)                                                   # 9 bits and a sign: two pieces
    W = mk(*((N, K) if tb else (K, N)), 20)
    bias, mask = mk(1, N, 70000)[0].contiguous(), mk(M, N, 1)
    pad = lambda x: torch.nn.functional.pad(x, (0, -x.shape[1] % 4 + 4), value=float("nan")).contiguous()  # noqa: E731
    Ad, Wd, Md = pad(A), pad(W), pad(mask)
    Ad[3, 0] = A[3, 0] = 2.0 ** 17 - 1                                  # 17 bits: three pieces
    plain = A.double() @ (W.T if tb else W).double()
    assert float(plain.abs().max()) < 2 ** 24 - 70000
    wsb = B.gemm_workspace_bytes(0, M, N, K)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    ldc = (N + 3) // 4 * 4 + 4
    for use_bias, relu, use_mask in ((False, 0, False), (True, 1, False), (False, 0, True)):
        say(f"gemm f32 many rows tb={tb} {M}x{N}x{K} bias={use_bias} relu={relu} mask={use_mask}")
        Cd = torch.full((M, ldc), 2.0, device="cuda")
        B.gemm(0, tb, M, N, K, Ad, Ad.shape[1], Wd, Wd.shape[1], Cd, ldc, B.F32, bias=bias if use_bias else None, relu=relu,
               relu_mask=Md if use_mask else None, ldm=Md.shape[1] if use_mask else 0, ws=ws, ws_bytes=wsb, f32_product=B.F32_PRODUCT_SPLIT)
        torch.cuda.synchronize()
        ref = plain + bias.double() if use_bias else plain
        ref = ref.clamp(min=0) if relu else ref
        ref = ref * (mask > 0) if use_mask else ref
        assert torch.equal(Cd[:, :N].double(), ref) and (Cd[:, N:] == 2.0).all()


@pytest.mark.parametrize("M,N,K,streamed", [(26_000, 128, 129, 0), (30_000, 128, 160, 0), (30_000, 100, 192, 0), (70_000, 256, 176, 0), (60_000, 132, 224, 0),
                                            (26_000, 96, 256, 0), (30_000, 122, 256, 0), (20_000, 200, 160, 1), (70_000, 100, 192, 1), (70_000, 200, 256, 1),
                                            (33_000, 128, 200, 1)])
def test_gemm_f32_reductions_of_129_to_256_in_one_chain_or_two(env, M, N, K, streamed):
    """Which of the two kernels for many rows forms a product in three bf16 pieces: above 128 k the one that keeps the weights in registers
    adds two chains, the tiled one, which also takes results whose rows do not start on 16 bytes, a single one.  So the results of
    aligned and unaligned rows are the same bits where the tiled kernel takes both (it is the faster one there), and differ somewhere
    where the other does."""
    torch, B = env["torch"], env["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    pad = lambda w: (w + 3) // 4 * 4  # noqa: E731
    A, W = torch.randn(M, pad(K), generator=gen, device="cuda"), torch.randn(K, N, generator=gen, device="cuda")
    wsb = B.gemm_workspace_bytes(0, M, N, K)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    got = []
    for ldc in (pad(N), pad(N) + 1):
        say(f"gemm f32 chains {M}x{N}x{K} pitch {ldc}")
        C = torch.zeros(M, ldc, device="cuda")
        B.gemm(0, 0, M, N, K, A, A.shape[1], W, N, C, ldc, B.F32, ws=ws, ws_bytes=wsb, f32_product=B.F32_PRODUCT_SPLIT)
        torch.cuda.synchronize()
        got.append(C[:, :N])
    ref = A[:, :K].double() @ W.double()
    assert all(float((c - ref).norm()) <= 4e-7 * float(ref.norm()) for c in got)
    assert torch.equal(*got) == (not streamed)


@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("M,N,K", [(1000, 30, 40), (4095, 130, 72), (10_001, 100, 100), (16_500, 41, 256), (30_001, 32, 20), (20_000, 41, 300), (13_001, 70, 300), (30_001, 100, 100),
                                   (30_017, 130, 300), (60_001, 47, 24), (60_001, 64, 100), (60_001, 201, 32), (50_001, 100, 20)])
def test_gemm_f32_epilogues_exact(env, tb, M, N, K):
    """C (+)= A W with bias, ReLU and mask on every kernel of the fp32 path, in both forms of the product: epilogue operands asked for
    ahead of the loop or behind it (two and three workgroups per compute unit), staged tiles of 64 and 128 columns that accumulate over
    one step of the reduction and over more, ragged last rows and columns.  Sums of integers that fit 24 bits: equality.  Padding of
    every operand is NaN and C's own stays as it is."""
    torch, B = env["torch"], env["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    mk = lambda r, c, m: torch.randint(-m, m + 1, (r, c), generator=gen, device="cuda").float()  # noqa: E731
    A, W, C0, mask, bias = mk(M, K, 511), mk(*((N, K) if tb else (K, N)), 20), mk(M, N, 70000), mk(M, N, 1), mk(1, N, 70000)[0].contiguous()
    plain = A.double() @ (W.T if tb else W).double()
    assert float(plain.abs().max()) < 2 ** 24 - 140000
    wsb = B.gemm_workspace_bytes(0, M, N, K)
    ws = torch.empty(max(wsb, 256), dtype=torch.uint8, device="cuda")
    for mult in (4, 1):                                                 # whole vectors, or the bare width plus one
        pad = lambda x: torch.nn.functional.pad(x, (0, -x.shape[1] % mult + mult), value=float("nan")).contiguous()  # noqa: E731
        Ad, Wd, Md = pad(A), pad(W), pad(mask)
        for form in (B.F32_PRODUCT_NATIVE, B.F32_PRODUCT_SPLIT):
            for acc, use_bias, relu, use_mask in ((1, False, 0, False), (0, False, 0, True), (1, True, 1, True), (0, True, 1, False)):
                say(f"gemm f32 epilogue tb={tb} {M}x{N}x{K} pitch {mult} form={form} accumulate={acc} bias={use_bias} mask={use_mask}")
                Cd = pad(C0)
                B.gemm(0, tb, M, N, K, Ad, Ad.shape[1], Wd, Wd.shape[1], Cd, Cd.shape[1], B.F32, accumulate=acc, bias=bias if use_bias else None,
                       relu=relu, relu_mask=Md if use_mask else None, ldm=Md.shape[1] if use_mask else 0, ws=ws, ws_bytes=wsb, f32_product=form)
                torch.cuda.synchronize()
                ref = plain + C0 if acc else plain
                ref = ref + bias.double() if use_bias else ref
                ref = ref.clamp(min=0) if relu else ref
                ref = ref * (mask > 0) if use_mask else ref
                assert torch.equal(Cd[:, :N].double(), ref) and Cd[:, N:].isnan().all()


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0)])
def test_gemm_f32_split_product(env, ta, tb):
    """fp32 operands cut into three bf16 pieces and multiplied on the bf16 matrix cores.  (1) With one operand a signed
    selection matrix (one +-2^e entry per output column / row) every output is a single product that fp32 holds exactly, so
    all 24 bits of the other operand must come through: bit-exact, which pins the cut, the piece order and the LDS
    layouts.  The last three plain shapes have more than 768 tiles of 64 x 64 and run gemm_split_kernel, in both of its widths; the
    others run gemm_split_mid_kernel.  (2) Random operands: within the fp32 tolerance of the fp64 oracle, and no further from it than four times
    the distance of the fp32 matrix instruction plus 2^-23, the bound on the three piece products that are dropped (both
    distances are rounding noise of the fp32 accumulation, a hundred times below the tolerance)."""
    torch, B, H, O, orc = env["torch"], env["B"], env["H"], env["O"], env["orc"]
    rng = np.random.default_rng(40 + ta * 2 + tb)

    def run(mode, A, Bm, M, N, K, pad):
        lda, ldb, ldc = A.shape[1] + pad, Bm.shape[1] + pad, N + pad
        Ad, Bd = H.padded_matrix(A, lda), H.padded_matrix(Bm, ldb)
        wsb = B.gemm_workspace_bytes(ta, M, N, K)
        ws = torch.empty(max(wsb, 256), dtype=torch.uint8, device="cuda")
        Cd = torch.full((M, ldc), 2.0, dtype=torch.float32, device="cuda")
        B.gemm(ta, tb, M, N, K, Ad, lda, Bd, ldb, Cd, ldc, B.F32, out_f32=1, ws=ws, ws_bytes=wsb, f32_product=mode)
        torch.cuda.synchronize()
        got = Cd.cpu().numpy()
        assert (got[:, N:] == 2.0).all()
        return got[:, :N]

    for (M, N, K) in [(1, 1, 1), (130, 41, 602), (257, 256, 100), (300, 130, 1000), (602, 256, 5000), (64, 200, 33)] + ([] if ta else [
            (49217, 64, 37), (50000, 41, 66), (16500, 200, 70)]):
        shapeA, shapeB = ((K, M) if ta else (M, K)), ((N, K) if tb else (K, N))
        for which in ("select_b", "select_a", "random"):
            say(f"gemm f32 split ta={ta} tb={tb} M={M} N={N} K={K} {which}")
            full = lambda shape: (rng.integers(1 << 23, 1 << 24, shape) * rng.choice([-1.0, 1.0], shape)
                                  * 2.0 ** rng.integers(-20, 20, shape)).astype(np.float32)
            if which == "select_b":              # B[k_j, j] = +-2^e, zero elsewhere
                A = full(shapeA)
                sel = np.zeros((K, N), np.float32)
                sel[rng.integers(0, K, N), np.arange(N)] = rng.choice([-1.0, 1.0], N) * 2.0 ** rng.integers(-8, 8, N)
                Bm = np.ascontiguousarray(sel.T) if tb else sel
            elif which == "select_a":            # A[i, k_i] = +-2^e (op(A) is M x K)
                Bm = full(shapeB)
                sel = np.zeros((M, K), np.float32)
                sel[np.arange(M), rng.integers(0, K, M)] = rng.choice([-1.0, 1.0], M) * 2.0 ** rng.integers(-8, 8, M)
                A = np.ascontiguousarray(sel.T) if ta else sel
            else:
                A = rng.standard_normal(shapeA).astype(np.float32)
                Bm = rng.standard_normal(shapeB).astype(np.float32)
            ref = orc.matmul(A, Bm, ta=bool(ta), tb=bool(tb))
            for pad in (0, 3):
                got = run(B.F32_PRODUCT_SPLIT, A, Bm, M, N, K, pad)
                if which != "random":
                    assert np.array_equal(got.astype(np.float64), ref)
                    continue
                nat = run(B.F32_PRODUCT_NATIVE, A, Bm, M, N, K, pad)
                e_split, e_nat = O.normwise(got, ref), O.normwise(nat, ref)
                say(f"   normwise error: split {e_split:.3e}, fp32 instruction {e_nat:.3e}")
                assert e_split <= TOL_F32 and e_nat <= TOL_F32
                assert e_split <= 4.0 * e_nat + 2.0 ** -23
    one = torch.zeros(1, device="cuda")
    with pytest.raises(B.CapgnnError):          # an unknown form is an argument error
        B.gemm(0, 0, 1, 1, 1, one, 1, one, 1, one, 1, B.F32, f32_product=7)


@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (63, 65, 15), (64, 64, 16), (65, 63, 31), (130, 128, 32), (257, 41, 33), (64, 200, 47), (300, 130, 127), (1000, 100, 128), (129, 64, 129),
                                   (4097, 200, 200), (2000, 256, 602), (21_557, 128, 257)])
def test_gemm_f32_split_quarters_exact(env, tb, M, N, K):
    """Three-piece products of few 64 x 64 tiles, whose four waves take quarters of the reduction: tiles whole and ragged, K around a step of 16, a pair
    of them and the eight of four waves; rows aligned and not; with the whole epilogue.  Integers of nine bits by -1, 0 and 1 (sums below
    2^24): equality.  Padding is NaN; the last rows end with the allocation."""
    torch, B = env["torch"], env["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    A = torch.randint(-400, 401, (M, K), generator=gen, device="cuda").float()
    W = torch.randint(-1, 2, (N, K) if tb else (K, N), generator=gen, device="cuda").float()
    mask, bias = torch.randint(-1, 2, (M, N), generator=gen, device="cuda").float(), torch.randint(-9, 9, (N,), generator=gen, device="cuda").float()
    ref = A.double() @ (W.T if tb else W).double()
    wsb = B.gemm_workspace_bytes(0, M, N, K)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    for pad in (0, 1, 4):
        flat = lambda x: torch.cat([torch.nn.functional.pad(x[:-1], (0, pad), value=float("nan")).reshape(-1), x[-1]])  # noqa: E731
        Ad, Wd, Md = flat(A), flat(W), flat(mask)
        for full in (0, 1):
            say(f"gemm split quarters tb={tb} {M}x{N}x{K} pad={pad} epilogue={full}")
            Cd = torch.full((M, N + pad), 2.0, device="cuda")
            B.gemm(0, tb, M, N, K, Ad, K + pad, Wd, W.shape[1] + pad, Cd, N + pad, B.F32, accumulate=full, bias=bias if full else None, relu=full,
                   relu_mask=Md if full else None, ldm=N + pad if full else 0, ws=ws, ws_bytes=wsb, f32_product=B.F32_PRODUCT_SPLIT)
            torch.cuda.synchronize()
            want = (ref + 2.0 + bias).clamp(min=0) * (mask > 0) if full else ref
            assert torch.equal(Cd[:, :N].double(), want.double()) and (Cd[:, N:] == 2.0).all()


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (127, 65, 15), (128, 64, 16), (129, 128, 17), (33, 129, 47), (130, 192, 64), (128, 128, 65), (257, 200, 600), (96, 256, 2049),
                                   (602, 100, 5000), (64, 41, 20_001), (300, 130, 38_401), (100, 256, 70_001), (128, 128, 300_000), (700, 600, 1600)])
def test_gemm_f32_split_vertex_reduction_exact(env, M, N, K):
    """X^T G in three bf16 pieces: tiles of 128 rows and of 64 and 128 columns whole and ragged, K around a step of 16, the two steps of a loop
    and the four waves of a workgroup, one split and many, one part of a split and several (300 000); rows aligned and not; with the workspace
    that was asked for, with as little as the call accepts, and, where there is one split, with the whole epilogue.  Integers of nine bits by
    -1, 0 and 1 (sums below 2^24): equality.  Padding is NaN; the last rows end with the allocation."""
    torch, B = env["torch"], env["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    A = torch.randint(-400, 401, (K, M), generator=gen, device="cuda").float()
    G = torch.randint(-1, 2, (K, N), generator=gen, device="cuda").float()
    ref = A.double().T @ G.double()
    assert float(ref.abs().max()) < 2 ** 24
    bias = torch.randint(-9, 9, (N,), generator=gen, device="cuda").float()
    splits = min(1536 // (-(-M // 128) * -(-N // (64 if N <= 64 else 128))), K // 512)
    least = splits * M * N * 4 if splits > 1 else 0
    for pad in (0, 1, 4):
        flat = lambda x: torch.cat([torch.nn.functional.pad(x[:-1], (0, pad), value=float("nan")).reshape(-1), x[-1]])  # noqa: E731
        Ad, Gd = flat(A), flat(G)
        for room, full in ((B.gemm_workspace_bytes(1, M, N, K), 0), (least, 0), (least, 1)):
            say(f"gemm split X^T G {M}x{N}x{K} pad={pad} workspace={room} epilogue={full}")
            ws = torch.empty(max(room, 1), dtype=torch.uint8, device="cuda")
            Cd = torch.full((M, N + 3), 2.0, device="cuda")
            B.gemm(1, 0, M, N, K, Ad, M + pad, Gd, N + pad, Cd, N + 3, B.F32, accumulate=full, bias=bias if full else None, relu=full, ws=ws,
                   ws_bytes=room, f32_product=B.F32_PRODUCT_SPLIT)
            torch.cuda.synchronize()
            want = (ref + 2.0 + bias).clamp(min=0) if full else ref
            assert torch.equal(Cd[:, :N].double(), want) and (Cd[:, N:] == 2.0).all()


@pytest.mark.parametrize("n,dims", [(100_000, (40, 100, 70)), (30_011, (130, 121, 9))])
def test_epoch_bias_gradient_of_split_weight_gradients(env, n, dims):
    """The hidden layer's bias gradient, whose columns the three-piece X^T G sums on its way (64 and 128 columns of a workgroup), on a graph of
    self loops.  Against fp64: each dZ is off by a few fp32 roundings of its terms, the sum by less than 1e-6 of the sum of their magnitudes."""
    torch, B = env["torch"], env["B"]
    assert n * dims[0] * dims[1] >= 1.375 * 2 ** 28
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    g = B.Graph(n, 0, np.arange(0, n + 1, dtype=np.int64), np.arange(n, dtype=np.int32), np.ones(n, np.float32), np.ones(n, np.float32))
    x = torch.randn(n, dims[0], generator=gen, device="cuda")
    w = [torch.randn(a, b, generator=gen, device="cuda") / a ** 0.5 for a, b in zip(dims, dims[1:])]
    b = [0.1 * torch.randn(d, generator=gen, device="cuda") for d in dims[1:]]
    labels = torch.randint(0, dims[-1], (n,), generator=gen, device="cuda", dtype=torch.int32)
    dw, db = [torch.zeros_like(t) for t in w], [torch.zeros_like(t) for t in b]
    layers = [B.make_layer(B.GCN, a, c, act, B.F32, w[i], None, b[i], B.AGG_FIRST)
              for i, (a, c, act) in enumerate(zip(dims, dims[1:], (B.ACT_RELU, B.ACT_NONE)))]
    wsb = B.epoch_workspace_bytes(g, None, layers)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    logits = torch.zeros(n, dims[-1], device="cuda")
    say(f"bias gradient beside a three-piece weight gradient n={n} {dims}")
    B.epoch(g, None, layers, x, dims[0], labels, None, 0.0, logits, dw, None, db, 0.0, ws, wsb, None, None, want_loss=False)
    torch.cuda.synchronize()
    h = (x.double() @ w[0].double() + b[0].double()).clamp(min=0)
    p = torch.softmax(h @ w[1].double() + b[1].double(), 1)
    p[torch.arange(n, device="cuda"), labels.long()] -= 1.0
    dz = (p / n) @ w[1].double().T * (h > 0)
    assert ((db[0].double() - dz.sum(0)).abs() <= 1e-6 * dz.abs().sum(0)).all()
    assert ((dw[0].double() - x.double().T @ dz).abs() <= 2e-6 * (x.abs().double().T @ dz.abs())).all()


@pytest.mark.parametrize("tb", [0, 1])
def test_gemm_f32_auto_form_is_the_documented_one(env, tb):
    """AUTO is the fp32 instruction below 2^28 multiply-adds and without a workspace, the three-piece form from there on: bit for bit
    what the caller gets who asks for that form.  On the fp32 instruction an infinite operand gives an infinity, and one above the
    largest bf16 number stays finite."""
    torch, B = env["torch"], env["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5 + tb)

    def run(form, M, N, K, A, W, with_ws):
        wsb = B.gemm_workspace_bytes(0, M, N, K) if with_ws else 0
        ws = torch.empty(max(wsb, 256), dtype=torch.uint8, device="cuda")
        Cd = torch.zeros(M, N, device="cuda")
        B.gemm(0, tb, M, N, K, A, K, W, K if tb else N, Cd, N, B.F32, ws=ws if with_ws else None, ws_bytes=wsb, f32_product=form)
        torch.cuda.synchronize()
        return Cd

    for M, N, K in [(21557, 64, 8), (4096, 256, 200), (8000, 128, 250), (200, 60, 602), (32767, 64, 128), (32768, 64, 128), (10875, 41, 602),
                    (10876, 41, 602), (49200, 64, 100), (30000, 300, 40)]:
        say(f"gemm f32 auto form tb={tb} {M}x{N}x{K}")
        below = M * N * K < 2 ** 28
        A = torch.randn(M, K, generator=gen, device="cuda")
        W = torch.rand((N, K) if tb else (K, N), generator=gen, device="cuda") + 0.25
        if below:
            A[0, 0], A[1, 0], A[1, 1:] = float("inf"), 3.4e38, 0.0
            W[0, 0] = 0.5                           # the weight of k = 0 in column 0, either way it is stored
        auto = run(B.F32_PRODUCT_AUTO, M, N, K, A, W, True)
        same = run(B.F32_PRODUCT_NATIVE if below else B.F32_PRODUCT_SPLIT, M, N, K, A, W, True)
        assert torch.equal(auto, same)
        if below:
            assert torch.isinf(auto[0]).all() and float(auto[1, 0]) == float(np.float32(3.4e38) * np.float32(0.5))
        nat = run(B.F32_PRODUCT_NATIVE, M, N, K, A, W, True)
        for form in (B.F32_PRODUCT_AUTO, B.F32_PRODUCT_SPLIT):
            assert torch.equal(run(form, M, N, K, A, W, False), nat), "without a workspace the fp32 instruction runs"


@pytest.mark.parametrize("kind", ["gcn", "sage"])
@pytest.mark.parametrize("n,f_in,f_out,split_fwd", [(3000, 200, 64, False), (20000, 100, 100, True), (12000, 128, 128, True)])
def test_layer_f32_auto_form_is_the_documented_one(env, kind, n, f_in, f_out, split_fwd):
    """A layer's products under AUTO, each below 2^28 multiply-adds: bit for bit those of NATIVE, forward and backward, both orders.
    The two forward products of a GraphSAGE layer in the AGG_FIRST order count as one: above 2^28 together (split_fwd) that launch
    is SPLIT's, and so is nothing else."""
    torch, B = env["torch"], env["B"]
    rng = np.random.default_rng(n)
    n_halo = n // 5
    assert n * 6 // 5 * f_in * f_out < 2 ** 28 and (2 * n * f_in * f_out >= 2 ** 28) == split_fwd
    g = B.Graph(n, n_halo, np.arange(0, 3 * n + 1, 3, dtype=np.int64), rng.integers(0, n + n_halo, 3 * n).astype(np.int32),
                rng.uniform(0.2, 0.5, n).astype(np.float32), rng.uniform(0.5, 1.5, n + n_halo).astype(np.float32))
    sage = kind == "sage"
    x = torch.randn(n + n_halo, f_in, device="cuda")
    w, w_self = (torch.randn(f_in, f_out, device="cuda") / 8 for _ in range(2))
    dh0 = torch.randn(n, f_out, device="cuda")
    bias = torch.randn(f_out, device="cuda")

    def run(order, form):
        l = B.make_layer(B.SAGE_MEAN if sage else B.GCN, f_in, f_out, B.ACT_NONE, B.F32, w, w_self if sage else None, bias, order, f32_product=form)
        size = B.layer_workspace_bytes(g, l)
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        saved = torch.empty(max(B.layer_saved_bytes(g, l), 256), dtype=torch.uint8, device="cuda")
        out = dict(h=torch.zeros(n, f_out, device="cuda"))
        B.layer_fwd(g, l, x, f_in, out["h"], f_out, saved, ws, size)
        for halo in (0, 1):
            dh = dh0.clone()
            dw, ds, db = torch.zeros(f_in, f_out, device="cuda"), torch.zeros(f_in, f_out, device="cuda"), torch.zeros(f_out, device="cuda")
            dx = torch.zeros(n + n_halo if halo else n, f_in, device="cuda")
            B.layer_bwd(g, l, x, f_in, out["h"], f_out, saved, dh, f_out, dw, ds if sage else None, db, dx, f_in, halo, ws, size)
            out.update({f"dw{halo}": dw, f"ds{halo}": ds, f"db{halo}": db, f"dx{halo}": dx})
        torch.cuda.synchronize()
        return out

    for order in (B.AGG_FIRST, B.XFORM_FIRST):
        say(f"layer auto form {kind} n={n} {f_in}-{f_out} order={order}")
        auto, nat, spl = (run(order, f) for f in (B.F32_PRODUCT_AUTO, B.F32_PRODUCT_NATIVE, B.F32_PRODUCT_SPLIT))
        for k in auto:
            as_split = k == "h" and sage and order == B.AGG_FIRST and split_fwd
            assert torch.equal(auto[k], (spl if as_split else nat)[k]), (order, k)
    g.close()


def sage_layer(env, dtype, form, n=2500, f_in=100, f_out=72, order=None, dw_is_self=False):
    """One GraphSAGE layer without halo, forward and backward, on inputs made from a fixed seed: every output."""
    torch, B = env["torch"], env["B"]
    rng = np.random.default_rng(3)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    dt, code = (torch.bfloat16, B.BF16) if dtype == "bf16" else (torch.float32, B.F32)
    mk = lambda *s: torch.randn(*s, generator=gen, device="cuda").to(dt)  # noqa: E731
    g = B.Graph(n, 0, np.arange(0, 5 * n + 1, 5, dtype=np.int64), rng.integers(0, n, 5 * n).astype(np.int32), np.full(n, 0.2, np.float32), None)
    pad = lambda x: torch.nn.functional.pad(x, (0, -x.shape[1] % 8)).contiguous()  # noqa: E731
    x, dh, w, w_self = pad(mk(n, f_in)), pad(mk(n, f_out)), mk(f_in, f_out), mk(f_in, f_out)
    l = B.make_layer(B.SAGE_MEAN, f_in, f_out, B.ACT_RELU, code, w, w_self, None, order or B.AGG_FIRST, f32_product=form)
    size = B.layer_workspace_bytes(g, l)
    ws, saved = torch.empty(size, dtype=torch.uint8, device="cuda"), torch.empty(B.layer_saved_bytes(g, l) + 256, dtype=torch.uint8, device="cuda")
    h, dx = torch.zeros_like(dh), torch.zeros_like(x)
    dw, ds, db = torch.zeros(f_in, f_out, device="cuda"), torch.zeros(f_in, f_out, device="cuda"), torch.zeros(f_out, device="cuda")
    B.layer_fwd(g, l, x, x.shape[1], h, h.shape[1], saved, ws, size)
    h0 = h.clone()
    B.layer_bwd(g, l, x, x.shape[1], h, h.shape[1], saved, dh, dh.shape[1], ds if dw_is_self else dw, ds, db, dx, x.shape[1], 0, ws, size)
    torch.cuda.synchronize()
    g.close()
    return dict(h=h0, dw=dw, dw_self=ds, db=db, dx=dx)


@pytest.mark.parametrize("order", [1, 2])
def test_bf16_products_do_not_depend_on_the_fp32_form(env, order):
    """f32_product says how products of fp32 operands are formed: bf16 results are the same bits for every value, of a single product
    in each orientation (below and above the sizes that the small kernel takes) and of a layer's products in pairs."""
    torch, B = env["torch"], env["B"]
    forms = (B.F32_PRODUCT_AUTO, B.F32_PRODUCT_NATIVE, B.F32_PRODUCT_SPLIT)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(order)
    for ta, tb, M, N, K in [(1, 0, 100, 64, 4000), (1, 1, 72, 130, 2000), (0, 0, 3000, 64, 100), (0, 1, 500, 300, 72), (1, 0, 512, 256, 16000)]:
        A = torch.randn(*((K, M) if ta else (M, K)), generator=gen, device="cuda").bfloat16()
        W = torch.randn(*((N, K) if tb else (K, N)), generator=gen, device="cuda").bfloat16()
        wsb = B.gemm_workspace_bytes(ta, M, N, K)
        ws = torch.empty(max(wsb, 256), dtype=torch.uint8, device="cuda")
        out = []
        for form in forms:
            say(f"bf16 product ta={ta} tb={tb} {M}x{N}x{K} form={form}")
            out.append(torch.zeros(M, N, device="cuda"))
            B.gemm(ta, tb, M, N, K, A, A.shape[1], W, W.shape[1], out[-1], N, B.BF16, out_f32=1, ws=ws, ws_bytes=wsb, f32_product=form)
        torch.cuda.synchronize()
        assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
    say(f"bf16 layer order={order}")
    a, b, c = (sage_layer(env, "bf16", f, order=order) for f in forms)
    for k in a:
        assert torch.equal(a[k], b[k]) and torch.equal(a[k], c[k]), k


@pytest.mark.parametrize("n,f_in,f_out", [(30017, 47, 100), (30016, 100, 256), (30001, 64, 130), (50017, 100, 47), (30000, 130, 72)])
def test_layer_sum_of_two_split_products(env, n, f_in, f_out):
    """The two forward products of a GraphSAGE layer in one launch, columns of the two operands meeting inside, at and beyond the 128 k of
    a wave: within 2e-6 of the fp32 instruction's (2-norm; each form lies within 4e-7 of fp64 at these widths)."""
    spl, nat = (sage_layer(env, "f32", f, n=n, f_in=f_in, f_out=f_out)["h"].double() for f in (env["B"].F32_PRODUCT_SPLIT, env["B"].F32_PRODUCT_NATIVE))
    assert float((spl - nat).norm()) <= 2e-6 * float(nat.norm())


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("order", [1, 2])
def test_layer_refuses_an_unknown_fp32_form(env, dtype, order):
    """Forward and backward of a GraphSAGE layer, whose products run in pairs: any other value of f32_product is CAPGNN_EINVAL."""
    torch, B = env["torch"], env["B"]
    n, f = 300, 40
    g = B.Graph(n, 0, np.arange(n + 1, dtype=np.int64), np.arange(n, dtype=np.int32), np.ones(n, np.float32), None)
    dt, code = (torch.bfloat16, B.BF16) if dtype == "bf16" else (torch.float32, B.F32)
    x, w, dw = (torch.zeros(n, f, device="cuda", dtype=t) for t in (dt, dt, torch.float32))
    for form in (-1, 3, 7):
        l = B.make_layer(B.SAGE_MEAN, f, f, B.ACT_NONE, code, w, w, None, order, f32_product=form)
        size = B.layer_workspace_bytes(g, l)
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        for call in (lambda: B.layer_fwd(g, l, x, f, x.clone(), f, ws.clone(), ws, size),
                     lambda: B.layer_bwd(g, l, x, f, x.clone(), f, ws.clone(), x.clone(), f, dw, dw.clone(), None, x.clone(), f, 0, ws, size)):
            say(f"unknown form {form} {dtype} order={order}")
            with pytest.raises(B.CapgnnError) as e:
                call()
            torch.cuda.synchronize()
            assert e.value.code == B.EINVAL
    g.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [300, 6000])
def test_layer_bwd_with_one_buffer_for_both_weight_gradients(env, dtype, n):
    """dW == dW_self: the self gradient is written last, as by two calls one after the other (with one and with several reduction
    splits); everything else as with two buffers."""
    torch, B = env["torch"], env["B"]
    for order in (B.AGG_FIRST, B.XFORM_FIRST):
        say(f"one weight gradient buffer {dtype} n={n} order={order}")
        two, one = (sage_layer(env, dtype, 0, n=n, order=order, dw_is_self=s) for s in (False, True))
        rel = (one["dw_self"].double() - two["dw_self"].double()).norm() / two["dw_self"].double().norm()
        other = (two["dw"].double() - two["dw_self"].double()).norm() / two["dw_self"].double().norm()
        assert rel <= 1e-5 < other       # fp32 sums of n products, possibly split another way
        for k in ("h", "db", "dx"):
            assert torch.equal(one[k], two[k]), k


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("n,f_in,f_out", [(50_000, 40, 60), (17_000, 150, 130), (50_000, 61, 37), (60_001, 100, 47), (30_017, 200, 121), (70_001, 100, 256),
                                          (66_001, 125, 47)])
def test_sage_layer_products_over_two_weight_matrices(env, order, n, f_in, f_out):
    """The sum of a GraphSAGE layer's two products as one launch over both weight matrices, in tiles 64 and 128 columns wide and with the
    weights in registers (more than 768 tiles of 64 x 64): the forward product of the AGG_FIRST order and the input gradient of
    XFORM_FIRST, with widths that fill their last step of 32, their last group of four columns, and that do not.  Self loops only, so both products read the layer's input itself.  Distance from float64
    no more than four times that of the fp32 instruction plus 2^-23 (see test_gemm_f32_split_product)."""
    torch, B = env["torch"], env["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + f_in)
    mk = lambda *s: torch.randn(*s, generator=gen, device="cuda")  # noqa: E731
    assert (n + 63) // 64 * ((min(f_in, f_out) + 63) // 64) > 768
    g = B.Graph(n, 0, np.arange(n + 1, dtype=np.int64), np.arange(n, dtype=np.int32), np.ones(n, np.float32), None)
    x, dh, w, w_self, bias = mk(n, f_in), mk(n, f_out), mk(f_in, f_out), mk(f_in, f_out), mk(f_out)
    ref = dict(h=x.double() @ (w.double() + w_self.double()) + bias.double(), dx=dh.double() @ (w.double() + w_self.double()).T)
    err = {}
    for form in (B.F32_PRODUCT_NATIVE, B.F32_PRODUCT_SPLIT):
        l = B.make_layer(B.SAGE_MEAN, f_in, f_out, B.ACT_NONE, B.F32, w, w_self, bias, order, f32_product=form)
        size = B.layer_workspace_bytes(g, l)
        ws, saved = torch.empty(size, dtype=torch.uint8, device="cuda"), torch.empty(B.layer_saved_bytes(g, l) + 256, dtype=torch.uint8, device="cuda")
        out = dict(h=torch.zeros(n, f_out, device="cuda"), dx=torch.zeros(n, f_in, device="cuda"))
        B.layer_fwd(g, l, x, f_in, out["h"], f_out, saved, ws, size)
        B.layer_bwd(g, l, x, f_in, out["h"], f_out, saved, dh.clone(), f_out, None, None, None, out["dx"], f_in, 0, ws, size)
        torch.cuda.synchronize()
        for k in out:
            err[k, form] = ((out[k].double() - ref[k]).abs().max() / ref[k].abs().max()).item()
    say(f"two weight matrices n={n} {f_in}-{f_out} order={order}: {err}")
    for k in ("h", "dx"):
        assert err[k, B.F32_PRODUCT_SPLIT] <= 4.0 * err[k, B.F32_PRODUCT_NATIVE] + 2.0 ** -23 and err[k, B.F32_PRODUCT_NATIVE] <= TOL_F32
    g.close()


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("n,f_in,f_out", [(37, 40, 30), (1003, 100, 64), (3001, 130, 200), (6400, 64, 128), (12_800, 96, 64), (12_801, 96, 64), (33_001, 64, 72)])
def test_bf16_sage_layer_rounds_as_two_launches_exact(env, order, n, f_in, f_out):
    """A bf16 GraphSAGE layer stores its self product, rounded, and adds the neighbour product to what it stored, at every number of rows: in the
    AGG_FIRST order forward, in XFORM_FIRST backward; the other direction rounds both terms and adds in the aggregation.  Small integers, whose
    sums are exact in float (below 2^24) and whose stored values are not in bf16 (beyond 2^8): equality with the same roundings."""
    torch, B = env["torch"], env["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + f_in + order)
    mk = lambda r, c: torch.randint(-8, 9, (r, c), generator=gen, device="cuda").double()  # noqa: E731
    rne = lambda t: t.float().bfloat16().double()  # noqa: E731
    bf = lambda t: torch.nn.functional.pad(t.bfloat16(), (0, -t.shape[1] % 8)).contiguous()  # noqa: E731
    col = torch.randint(0, n, (n,), generator=gen, device="cuda")
    g = B.Graph(n, 0, np.arange(0, n + 1, dtype=np.int64), col.int().cpu().numpy(), np.ones(n, np.float32), np.ones(n, np.float32))
    x, dh, w, w_self, bias = mk(n, f_in), mk(n, f_out), mk(f_in, f_out), mk(f_in, f_out), mk(1, f_out)[0]
    summed = lambda t: torch.zeros_like(t).index_add_(0, col, t)  # noqa: E731
    if order == B.AGG_FIRST:
        h = rne(x[col] @ w + rne(x @ w_self) + bias)
        dx = rne(summed(rne(dh @ w.T)) + rne(dh @ w_self.T))
        dw = x[col].T @ dh
    else:
        back = summed(dh)                    # (a few terms of at most 8: bf16 holds it)
        h = rne(rne(x @ w)[col] + rne(x @ w_self) + bias)
        dx = rne(back @ w.T + rne(dh @ w_self.T))
        dw = x.T @ back
    assert n < 1000 or not torch.equal(h, rne((x[col] @ w) + x @ w_self + bias))
    xb, db, wb, wb_self, bias = bf(x), bf(dh), w.bfloat16(), w_self.bfloat16(), bias.float()       # (the layer keeps pointers)
    l = B.make_layer(B.SAGE_MEAN, f_in, f_out, B.ACT_NONE, B.BF16, wb, wb_self, bias, order)
    ldi, ldo = xb.shape[1], db.shape[1]
    size = B.layer_workspace_bytes(g, l)
    ws, saved = torch.empty(size, dtype=torch.uint8, device="cuda"), torch.empty(B.layer_saved_bytes(g, l) + 256, dtype=torch.uint8, device="cuda")
    hd, dxd = torch.zeros(n, ldo, dtype=torch.bfloat16, device="cuda"), torch.zeros(n, ldi, dtype=torch.bfloat16, device="cuda")
    dwd, dwsd, dbd = torch.zeros(f_in, f_out, device="cuda"), torch.zeros(f_in, f_out, device="cuda"), torch.zeros(f_out, device="cuda")
    say(f"bf16 GraphSAGE layer's roundings order={order} n={n} {f_in}-{f_out}")
    B.layer_fwd(g, l, xb, ldi, hd, ldo, saved, ws, size)
    B.layer_bwd(g, l, xb, ldi, hd, ldo, saved, db.clone(), ldo, dwd, dwsd, dbd, dxd, ldi, 0, ws, size)
    torch.cuda.synchronize()
    assert torch.equal(hd[:, :f_out].double(), h) and torch.equal(dxd[:, :f_in].double(), dx)
    assert torch.equal(dwd.double(), dw) and torch.equal(dwsd.double(), x.T @ dh) and torch.equal(dbd.double(), dh.sum(0))
    g.close()


@pytest.mark.parametrize("n,f_in,f_out", [(60_001, 47, 100), (30_017, 100, 128), (66_001, 125, 100), (30_017, 130, 300), (20_011, 200, 256), (9001, 40, 30)])
def test_layer_input_gradient_with_scaled_rows(env, n, f_in, f_out):
    """The input gradient of a GCN layer in the AGG_FIRST order, whose product dZ W^T multiplies each row by its scale: in tiles of 64 and 128
    columns, with the weights in registers (whole and ragged groups of columns) and small.  One entry per row.  Distance from float64 no
    more than four times that of the fp32 instruction plus 2^-23 (see test_gemm_f32_split_product)."""
    torch, B = env["torch"], env["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + f_in)
    mk = lambda *s: torch.randn(*s, generator=gen, device="cuda")  # noqa: E731
    rng = np.random.default_rng(n)
    col, r, c = rng.permutation(n).astype(np.int32), rng.uniform(0.5, 2, n).astype(np.float32), rng.uniform(0.5, 2, n).astype(np.float32)
    g = B.Graph(n, 0, np.arange(n + 1, dtype=np.int64), col, r, c)
    pad = lambda x: torch.nn.functional.pad(x, (0, -x.shape[1] % 4)).contiguous()  # noqa: E731
    x, dh, w = pad(mk(n, f_in)), pad(mk(n, f_out)), mk(f_in, f_out)
    at, rd, cd = (torch.from_numpy(v).cuda() for v in (col.astype(np.int64), r, c))
    ref = torch.zeros(n, f_in, dtype=torch.float64, device="cuda")
    ref[at] = (dh[:, :f_out].double() @ w.double().T) * rd.double()[:, None] * cd.double()[at][:, None]
    err = {}
    for form in (B.F32_PRODUCT_NATIVE, B.F32_PRODUCT_SPLIT):
        l = B.make_layer(B.GCN, f_in, f_out, B.ACT_NONE, B.F32, w, None, None, B.AGG_FIRST, f32_product=form)
        size = B.layer_workspace_bytes(g, l)
        ws, saved = torch.empty(size, dtype=torch.uint8, device="cuda"), torch.empty(B.layer_saved_bytes(g, l) + 256, dtype=torch.uint8, device="cuda")
        h, dx = torch.zeros_like(dh), torch.zeros_like(x)
        say(f"layer input gradient with scaled rows {n} {f_in}-{f_out} form={form}")
        B.layer_fwd(g, l, x, x.shape[1], h, h.shape[1], saved, ws, size)
        B.layer_bwd(g, l, x, x.shape[1], h, h.shape[1], saved, dh.clone(), dh.shape[1], None, None, None, dx, dx.shape[1], 0, ws, size)
        torch.cuda.synchronize()
        err[form] = ((dx[:, :f_in].double() - ref).abs().max() / ref.abs().max()).item()
    assert err[B.F32_PRODUCT_SPLIT] <= 4.0 * err[B.F32_PRODUCT_NATIVE] + 2.0 ** -23 and err[B.F32_PRODUCT_NATIVE] <= TOL_F32
    g.close()


def test_mfma_peak_loop_runs_and_counts_its_work(env):
    """The register-resident matrix-instruction loop: the reported work is 4 tiles x 4 waves x iterations x workgroups x
    the instruction's 2 * 32 * 32 * k FLOPs, and every thread writes a finite, positive checksum (its operands are
    positive)."""
    torch, B = env["torch"], env["B"]
    wgs, iters = 8, 16
    out = torch.full((wgs * 256,), -1.0, dtype=torch.float32, device="cuda")
    for dt, k in ((B.F32, 2), (B.BF16, 16)):
        flop = B.mfma_peak(dt, wgs, iters, out)
        torch.cuda.synchronize()
        assert flop == 2.0 * 32 * 32 * k * 4 * iters * 4 * wgs
        got = out.cpu().numpy()
        assert np.isfinite(got).all() and (got > 0).all()
    with pytest.raises(B.CapgnnError):
        B.mfma_peak(B.F32, 0, iters, out)


def test_gemm_relu_mask_epilogue(env):
    torch, B, H, O, orc = env["torch"], env["B"], env["H"], env["O"], env["orc"]
    rng = np.random.default_rng(3)
    M, N, K = 333, 70, 50
    A, Bm = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    mask = rng.standard_normal((M, N)).astype(np.float32)
    mask[0, :5] = 0.0
    Cd = torch.zeros((M, N), device="cuda")
    B.gemm(0, 1, M, N, K, H.np_to_dev(A), K, H.np_to_dev(Bm), K, Cd, N, B.F32, relu_mask=H.np_to_dev(mask), ldm=N)
    torch.cuda.synchronize()
    ref = orc.matmul(A, Bm, tb=True) * (mask > 0)
    assert O.normwise(Cd.cpu().numpy(), ref) <= TOL_F32


# ----------------------------------------------------------------------------- loss
@pytest.mark.parametrize("C", [1, 8, 41, 47, 100, 300])
def test_softmax_ce_vs_oracle(env, C):
    torch, B, H, O, orc = env["torch"], env["B"], env["H"], env["O"], env["orc"]
    rng = np.random.default_rng(C)
    n = 1237
    Z = (rng.standard_normal((n, C)) * 4).astype(np.float32)
    y = rng.integers(0, C, n).astype(np.int32)
    mask = (rng.random(n) < 0.6).astype(np.uint8)
    ws_b = B.loss_workspace_bytes(n)
    ws = torch.empty(ws_b, dtype=torch.uint8, device="cuda")
    for m, norm in ((mask, 0.0), (None, 0.0), (mask, 777.0)):
        loss_d = torch.zeros(1, device="cuda")
        dZ = torch.full((n, C + 2), 9.0, device="cuda")
        B.softmax_ce(n, C, H.np_to_dev(Z), C, H.np_to_dev(y), None if m is None else H.np_to_dev(m), norm, loss_d, dZ,
                     C + 2, B.F32, ws, ws_b)
        torch.cuda.synchronize()
        ref_loss, ref_dZ = orc.softmax_ce(Z.astype(np.float64), y, m, norm)
        assert abs(float(loss_d.item()) - ref_loss) <= 1e-5 * max(1.0, abs(ref_loss))
        got = dZ.cpu().numpy()
        assert O.normwise(got[:, :C], ref_dZ) <= TOL_F32
        assert (got[:, C:] == 9.0).all()
