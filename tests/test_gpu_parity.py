"""GPU parity: the HIP path, called through the C ABI, against the fp64 oracle on the same
seeded inputs.  Index sets, routes and permutations bit-exact; outputs within max-abs
1e-5 (fp32) and 2e-2 (bf16, unit-variance inputs)."""
import sys

import numpy as np
import pytest
import torch

import paper_2505_18809_amd as vorta
from oracle import vorta_oracle as vo
from synth_inputs import LayerConfig, get_config, make_qkv, make_routes
from helpers import PIPE, PIPE_SPLIT_WIN, PIPE_WIN_128, SPLIT2, SPLIT4, f64, force_form, spec_of

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-5, "bf16": 2e-2}
DEV = "cuda"


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def bf16_round(x: np.ndarray) -> np.ndarray:
    return torch.from_numpy(np.asarray(x, dtype=np.float64)).to(torch.bfloat16).double().numpy()


def small_cfg(name, grid, heads, dtype, tile, window, routes, d=128, n_text=0, seed=11, **kw):
    return LayerConfig(name, grid, heads, d, dtype, tile, window, seed=seed, n_text=n_text,
                       fixed_routes=tuple(routes), **kw)


def run_layer(cfg, q, k, v, routes, layout=1, **plan_over):
    plan = vorta.plan_for(cfg, layout=layout, **plan_over)
    out = vorta.vorta_routed_attention_layer(plan, q, k, v, routes)
    torch.cuda.synchronize()
    return plan, out


def hnd(t, layout):
    return t if layout == 1 else t.transpose(0, 1)


# ------------------------------------------------------------------ memory passes --------

@pytest.mark.parametrize("layout", [1, 0])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("fp32", 64), ("fp32", 128)])
def test_reorder_to_tiles_and_back_is_the_tile_permutation(dtype, d, layout):
    cfg = small_cfg("reorder", (4, 6, 8), 5, dtype, (2, 3, 4), (3, 3, 3), [1, 0, 1, 2, 1], d=d, n_text=7)
    say(f"reorder {dtype} d={d} layout={layout}")
    q, _, _ = make_qkv(cfg, DEV, layout)
    plan = vorta.plan_for(cfg, layout=layout)
    routes = np.array(cfg.fixed_routes, dtype=np.uint8)
    tiled = vorta.vorta_reorder_to_tiles(plan, q, routes)
    torch.cuda.synchronize()
    perm = torch.from_numpy(vorta.vorta_tile_permutation(plan).astype(np.int64)).to(DEV)
    L = cfg.n_video
    src = hnd(q, layout)
    for slot, h in enumerate([0, 2, 4]):
        want = torch.empty_like(src[h])
        want[perm] = src[h][:L]
        want[L:] = src[h][L:]
        assert torch.equal(tiled[slot], want), (slot, h)
    back = torch.full_like(q, 7.0)
    vorta.vorta_reorder_from_tiles(plan, tiled, routes, back)
    torch.cuda.synchronize()
    b = hnd(back, layout)
    for h in range(5):
        if routes[h] == 1:
            assert torch.equal(b[h], src[h])
        else:
            assert (b[h] == 7.0).all()          # other heads' rows are not touched


@pytest.mark.parametrize("name,grid,bucket,num,den,dtype,d", [
    ("even", (4, 6, 8), (2, 3, 2), 1, 2, "bf16", 128),
    ("ragged", (5, 7, 9), (2, 3, 2), 1, 2, "bf16", 128),
    ("quarter", (4, 8, 8), (2, 2, 4), 1, 4, "bf16", 128),
    ("keepall", (3, 4, 5), (2, 3, 2), 1, 1, "bf16", 128),
    ("fp32", (4, 8, 8), (2, 3, 2), 1, 2, "fp32", 64),
    ("fp32d128", (3, 5, 4), (3, 2, 2), 2, 3, "fp32", 128),
])
def test_bcs_index_pool_and_unpool_match_oracle(name, grid, bucket, num, den, dtype, d):
    cfg = small_cfg(name, grid, 3, dtype, (1, 1, 1), (1, 1, 1), [2, 0, 2], d=d, n_text=3, bucket=bucket,
                    keep_num=num, keep_den=den)
    say(f"bcs {name}")
    q, k, v = make_qkv(cfg, DEV)
    plan = vorta.plan_for(cfg)
    routes = np.array(cfg.fixed_routes, dtype=np.uint8)
    keep_idx, assign = vorta.vorta_bcs_build_index(plan, k, routes)
    pooled = vorta.vorta_bcs_pool(plan, v, routes, keep_idx, assign)
    torch.cuda.synchronize()
    L = cfg.n_video
    for slot, h in enumerate([0, 2]):
        ki, asg, gap = vo.bcs_select(f64(k[h])[:L], grid, bucket, num, den)
        assert gap > 1e-9, "tie-proof input expected"
        assert np.array_equal(keep_idx[slot].cpu().numpy(), ki)
        assert np.array_equal(assign[slot].cpu().numpy(), asg)
        want = np.concatenate([vo.bcs_pool(f64(v[h])[:L], ki, asg), f64(v[h])[L:]])
        got = f64(pooled[slot])
        if dtype == "bf16":
            assert np.abs(got - want).max() <= 2.0 ** -8 * max(1.0, np.abs(want).max())
            single = np.bincount(asg, minlength=len(ki)) == 1
            assert np.array_equal(got[:len(ki)][single], want[:len(ki)][single])     # kept rows are copies
        else:
            assert np.abs(got - want).max() < 1e-6
    # unpool: every token reads its slot, text rows their own
    o_c = torch.randn(2, plan.n_core_tokens, d, device=DEV).to(q.dtype)
    out = torch.zeros_like(q)
    vorta.vorta_scatter_back(plan, routes, None, o_c, assign, out)
    torch.cuda.synchronize()
    for slot, h in enumerate([0, 2]):
        src = torch.cat([assign[slot].long(), plan.n_core + torch.arange(3, device=DEV)])
        assert torch.equal(out[h], o_c[slot][src])
    assert (out[1] == 0).all()


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("fp32", 64)])
@pytest.mark.parametrize("grid", [(4, 6, 8), (5, 7, 9)])
@pytest.mark.parametrize("bucket", [(2, 1, 1), (1, 2, 1), (1, 1, 2)])
def test_two_token_buckets_are_average_pooling(bucket, grid, dtype, d):
    """The ablation's average-pooling variants (section 4.3) are the core-set route with a bucket
    of two at ratio 1/2.  Which of the two tokens is the centre is a tie, so a slot's index may be
    either; what is unique -- the slot every token reads, the pooled rows, the layer's output --
    is held to the oracle.  On the odd grid the last bucket of the axis is a single token."""
    cfg = small_cfg("avgpool", grid, 3, dtype, (1, 1, 1), (1, 1, 1), [2, 0, 2], d=d, n_text=5, bucket=bucket)
    say(f"average pooling {bucket} on {grid} {dtype}")
    q, k, v = make_qkv(cfg, DEV)
    plan = vorta.plan_for(cfg)
    routes = np.array(cfg.fixed_routes, dtype=np.uint8)
    keep_idx, assign = vorta.vorta_bcs_build_index(plan, k, routes)
    pooled = vorta.vorta_bcs_pool(plan, v, routes, keep_idx, assign)
    torch.cuda.synchronize()
    L = cfg.n_video
    for slot, h in enumerate([0, 2]):
        ki, asg, _ = vo.bcs_select(f64(k[h])[:L], grid, bucket, 1, 2)
        got_ki, got_asg = keep_idx[slot].cpu().numpy(), assign[slot].cpu().numpy()
        assert np.array_equal(got_asg, asg)
        assert np.array_equal(got_asg[got_ki], np.arange(len(ki)))           # a slot's index is one of its tokens
        want = np.concatenate([vo.bcs_pool(f64(v[h])[:L], ki, asg), f64(v[h])[L:]])
        tol = 2.0 ** -8 * max(1.0, np.abs(want).max()) if dtype == "bf16" else 1e-6
        assert np.abs(f64(pooled[slot]) - want).max() <= tol
    check_layer(cfg, cfg.fixed_routes)


# ------------------------------------------------------------------ whole layer ----------

def check_layer(cfg, routes, layout=1, rows=None, **plan_over):
    q, k, v = make_qkv(cfg, DEV, layout)
    plan, out = run_layer(cfg, q, k, v, routes, layout, **plan_over)
    over = {}
    if "center_mode" in plan_over:
        over["center_mode"] = ("clamp", "identity", "block")[plan_over["center_mode"]]
    spec = spec_of(cfg, **over)
    qh, kh, vh, oh = (hnd(t, layout) for t in (q, k, v, out))
    worst = 0.0
    for h, r in enumerate(routes):
        want = vo.head_attention(int(r), f64(qh[h]), f64(kh[h]), f64(vh[h]), spec, rows)
        got = f64(oh[h]) if rows is None else f64(oh[h][torch.as_tensor(rows, device=DEV)])
        err = np.abs(got - want).max()
        worst = max(worst, err)
        assert err <= TOL[cfg.dtype], f"{cfg.name} head {h} route {r}: max-abs {err:.3e}"
    say(f"{cfg.name} layout={layout} routes={list(map(int, routes))}: max-abs {worst:.3e}")
    return plan, out


@pytest.mark.parametrize("route", [0, 1, 2])
def test_tiny_config_every_head_under_every_route(route):
    cfg = get_config("tiny")
    check_layer(cfg, [route] * cfg.heads)


@pytest.mark.parametrize("layout", [1, 0])
def test_single_layer_config(layout):
    cfg = get_config("single")
    check_layer(cfg, make_routes(cfg).numpy(), layout)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("fp32", 64), ("fp32", 128)])
def test_ragged_shapes_text_tokens_and_mixed_routes(dtype, d):
    # N = 5*6*9 + 37 = 307: not a multiple of any block size; 90-token tiles; clipped buckets
    cfg = small_cfg("ragged", (5, 6, 9), 4, dtype, (5, 2, 3), (1, 3, 3), [2, 1, 0, 1], d=d, n_text=37)
    check_layer(cfg, cfg.fixed_routes)
    check_layer(cfg, cfg.fixed_routes, layout=0)


@pytest.mark.parametrize("seed", range(64))
def test_seeded_random_small_layers(seed):
    """Shapes drawn from a seed: grids that make ragged last blocks, one- and many-run windows,
    run lists crossing 64-key blocks, tiles above and below a query block, text tokens or none,
    both layouts, every route mix -- each head against the oracle on all rows."""
    rng = np.random.default_rng(1000 + seed)
    big = seed % 3 == 2                     # tiles of more than 128 tokens (layers this small run on the split kernel)
    tile = tuple(int(rng.integers(4, 8)) for _ in range(3)) if big else tuple(int(rng.integers(1, 5)) for _ in range(3))
    reps = tuple(int(rng.integers(1, 4 if big else 5)) for _ in range(3))
    grid = tuple(t * r for t, r in zip(tile, reps))
    window = tuple(int(rng.choice([1, 3, 5])) for _ in range(3))
    heads = int(rng.integers(1, 6))
    routes = [int(r) for r in rng.integers(0, 3, heads)]
    n_text = int(rng.choice([0, 0, 5, 70]))
    # fp32: the exact path (fp64 inside) and the reorder passes
    dtype, d = (("fp32", 64) if seed % 4 == 3 else ("bf16", 128))
    cfg = small_cfg(f"rand{seed}", grid, heads, dtype, tile, window, routes, d=d, n_text=n_text, seed=50 + seed,
                    bucket=tuple(int(b) for b in rng.choice([1, 2, 3], 3)))
    say(f"seed {seed}: grid {grid} tile {tile} window {window} text {n_text} routes {routes} bucket {cfg.bucket}")
    check_layer(cfg, routes, layout=int(rng.integers(0, 2)), center_mode=int(rng.integers(0, 2)) if seed < 44 else 2)


@pytest.mark.parametrize("dtype,d", [("fp32", 64), ("fp32", 128)])
def test_fp32_path_holds_its_tolerance_over_thousands_of_keys(dtype, d):
    """The fp32 path computes in fp64 between its fp32 inputs and outputs, so its 1e-5 bar does
    not depend on the number of keys: 3,072 video + 50 text tokens (the Single layer's grid),
    one head per route, sampled rows."""
    cfg = small_cfg("fp32_3k", (12, 16, 16), 3, dtype, (4, 4, 4), (3, 3, 3), [0, 1, 2], d=d, n_text=50, seed=37)
    rows = np.unique(np.concatenate([np.arange(1, cfg.n_video, 13), np.arange(cfg.n_video, cfg.n_tokens)]))
    check_layer(cfg, cfg.fixed_routes, rows=rows)


@pytest.mark.parametrize("tile,bucket", [((2, 99, 4), (2, 3, 2)), ((50, 50, 50), (9, 2, 2)), ((3, 4, 70000), (2, 3, 99))])
def test_tiles_and_buckets_that_exceed_the_grid(tile, bucket):
    """A tile or bucket extent beyond its axis is the whole axis: (2,99,4) on a 4x6x8 grid is a
    (2,6,4) tile, (50,50,50) one tile of all 192 tokens (more than one 128-row query block).
    The oracle gets the extents as given -- integer division by an oversized tile is tile 0."""
    cfg = small_cfg("over", (4, 6, 8), 4, "bf16", tile, (3, 1, 3), [1, 2, 0, 1], n_text=4, seed=29, bucket=bucket)
    check_layer(cfg, cfg.fixed_routes)


@pytest.mark.parametrize("n_text,layout", [(300, 1), (515, 0)])
def test_text_rows_spanning_several_query_blocks(n_text, layout):
    """Text rows of a window head attend to every row and run as items of their own, next to those of the
    dense heads: more text rows than an item holds (64 on the split kernel, which layers this small run on),
    and a ragged last item.  (256-row items and half-row items of text rows: test_gpu_attention_forms.py.)"""
    cfg = small_cfg(f"text{n_text}", (4, 6, 8), 4, "bf16", (2, 3, 4), (3, 3, 3), [1, 0, 2, 1], n_text=n_text, seed=31)
    check_layer(cfg, cfg.fixed_routes, layout=layout)


@pytest.mark.parametrize("grid,tile,dtype", [((5, 7, 6), (2, 3, 4), "bf16"), ((5, 7, 6), (2, 3, 4), "fp32"),
                                             ((7, 10, 13), (3, 4, 5), "bf16"), ((9, 11, 14), (4, 6, 8), "bf16"),
                                             ((3, 5, 5), (4, 2, 6), "bf16"), ((10, 12, 9), (6, 9, 8), "bf16")])
@pytest.mark.parametrize("layout", [1, 0])
def test_layers_whose_tiles_do_not_divide_the_grid(grid, tile, dtype, layout):
    """Edge tiles clipped to the grid: ragged tile sizes in the tile order, in the run lists and
    in the work items (a clipped tile can have fewer query blocks than a full one).  Tiles below
    and above 128 tokens, text rows, every route, both centre rules."""
    d = 64 if dtype == "fp32" else 128
    cfg = small_cfg(f"clip{grid}", grid, 5, dtype, tile, (3, 3, 3), [1, 0, 1, 2, 1], d=d, n_text=9, seed=61)
    check_layer(cfg, cfg.fixed_routes, layout=layout)
    check_layer(cfg, cfg.fixed_routes, layout=layout, center_mode=1)
    # the staged path over tile-ordered copies
    if layout == 1 and dtype == "bf16":
        routes = np.array(cfg.fixed_routes, dtype=np.uint8)
        q, k, v = make_qkv(cfg, DEV)
        plan = vorta.plan_for(cfg)
        q_t, k_t, v_t = (vorta.vorta_reorder_to_tiles(plan, t, routes) for t in (q, k, v))
        perm = torch.as_tensor(vorta.vorta_tile_permutation(plan), device=DEV, dtype=torch.long)
        for slot, h in enumerate(np.nonzero(routes == 1)[0]):
            want = torch.empty_like(q[h])
            want[perm] = q[h][: cfg.n_video]
            want[cfg.n_video:] = q[h][cfg.n_video:]
            assert torch.equal(q_t[slot], want)
        o_t, staged = torch.empty_like(q_t), torch.zeros_like(q)
        only_win = np.where(routes == 1, 1, 0).astype(np.uint8)      # window heads; the rest as dense heads
        vorta.vorta_attention_routed(plan, only_win, q=q, k=k, v=v, out=staged, q_t=q_t, k_t=k_t, v_t=v_t, o_t=o_t)
        vorta.vorta_scatter_back(plan, only_win, o_t, None, None, staged)
        torch.cuda.synchronize()
        spec = spec_of(cfg)
        for h in np.nonzero(routes == 1)[0]:
            want = vo.head_attention(1, f64(q[h]), f64(k[h]), f64(v[h]), spec, None)
            err = np.abs(f64(staged[h]) - want).max()
            assert err <= TOL["bf16"], f"staged window head {h}: max-abs {err:.3e}"


@pytest.mark.parametrize("layout", [1, 0])
def test_maximum_head_count(layout):
    """128 heads (the most a plan takes), routes cycling 0, 1, 2: the per-route head lists fill up
    and every head must still read and write its own rows."""
    heads = 128
    routes = [h % 3 for h in range(heads)]
    cfg = small_cfg("heads128", (2, 4, 6), heads, "bf16", (1, 2, 3), (3, 3, 3), routes, n_text=3, seed=77)
    check_layer(cfg, routes, layout=layout)


def test_window_identity_centres_and_wide_windows():
    cfg = small_cfg("ident", (4, 8, 8), 2, "bf16", (2, 2, 2), (1, 3, 5), [1, 1])
    check_layer(cfg, cfg.fixed_routes, center_mode=1)
    check_layer(cfg, cfg.fixed_routes, center_mode=0)


def test_degenerate_cases():
    # one tile, one bucket row, window of one tile, core-set keeping everything
    cfg = small_cfg("one_tile", (1, 2, 3), 3, "bf16", (1, 2, 3), (1, 1, 1), [0, 1, 2])
    check_layer(cfg, cfg.fixed_routes)
    keep = small_cfg("keep_all", (2, 3, 4), 2, "fp32", (1, 1, 1), (1, 1, 1), [2, 0], d=64, keep_num=1, keep_den=1)
    plan, out = check_layer(keep, keep.fixed_routes)
    # no head on some routes; empty route groups must be no-ops
    only_full = small_cfg("only_full", (2, 4, 4), 2, "bf16", (1, 2, 2), (3, 3, 3), [0, 0])
    check_layer(only_full, only_full.fixed_routes)
    # tile larger than a query block: several q-blocks per tile
    big_tile = small_cfg("big_tile", (4, 8, 10), 1, "bf16", (4, 8, 5), (1, 1, 1), [1])
    check_layer(big_tile, big_tile.fixed_routes)


@pytest.mark.parametrize("form", [0, SPLIT2, SPLIT4, PIPE, PIPE_SPLIT_WIN, PIPE_WIN_128])
@pytest.mark.parametrize("tile", [(4, 4, 4), (4, 8, 8)], ids=["tile64", "tile256"])
def test_row_maxima_that_jump_or_creep_late_in_the_key_stream(tile, form):
    """The attention kernels keep a lagging row reference instead of the running maximum.
    Inputs built to move the maxima late: one key far down the key stream that dominates a
    few rows outright, and scores that rise steadily along the key axis for half the rows.
    Window heads get their dominating keys at the end of the row's key set in tile order.  In the form the
    rule chooses (at this size the split kernel) and in every other one; tiles of 64 tokens give the
    pipelined kernels window items of 129 to 256 rows and of at most 128, tiles of 256 the former only."""
    cfg = small_cfg("late_max", (12, 16, 16), 6, "bf16", tile, (3, 3, 3), [0, 0, 2, 2, 1, 1], seed=23)
    q, k, v = make_qkv(cfg, DEV, 1)
    N, d = cfg.n_tokens, cfg.head_dim
    gen = torch.Generator(device="cpu").manual_seed(5)
    u = torch.randn(d, generator=gen)
    u = (u / u.norm()).to(DEV)
    ramp = torch.linspace(0.0, 1.0, N, device=DEV)[:, None]

    def last_window_token(row, back):
        """Token `back` places before the end of the row's key set (tile order = the order the
        window kernels stream keys in; the mask is the oracle's)."""
        keys = np.nonzero(vo.sta_mask_row(row, cfg.grid, cfg.tile, cfg.window))[0]
        order = sorted(keys, key=lambda j: (vo.get_tile_id_3d(int(j), cfg.grid, cfg.tile), j))
        return order[-1 - back]

    for h in range(cfg.heads):
        r = cfg.fixed_routes[h]
        kh = k[h].float()
        # scores creep up (or down) along the keys, by up to 60 / sqrt(d) = 5.3 per unit of <q, u>
        kh = kh + 60.0 * ramp * u[None, :]
        late = ((int(0.45 * N), 100), (int(0.93 * N), 2000), (N - 1, 7))
        if r == 1:
            late = tuple((int(last_window_token(row, back)), row) for back, row in ((0, 100), (5, 2000), (40, 7)))
        for j, row in late:
            kh[j] = (1.5 if r == 2 else 4.0) * q[h, row].float()   # a late key that dominates one row
        k[h] = kh.to(torch.bfloat16)
    routes = np.array(cfg.fixed_routes, dtype=np.uint8)
    out = vorta.vorta_routed_attention_layer(force_form(vorta.plan_for(cfg), form), q, k, v, routes)
    torch.cuda.synchronize()
    spec = spec_of(cfg)
    for h, r in enumerate(routes):
        want = vo.head_attention(int(r), f64(q[h]), f64(k[h]), f64(v[h]), spec, None)
        err = np.abs(f64(out[h]) - want)
        # A row that one key dominates outright returns that key's value row, and with unit-variance
        # V some of its 128 entries exceed 4, where half a bf16 ulp is already 1.6e-2: the 2e-2 bar
        # (derived for |O| of about 2 and less) is held wherever |O| <= 2.5 and widened in
        # proportion beyond, to 2^-7 |O| (output rounding 2^-8 |O| + rounding of P 2^-9 |O|, and margin).
        bar = np.maximum(TOL["bf16"], 2.0 ** -7 * np.abs(want))
        say(f"late_max {tile} head {h} route {r}: max-abs {err.max():.3e} (largest |O| {np.abs(want).max():.2f}, "
            f"entries over 2e-2: {(err > TOL['bf16']).sum()})")
        assert (err <= bar).all(), f"head {h} route {r}: max-abs {err.max():.3e}"
        assert (err > TOL["bf16"]).sum() <= 8                 # and those entries are a handful


def test_layer_equals_the_staged_calls_and_is_deterministic():
    cfg = get_config("single")
    routes = make_routes(cfg).numpy()
    q, k, v = make_qkv(cfg, DEV)
    plan, out = run_layer(cfg, q, k, v, routes)
    out2 = vorta.vorta_routed_attention_layer(plan, q, k, v, routes)
    torch.cuda.synchronize()
    assert torch.equal(out, out2)
    q_t, k_t, v_t = (vorta.vorta_reorder_to_tiles(plan, t, routes) for t in (q, k, v))
    keep_idx, assign = vorta.vorta_bcs_build_index(plan, k, routes)
    q_c, k_c, v_c = (vorta.vorta_bcs_pool(plan, t, routes, keep_idx, assign) for t in (q, k, v))
    o_t, o_c, staged = torch.empty_like(q_t), torch.empty_like(q_c), torch.zeros_like(q)
    vorta.vorta_attention_routed(plan, routes, q=q, k=k, v=v, out=staged, q_t=q_t, k_t=k_t, v_t=v_t, o_t=o_t,
                                 q_c=q_c, k_c=k_c, v_c=v_c, o_c=o_c)
    vorta.vorta_scatter_back(plan, routes, o_t, o_c, assign, staged)
    torch.cuda.synchronize()
    # over tile-ordered copies the text rows of window heads meet their keys in tile order, another order of
    # summation: those heads are held to the oracle, the others are the same launch
    spec = spec_of(cfg)
    for h, r in enumerate(routes):
        if r != 1:
            assert torch.equal(out[h], staged[h]), f"head {h} route {r}"
            continue
        want = vo.head_attention(1, f64(q[h]), f64(k[h]), f64(v[h]), spec, None)
        err = np.abs(f64(staged[h]) - want).max()
        say(f"staged over tile-ordered copies, head {h}: max-abs {err:.3e}")
        assert err <= TOL["bf16"], f"head {h}: max-abs {err:.3e}"
    # the same without tile-ordered copies: the window kernel gathers rows through the tile
    # permutation and writes its rows to their places itself
    direct = torch.zeros_like(q)
    vorta.vorta_attention_routed(plan, routes, q=q, k=k, v=v, out=direct, q_c=q_c, k_c=k_c, v_c=v_c, o_c=o_c)
    vorta.vorta_scatter_back(plan, routes, None, o_c, assign, direct)
    torch.cuda.synchronize()
    assert torch.equal(out, direct)


def test_layer_call_replays_from_a_hip_graph():
    """The layer call is plain kernel launches on the caller's stream (no allocation, no host
    synchronisation once the plan's tables are on the device), so it can be captured; every
    replay, with eager work and synchronisations in between, must reproduce the eager output."""
    cfg = get_config("single")
    routes = make_routes(cfg).numpy()
    q, k, v = make_qkv(cfg, DEV)
    plan = vorta.plan_for(cfg)
    ws = torch.empty(vorta.vorta_workspace_bytes(plan, routes), dtype=torch.uint8, device=DEV)
    eager = vorta.vorta_routed_attention_layer(plan, q, k, v, routes, workspace=ws)   # also uploads the tables
    torch.cuda.synchronize()
    out = torch.empty_like(q)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            vorta.vorta_routed_attention_layer(plan, q, k, v, routes, out=out, workspace=ws, stream=side)
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(3):
        out.fill_(float("nan"))
        ws.random_(0, 255)                      # eager work between replays; every buffer is rewritten by the graph
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager), f"replay {rep}"


def test_soft_mixture_blends_the_three_branches():
    cfg = small_cfg("mix", (4, 4, 6), 3, "bf16", (2, 2, 3), (1, 3, 1), [0, 1, 2])
    q, k, v = make_qkv(cfg, DEV)
    plan = vorta.plan_for(cfg)
    alpha = np.array([[0.2, 0.5, 0.3], [1.0, 0.0, 0.0], [0.1, 0.1, 0.8]])
    out = vorta.vorta_soft_mixture_layer(plan, q, k, v, alpha)
    torch.cuda.synchronize()
    want = vo.soft_mixture_layer(f64(q), f64(k), f64(v), alpha, spec_of(cfg))
    err = np.abs(f64(out) - want).max()
    say(f"soft mixture max-abs {err:.3e}")
    assert err <= 2e-2


def test_error_paths_do_not_launch():
    cfg = get_config("tiny")
    q, k, v = make_qkv(cfg, DEV)
    plan = vorta.plan_for(cfg)
    with pytest.raises(vorta.VortaError) as e:
        vorta.vorta_routed_attention_layer(plan, q, k, v, [0, 5])
    assert e.value.code == -5
    with pytest.raises(vorta.VortaError) as e:
        vorta.vorta_routed_attention_layer(plan, q, k, v, [1, 2], workspace=torch.empty(512, dtype=torch.uint8, device=DEV))
    assert e.value.code == -4
    # tensors that do not fit the plan are stopped in the binding, before any C call
    half = q[:, : cfg.n_tokens // 2].contiguous()
    for bad, code in ((dict(q=half), -2),                                  # fewer tokens
                      (dict(q=q[:1].contiguous()), -2),                    # fewer heads
                      (dict(q=q.to(torch.bfloat16)), -3),                  # dtype of another plan
                      (dict(q=q.transpose(0, 1).contiguous()), -2),        # the other layout
                      (dict(q=q.transpose(1, 2)), -2),                     # not even the same rank order
                      (dict(out=torch.empty_like(half)), -2),
                      (dict(workspace=torch.empty(1 << 20, dtype=torch.float32, device=DEV)), -1),
                      (dict(routes=[0]), -1), (dict(routes=[0, 1, 2]), -1)):
        kw = dict(q=q, k=k, v=v, routes=[0, 0])
        kw.update(bad)
        with pytest.raises(vorta.VortaError) as e:
            vorta.vorta_routed_attention_layer(plan, kw.pop("q"), kw.pop("k"), kw.pop("v"), kw.pop("routes"), **kw)
        assert e.value.code == code, bad.keys()
    routes = np.array([1, 2], dtype=np.uint8)
    with pytest.raises(vorta.VortaError) as e:
        vorta.vorta_bcs_build_index(plan, k, routes, keep_idx=torch.empty(1, plan.n_core + 1, dtype=torch.int32, device=DEV))
    assert e.value.code == -2
    with pytest.raises(vorta.VortaError) as e:
        vorta.vorta_bcs_pool(plan, q, routes, torch.empty(1, plan.n_core, dtype=torch.int64, device=DEV),
                             torch.empty(1, plan.n_video, dtype=torch.int32, device=DEV))
    assert e.value.code == -3
    with pytest.raises(vorta.VortaError) as e:
        vorta.vorta_attention_routed(plan, routes, q=q, k=k, v=v, out=torch.empty_like(q),
                                     q_c=torch.empty(2, plan.n_core_tokens, cfg.head_dim, device=DEV))   # two slots, one route-2 head
    assert e.value.code == -2
    # fp32 plans have no gathering window kernel: scatter_back without o_t would leave rows unwritten
    o_c = torch.empty(1, plan.n_core_tokens, cfg.head_dim, device=DEV)
    assign = torch.zeros(1, plan.n_video, dtype=torch.int32, device=DEV)
    with pytest.raises(vorta.VortaError) as e:
        vorta.vorta_scatter_back(plan, routes, None, o_c, assign, torch.empty_like(q))
    assert e.value.code == -1 and "o_t" in str(e.value)
    # a misaligned pointer reaches the library and is refused there (ctypes, past the binding's checks)
    import ctypes
    lib = vorta.load_library()
    r = (ctypes.c_uint8 * 2)(0, 0)
    ws = torch.empty(vorta.vorta_workspace_bytes(plan, [0, 0]), dtype=torch.uint8, device=DEV)
    rc = lib.vorta_routed_attention_layer(plan.handle, ctypes.c_void_p(q.data_ptr() + 4), ctypes.c_void_p(k.data_ptr()),
                                          ctypes.c_void_p(v.data_ptr()), r, ctypes.c_void_p(q.data_ptr()),
                                          ctypes.c_void_p(ws.data_ptr()), ctypes.c_size_t(ws.numel()), None)
    assert rc == -7


# ------------------------------------------------------------------ full-size layers -----

def sampled_rows(cfg, plan, head, rng):
    """Rows the oracle evaluates one by one: seeded random rows, every row of a corner tile
    and of an interior tile, the last rows, and all text rows."""
    L = cfg.n_video
    perm = vorta.vorta_tile_permutation(plan)
    tile_of = np.searchsorted(vorta.vorta_tile_row0(plan), perm, side="right") - 1
    corner = np.nonzero(tile_of == 0)[0]
    mid = np.nonzero(tile_of == plan.n_tiles // 2 + plan.tiles[2] // 2)[0]
    last = np.nonzero(tile_of == plan.n_tiles - 1)[0]      # clipped on every axis the tile does not divide
    # 512 random rows, every row of a corner tile and of a tile in the middle of the grid, the
    # last video rows (ragged tail of the last query block) and every text row
    # (tiles of more than 128 tokens: every other / third ... row, so that they cost no more)
    step = max(1, len(corner) // 128)
    n_random = 512 if plan.tile_tokens <= 128 else 192
    rows = np.concatenate([rng.choice(L, n_random, replace=False), corner[::step], mid[::step], last[::step],
                           np.arange(L - 3, L), L + np.arange(cfg.n_text)])
    return np.unique(rows)


@pytest.mark.parametrize("name", ["wan480p", "wan720p", "hunyuan720p", "paper720p", "paper_wan720p"])
def test_full_size_layer_on_sampled_rows(name):
    cfg = get_config(name)
    routes = make_routes(cfg).numpy()
    say(f"{name}: generating inputs")
    q, k, v = make_qkv(cfg, DEV)
    plan = vorta.plan_for(cfg)
    ws = torch.empty(vorta.vorta_workspace_bytes(plan, routes), dtype=torch.uint8, device=DEV)
    out = vorta.vorta_routed_attention_layer(plan, q, k, v, routes, workspace=ws)
    torch.cuda.synchronize()
    say(f"{name}: layer done, checking against the oracle")
    off = vorta.vorta_workspace_layout(plan, routes)
    n_lr = int((routes == 2).sum())
    keep_idx = ws[off[8]: off[8] + n_lr * plan.n_core * 4].view(torch.int32).view(n_lr, plan.n_core).cpu().numpy()
    assign = ws[off[9]: off[9] + n_lr * plan.n_video * 4].view(torch.int32).view(n_lr, plan.n_video).cpu().numpy()
    spec = spec_of(cfg)
    rng = np.random.default_rng(cfg.seed)
    worst = [0.0, 0.0, 0.0]
    lr_slot = 0
    L = cfg.n_video
    for h, r in enumerate(routes):
        rows = sampled_rows(cfg, plan, h, rng)
        Q, K, V = f64(q[h]), f64(k[h]), f64(v[h])
        if r == 2:
            ki, asg, gap = vo.bcs_select(K[:L], cfg.grid, cfg.bucket, cfg.keep_num, cfg.keep_den)
            assert gap > 1e-12
            assert np.array_equal(keep_idx[lr_slot], ki) and np.array_equal(assign[lr_slot], asg), f"head {h}"
            lr_slot += 1
            want = vo.coreset_attention(Q, K, V, spec, rows, index=(ki, asg))
        else:
            want = vo.head_attention(int(r), Q, K, V, spec, rows)
        got = f64(out[h][torch.as_tensor(rows, device=DEV)])
        err = np.abs(got - want).max()
        worst[r] = max(worst[r], err)
        say(f"  {name} head {h:2d} route {r}: {len(rows)} rows, max-abs {err:.3e}")
        assert err <= TOL[cfg.dtype], f"{name} head {h} route {r}: {err}"
    assert torch.isfinite(out.float()).all()
    say(f"{name}: worst max-abs per route {worst}")


@pytest.mark.parametrize("tile", [(4, 4, 6), (4, 8, 6)])
def test_largest_tensors_a_plan_accepts(tile):
    """131,071 tokens x 128 heads x 128 = 2^31 - 16,384 elements per tensor (4 GiB in bf16), the
    most a plan takes, in the token-major layout, where every head's rows are spread over the
    whole tensor: the 32-bit element and byte offsets of the kernels run up to their limits.
    Tiles of 96 and of 192 tokens take the 4- and the 8-wavefront window kernel.  The first and
    the last heads of every route are held to the oracle on sampled rows, the last rows among
    them; the 31-frame grid is divided by neither the tile nor the bucket."""
    heads = vorta.VORTA_MAX_HEADS if hasattr(vorta, "VORTA_MAX_HEADS") else 128
    routes = np.array([0, 1, 2] + [1, 2] * 61 + [2, 1, 0], dtype=np.uint8)
    assert len(routes) == heads == 128
    cfg = small_cfg("largest", (31, 64, 66), heads, "bf16", tile, (3, 3, 3), routes.tolist(), n_text=127, seed=23)
    N, L = cfg.n_tokens, cfg.n_video
    assert N * heads * 128 == 2 ** 31 - 16384
    say(f"largest tile {tile}: generating {3 * N * heads * 128 * 2 / 2 ** 30:.1f} GiB of inputs")
    q, k, v = make_qkv(cfg, DEV, layout=0)
    plan = vorta.plan_for(cfg, layout=0)
    ws = torch.empty(vorta.vorta_workspace_bytes(plan, routes), dtype=torch.uint8, device=DEV)
    out = vorta.vorta_routed_attention_layer(plan, q, k, v, routes, workspace=ws)
    torch.cuda.synchronize()
    say("largest: layer done, checking against the oracle")
    off = vorta.vorta_workspace_layout(plan, routes)
    n_lr = int((routes == 2).sum())
    keep_idx = ws[off[8]: off[8] + n_lr * plan.n_core * 4].view(torch.int32).view(n_lr, plan.n_core)
    assign = ws[off[9]: off[9] + n_lr * plan.n_video * 4].view(torch.int32).view(n_lr, plan.n_video)
    spec = spec_of(cfg)
    rng = np.random.default_rng(cfg.seed)
    rows = np.unique(np.concatenate([rng.choice(L, 48, replace=False), [0, L - 2, L - 1, L, N - 2, N - 1]]))
    lr_slot_of = {int(h): i for i, h in enumerate(np.nonzero(routes == 2)[0])}
    for h in (0, 1, 2, 125, 126, 127):
        r = int(routes[h])
        Q, K, V = f64(q[:, h]), f64(k[:, h]), f64(v[:, h])
        if r == 2:
            ki, asg, gap = vo.bcs_select(K[:L], cfg.grid, cfg.bucket, cfg.keep_num, cfg.keep_den)
            assert gap > 1e-12
            slot = lr_slot_of[h]
            assert np.array_equal(keep_idx[slot].cpu().numpy(), ki) and np.array_equal(assign[slot].cpu().numpy(), asg), f"head {h}"
            want = vo.coreset_attention(Q, K, V, spec, rows, index=(ki, asg))
        else:
            want = vo.head_attention(r, Q, K, V, spec, rows)
        got = f64(out[:, h][torch.as_tensor(rows, device=DEV)])
        err = np.abs(got - want).max()
        say(f"  largest head {h:3d} route {r}: {len(rows)} rows, max-abs {err:.3e}")
        assert err <= TOL["bf16"], f"head {h} route {r}: {err}"
    assert torch.isfinite(out[-1024:].float()).all() and torch.isfinite(out[:1024].float()).all()
