"""Attention kernels at the sizes where their splits can go wrong: fewer keys than one block, fewer
blocks than key groups, remainders of rows and keys, run lists that end inside a block, and scores
that leave the range of the lagging row reference.  Against the fp64 oracle."""
import sys

import numpy as np
import pytest
import torch

import paper_2505_18809_amd as vorta
from oracle import vorta_oracle as vo
from synth_inputs import LayerConfig, make_qkv
from helpers import PIPE, f32_wavefronts, f64, force_form, spec_of

pytestmark = pytest.mark.gpu
DEV = "cuda"


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def layer_error(cfg, q, k, v, layout, bar):
    """Runs the layer, holds every head to the oracle within bar(want)."""
    plan = vorta.plan_for(cfg, layout=layout)
    out = vorta.vorta_routed_attention_layer(plan, q, k, v, cfg.fixed_routes)
    torch.cuda.synchronize()
    hnd = (lambda t: t) if layout == 1 else (lambda t: t.transpose(0, 1))
    spec = spec_of(cfg)
    for h, r in enumerate(cfg.fixed_routes):
        want = vo.head_attention(int(r), f64(hnd(q)[h]), f64(hnd(k)[h]), f64(hnd(v)[h]), spec, None)
        err = np.abs(f64(hnd(out)[h]) - want)
        say(f"{cfg.name} head {h} route {r}: max-abs {err.max():.3e}")
        assert (err <= bar(want)).all(), f"head {h} route {r}: {err.max():.3e}"


# fp64 inside, one rounding to fp32: half an ulp of the result, and as much again for the sums
def fp32_bar(want):
    return 2.0 ** -23 * np.maximum(1.0, np.abs(want))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("grid,tile,n_text,layout", [
    ((1, 1, 1), (1, 1, 1), 0, 1),          # one key: three wavefronts without any
    ((1, 3, 5), (1, 2, 3), 0, 0),          # 15 keys, tiles of 1 to 6 rows
    ((2, 3, 3), (2, 3, 2), 15, 1),         # 33 keys: two blocks and one key
    ((3, 7, 7), (2, 3, 5), 3, 0),          # runs that end inside a block
    ((4, 14, 18), (3, 4, 7), 16, 1),       # 1,024 rows and fewer items than CUs: eight-wavefront workgroups
    ((8, 16, 20), (3, 4, 7), 17, 1),       # 2,577 rows: more items than CUs
])
def test_fp32_attention_at_the_edges_of_its_split(grid, tile, n_text, layout, d):
    cfg = LayerConfig(f"edge{grid}d{d}", grid, 3, d, "fp32", tile, (3, 1, 3), seed=5, n_text=n_text, fixed_routes=(0, 1, 2))
    say(cfg.name)
    q, k, v = make_qkv(cfg, DEV, layout)
    layer_error(cfg, q, k, v, layout, fp32_bar)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("grid,routes,n_text,wavefronts", [
    ((1, 16, 31), (0,), 0, 4), ((1, 7, 71), (0,), 0, 8),           # 31 whole key blocks; 31 and one key
    ((2, 16, 32), (2,), 0, 8), ((8, 9, 9), (1,), 0, 8),            # core-set rows, window items of 32 blocks and more
    ((4, 9, 15), (1, 2), 16, 8),                                   # text rows over 35 blocks, window items of fewer blocks than wavefronts
])
def test_fp32_attention_on_either_side_of_its_number_of_wavefronts(grid, routes, n_text, wavefronts, d):
    cfg = LayerConfig(f"waves{grid}d{d}", grid, len(routes), d, "fp32", (2, 3, 3) if n_text else (3, 3, 3), (1, 1, 1) if n_text else (3, 3, 3),
                      seed=15, n_text=n_text, fixed_routes=routes, bucket=(2, 1, 1), keep_num=1, keep_den=2)
    say(cfg.name)
    assert f32_wavefronts(vorta.plan_for(cfg), routes) == wavefronts
    q, k, v = make_qkv(cfg, DEV, 1)
    # pooled rows are rounded to fp32 on their way: 2^-24 of V (up to 4.5), and of each of the 2 d factors of a score, which
    # moves the weights by scale * 2^-24 * sqrt(2 d) * |q k| (about 1e-7 for the largest): the layer's own bar of 1e-5 holds both
    layer_error(cfg, q, k, v, 1, (lambda want: 1e-5) if 2 in routes else fp32_bar)


def test_fp32_row_reference_follows_scores_far_beyond_its_slack():
    """Scores that rise by thousands of log2 units along the keys (and fall again): the row reference has
    to be raised block after block, and shares of the key stream whose reference is far below the
    largest have to vanish from the merge."""
    cfg = LayerConfig("far_scores", (4, 6, 8), 3, 64, "fp32", (2, 3, 4), (3, 3, 3), seed=9, fixed_routes=(0, 1, 2))
    say(cfg.name)
    q, k, v = make_qkv(cfg, DEV)
    n = cfg.n_tokens
    ramp = torch.sin(torch.linspace(0.0, 9.0, n, device=DEV))[:, None] * 3000.0
    u = torch.zeros(64, device=DEV)
    u[3] = 1.0
    k = (k + ramp * u).contiguous()
    layer_error(cfg, q, k, v, 1, lambda want: 1e-5 * np.maximum(1.0, np.abs(want)))


@pytest.mark.parametrize("layout", [1, 0])
@pytest.mark.parametrize("grid,n_text", [((1, 1, 1), 0), ((1, 4, 32), 0), ((1, 3, 43), 5), ((2, 8, 16), 0), ((1, 1, 257), 3),
                                         ((4, 8, 12), 0), ((5, 7, 11), 70)])
def test_bf16_window_rows_cut_across_tile_borders(grid, n_text, layout):
    """Windows that cover the grid: every tile (of 1 to 6 tokens, clipped ones among them) has one key set, so
    the rows of all tiles are one sequence of 1, 128, 129, 256, 257, 384 and 385 rows, cut into blocks of 64 (the
    split kernel, which the rule takes at these sizes; blocks of 256 with a rest: test_gpu_attention_forms.py).
    Gathered from the caller's tensors and over tile-ordered copies."""
    cfg = LayerConfig(f"cut{grid}", grid, 3, 128, "bf16", (1, 2, 3), (99, 99, 999), seed=17, n_text=n_text, fixed_routes=(1, 0, 1))
    say(cfg.name)
    q, k, v = make_qkv(cfg, DEV, layout)
    layer_error(cfg, q, k, v, layout, lambda want: 2e-2)
    plan = vorta.plan_for(cfg, layout=layout)
    r = cfg.fixed_routes
    q_t, k_t, v_t = (vorta.vorta_reorder_to_tiles(plan, t, r) for t in (q, k, v))
    o_t, out = torch.empty_like(q_t), torch.zeros_like(q)
    vorta.vorta_attention_routed(plan, r, q=q, k=k, v=v, out=out, q_t=q_t, k_t=k_t, v_t=v_t, o_t=o_t)
    vorta.vorta_scatter_back(plan, r, o_t, None, None, out)
    torch.cuda.synchronize()
    # video rows: the same items over the same rows, read from other places.  Text rows of the window heads meet
    # all keys in sequence order here and in tile order there: equal up to the rounding of P and the output.
    layer = vorta.vorta_routed_attention_layer(plan, q, k, v, r)
    if layout == 0:
        out, layer = out.transpose(0, 1), layer.transpose(0, 1)
    n = cfg.n_video
    assert torch.equal(out[:, :n], layer[:, :n]) and torch.equal(out[1], layer[1])
    assert n_text == 0 or (out[:, n:].float() - layer[:, n:].float()).abs().max().item() <= 2e-2


@pytest.mark.parametrize("grid,heads,n_text,layout", [
    ((1, 1, 1), 3, 0, 1),             # one key: shares of the key stream without any
    ((1, 1, 31), 3, 2, 0),            # 33 keys
    ((1, 8, 8), 3, 1, 1),             # 65 rows and keys: a second item of one row
    ((2, 8, 8), 3, 0, 0),             # 128
    ((3, 6, 9), 3, 31, 1),            # 193 keys, odd and even superblocks of the routes
    ((1, 31, 31), 3, 0, 1),           # 961 keys
    ((3, 7, 49), 3, 124, 0),          # 1,153 keys: nine superblocks of 128 and one key
    ((1, 47, 49), 3, 2, 0),           # 2,305: four shares, 18 superblocks and one key
    ((4, 12, 16), 42, 0, 1),          # 42 heads of 768 tokens: more items than CUs
])
def test_bf16_attention_at_the_edges_of_its_key_split(grid, heads, n_text, layout):
    """Small launches share the key stream of 64 query rows among two or four wavefronts: row and key
    remainders, superblock counts of both parities, shares without a key, every route in one launch."""
    cfg = LayerConfig(f"split{grid}", grid, heads, 128, "bf16", (2, 3, 4), (3, 1, 3), seed=41, n_text=n_text,
                      fixed_routes=tuple(h % 3 for h in range(heads)))
    say(cfg.name)
    q, k, v = make_qkv(cfg, DEV, layout)
    layer_error(cfg, q, k, v, layout, lambda want: 2e-2)
    again = vorta.vorta_routed_attention_layer(vorta.plan_for(cfg, layout=layout), q, k, v, cfg.fixed_routes)
    assert torch.equal(again, vorta.vorta_routed_attention_layer(vorta.plan_for(cfg, layout=layout), q, k, v, cfg.fixed_routes))


def test_bf16_split_rows_whose_maxima_jump_from_share_to_share():
    """Scores that rise and fall by hundreds of log2 units along the keys, so that the shares of one row end on
    references far apart and all but one vanish from the merge."""
    cfg = LayerConfig("jumps", (4, 16, 18), 3, 128, "bf16", (2, 4, 6), (3, 3, 3), seed=43, fixed_routes=(0, 1, 2))
    say(cfg.name)
    q, k, v = make_qkv(cfg, DEV)
    ramp = torch.sin(torch.linspace(0.0, 25.0, cfg.n_tokens, device=DEV))[:, None] * 400.0
    u = torch.zeros(128, device=DEV)
    u[5] = 1.0
    k = (k.float() + ramp * u).to(torch.bfloat16)
    # rows that few keys dominate return those value rows: half an ulp of the output, and P's rounding
    layer_error(cfg, q, k, v, 1, lambda want: np.maximum(2e-2, 2.0 ** -7 * np.abs(want)))


@pytest.mark.parametrize("grid,bucket,keep,heads,dtype,d,n_text,layout", [
    ((4, 8, 8), (2, 3, 2), (1, 2), 3, "bf16", 128, 0, 1),
    ((5, 7, 9), (4, 4, 4), (1, 4), 3, "bf16", 128, 21, 0),       # up to 64 tokens a bucket, most of them merged, clipped
    ((5, 9, 11), (1, 17, 1), (1, 3), 4, "bf16", 128, 0, 1),
    ((3, 4, 5), (1, 1, 1), (1, 2), 2, "bf16", 128, 5, 1),        # every token its own bucket
    ((21, 30, 52), (3, 5, 4), (3, 4), 6, "bf16", 128, 40, 0),    # long items: the pipelined kernel
    ((21, 30, 52), (2, 3, 2), (1, 2), 8, "bf16", 128, 0, 1),
    ((5, 7, 9), (4, 4, 4), (1, 4), 3, "fp32", 64, 21, 0),
    ((4, 8, 8), (2, 3, 2), (1, 2), 3, "fp32", 128, 2, 1),
])
def test_core_set_rows_written_to_their_tokens_equal_the_staged_unpool(grid, bucket, keep, heads, dtype, d, n_text, layout):
    """The layer call writes core-set rows from the attention kernel to the tokens that read them; the staged
    calls leave them in o_c and unpool in a pass.  Same launches otherwise: equal bit for bit."""
    cfg = LayerConfig(f"unpool{bucket}", grid, heads, d, dtype, (2, 4, 4), (3, 3, 3), seed=47, n_text=n_text, bucket=bucket,
                      keep_num=keep[0], keep_den=keep[1], fixed_routes=(2,) * heads)
    say(f"{cfg.name} {grid} {dtype}")
    q, k, v = make_qkv(cfg, DEV, layout)
    plan = vorta.plan_for(cfg, layout=layout)
    r = cfg.fixed_routes
    out = torch.full_like(q, float("nan"))
    vorta.vorta_routed_attention_layer(plan, q, k, v, r, out=out)
    _, assign, q_c, k_c, v_c = vorta.vorta_bcs_select_pool(plan, q, k, v, r)
    o_c, staged = torch.empty_like(q_c), torch.full_like(q, float("nan"))
    vorta.vorta_attention_routed(plan, r, q_c=q_c, k_c=k_c, v_c=v_c, o_c=o_c)
    vorta.vorta_scatter_back(plan, r, None, o_c, assign, staged)
    torch.cuda.synchronize()
    assert torch.equal(out, staged)


@pytest.mark.parametrize("grid,bucket,keep,heads,d,n_text", [
    ((3, 17, 7), (1, 17, 1), (1, 3), 3, 128, 3),     # 17 tokens a bucket: one more than a turn of the look-ups
    ((3, 16, 7), (1, 16, 1), (1, 8), 2, 64, 0),      # exactly a turn, nearly all merged
    ((9, 12, 14), (3, 3, 3), (2, 3), 1, 64, 0),      # eight wavefronts and four pieces of a row
    ((9, 12, 14), (3, 3, 3), (1, 3), 1, 128, 19),    # eight wavefronts and eight pieces
])
def test_fp32_core_set_rows_of_pieces_from_all_wavefronts(grid, bucket, keep, heads, d, n_text):
    test_core_set_rows_written_to_their_tokens_equal_the_staged_unpool(grid, bucket, keep, heads, "fp32", d, n_text, 1)


@pytest.mark.parametrize("n_text,layout,halves", [(0, 1, 0), (0, 1, 128), (77, 0, 131)])
def test_long_and_window_items_in_one_launch(n_text, layout, halves):
    """A layer large enough for 256-row items on every route: window items follow the long ones in one launch, the last
    of them in halves.  Sampled rows of one head per route."""
    cfg = LayerConfig("one_launch", (21, 29, 52), 8, 128, "bf16", (3, 6, 4), (3, 3, 3), seed=53, n_text=n_text,
                      fixed_routes=(1, 0, 2, 1, 2, 1, 2, 1))
    say(cfg.name)
    q, k, v = make_qkv(cfg, DEV, layout)
    plan = force_form(vorta.plan_for(cfg, layout=layout), PIPE, halves)
    out = vorta.vorta_routed_attention_layer(plan, q, k, v, cfg.fixed_routes)
    torch.cuda.synchronize()
    hnd = (lambda t: t) if layout == 1 else (lambda t: t.transpose(0, 1))
    rows = np.unique(np.concatenate([np.arange(0, cfg.n_tokens, 397), np.arange(cfg.n_tokens - 9, cfg.n_tokens)]))
    for h in (0, 7, 1, 6):
        r = cfg.fixed_routes[h]
        want = vo.head_attention(r, f64(hnd(q)[h]), f64(hnd(k)[h]), f64(hnd(v)[h]), spec_of(cfg), rows)
        err = np.abs(f64(hnd(out)[h][torch.as_tensor(rows, device=DEV)]) - want).max()
        say(f"one launch, head {h} route {r}: max-abs {err:.3e}")
        assert err <= 2e-2


@pytest.mark.parametrize("dtype,d,routes,rope,shared", [
    ("fp32", 64, (1, 2, 1), None, "qkv"),             # window heads over tile-ordered copies where k or v is overwritten
    ("fp32", 128, (1, 2, 1, 1, 2), None, "qkv"),
    ("fp32", 128, (1, 2, 1), (44, 42, 42), "qkv"),
    ("fp32", 128, (0, 2, 1), (44, 42, 42), "qk"),     # attention reads the rotated copies of q and k
    ("fp32", 64, (0, 1, 2), None, "q"),
    ("bf16", 128, (2, 2, 2), None, "qkv"),
    ("bf16", 128, (0, 1, 2), (44, 42, 42), "qk"),
    ("bf16", 128, (0, 1, 2), None, "q"),
])
@pytest.mark.parametrize("layout,n_text", [(1, 0), (0, 19)])
def test_output_in_the_memory_of_an_input(dtype, d, routes, rope, shared, layout, n_text):
    """The layer call with `out` in the memory of q, k or v, where that is allowed, gives what it gives with a tensor of
    its own: bit for bit, but for text rows of fp32 window heads over copies, which meet their keys in another
    order (half an ulp of the result either way)."""
    cfg = LayerConfig(f"shared{dtype}", (7, 12, 13), len(routes), d, dtype, (2, 3, 4), (3, 3, 3), seed=59, n_text=n_text,
                      fixed_routes=routes, rope_dims=rope)
    say(f"{cfg.name} {routes} layout {layout}")
    plan = vorta.plan_for(cfg, layout=layout)
    vorta.vorta_plan_upload(plan)
    inputs = make_qkv(cfg, DEV, layout)
    want = vorta.vorta_routed_attention_layer(plan, *inputs, routes)
    ws = torch.empty(vorta.vorta_workspace_bytes(plan, routes), dtype=torch.uint8, device=DEV)
    for name in shared:
        for static in (False, True):
            x = [t.clone() for t in inputs]
            out = x["qkv".index(name)]
            if static:
                vorta.vorta_routed_attention_layer_static(plan, *x, routes, out)
            else:
                vorta.vorta_routed_attention_layer(plan, *x, routes, out=out, workspace=ws.random_(0, 255))
            torch.cuda.synchronize()
            a, b = (out, want) if layout == 1 else (out.transpose(0, 1), want.transpose(0, 1))
            assert torch.equal(a[:, :cfg.n_video], b[:, :cfg.n_video]), name
            a, b = a[:, cfg.n_video:].double(), b[:, cfg.n_video:].double()
            assert ((a - b).abs() <= 2.0 ** -23 * b.abs()).all(), name


@pytest.mark.parametrize("masked", [-float("inf"), torch.finfo(torch.bfloat16).min], ids=["inf", "lowest"])
@pytest.mark.parametrize("grid,heads,dtype", [((21, 29, 52), 8, "bf16"),      # the pipelined kernel on every route
                                              ((9, 8, 12), 4, "bf16"),        # the split kernel
                                              ((9, 8, 12), 4, "fp32")])
def test_rows_whose_first_keys_are_all_masked(grid, heads, dtype, masked):
    """Masked keys as programs mark them: a channel in which every query is at least 1.5 holds -inf, or the
    lowest bf16 value, in the keys of the first six frames, so the scores of the first blocks of many rows are
    -inf (in fp32 arithmetic also for the lowest value).  No row sees masked keys only, and masked keys weigh 0.
    The core-set branch takes the finite mask only, and its rows of those frames are left out: the
    similarities of masked tokens are ties of a rounding's size."""
    if dtype == "fp32" and masked != -float("inf"):
        masked = torch.finfo(torch.float32).min
    routes = (0, 1, 2, 1, 0, 1, 2, 1)[:heads] if masked != -float("inf") else (0, 1, 1, 0, 1, 1, 1, 1)[:heads]
    cfg = LayerConfig("masked", grid, heads, 128, dtype, (3, 6, 4), (3, 3, 3), seed=61, n_text=21, fixed_routes=routes)
    say(f"{cfg.name} {grid} {dtype} {masked}")
    q, k, v = make_qkv(cfg, DEV)
    q[..., 7] = q[..., 7].abs() + 1.5
    k[:, : 6 * grid[1] * grid[2], 7] = masked
    plan = vorta.plan_for(cfg)
    out = vorta.vorta_routed_attention_layer(plan, q, k, v, routes)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.arange(0, cfg.n_tokens, max(1, cfg.n_tokens // 97)), np.arange(cfg.n_tokens - 9, cfg.n_tokens)]))
    for h in range(min(heads, 4)):
        some = rows[rows >= 6 * grid[1] * grid[2]] if routes[h] == 2 else rows
        with np.errstate(all="ignore"):
            want = vo.head_attention(routes[h], f64(q[h]), f64(k[h]), f64(v[h]), spec_of(cfg), some)
        assert np.isfinite(want).all()
        err = np.abs(f64(out[h][torch.as_tensor(some, device=DEV)]) - want).max()
        say(f"masked, head {h} route {routes[h]}: max-abs {err:.3e}")
        assert err <= (2e-2 if dtype == "bf16" else 1e-5)
