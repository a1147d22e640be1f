"""Every form of the bf16 attention launch at the sizes where it can go wrong.  The library chooses the form from
the size of the layer, and small layers run on the split kernel; here each of them is held to the fp64
oracle on the same small layers: split kernel with two and four key shares, pipelined kernels with none, some
and all items issued as half-row items, and pipelined with the window rows on the split kernel or all of them in
128-row items."""
import sys

import numpy as np
import pytest
import torch

import paper_2505_18809_amd as vorta
from oracle import vorta_oracle as vo
from synth_inputs import LayerConfig, make_qkv
from helpers import PIPE, PIPE_SPLIT_WIN, PIPE_WIN_128, SPLIT2, SPLIT4, f64, force_form, spec_of

pytestmark = pytest.mark.gpu
DEV = "cuda"
FORMS = [(SPLIT2, -1), (SPLIT4, -1), (PIPE, 0), (PIPE, 2), (PIPE, 1 << 20), (PIPE_SPLIT_WIN, 0), (PIPE_SPLIT_WIN, 1 << 20),
         (PIPE_WIN_128, 0), (PIPE_WIN_128, 1 << 20)]


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def by_head(t, layout):
    return t if layout == 1 else t.transpose(0, 1)


def oracle(cfg, q, k, v, layout, **over):
    q, k, v = (by_head(t, layout) for t in (q, k, v))
    return [vo.head_attention(int(r), f64(q[h]), f64(k[h]), f64(v[h]), spec_of(cfg, **over), None)
            for h, r in enumerate(cfg.fixed_routes)]


def close(out, want, layout, what, bar=2e-2):
    for h, w in enumerate(want):
        err = np.abs(f64(by_head(out, layout)[h]) - w)
        assert (err <= bar).all(), f"{what} head {h}: {err.max():.3e}"


LAYERS = [
    # grid, tile, window, text rows, routes, layout
    ((1, 1, 1), (1, 1, 1), (1, 1, 1), 0, (1, 0, 2), 1),                    # one key
    ((1, 8, 8), (1, 2, 3), (99, 99, 99), 1, (1, 0, 2), 0),                 # 65 rows and keys
    ((1, 4, 32), (1, 2, 3), (99, 99, 999), 0, (1, 1), 1),                  # window rows: 128, no long item
    ((1, 3, 43), (1, 2, 3), (99, 99, 999), 5, (1, 0, 1), 1),               # 129 rows, a block of more than 128
    ((2, 8, 16), (1, 2, 3), (99, 99, 999), 0, (1, 1, 2), 0),               # 256
    ((1, 1, 257), (1, 2, 3), (99, 99, 999), 3, (1, 2, 0), 0),              # 257: a block and one row
    ((5, 7, 11), (1, 2, 3), (99, 99, 999), 70, (1, 0, 1), 1),              # 385: a block and 129
    ((10, 12, 9), (6, 9, 8), (3, 3, 3), 9, (1, 0, 1, 2, 1), 0),            # tiles of up to 432 tokens, clipped
    ((9, 11, 14), (4, 6, 8), (3, 1, 3), 0, (1, 1, 1), 1),                  # window items alone, both sizes
    ((7, 10, 13), (3, 4, 5), (3, 3, 3), 300, (1, 0, 2, 1), 1),             # text rows over two long items
    ((3, 7, 49), (2, 3, 4), (3, 1, 3), 124, (0, 1, 2), 0),                 # 1,153 keys: one more than 18 blocks
    ((4, 8, 16), (2, 4, 4), (3, 3, 3), 0, (0, 2, 0, 1), 1),                # 512 keys: whole blocks
    ((1, 31, 31), (2, 3, 4), (3, 1, 3), 0, (0, 1, 2), 1),                  # 961
]


@pytest.mark.parametrize("grid,tile,window,n_text,routes,layout", LAYERS)
def test_layer_and_staged_calls_in_every_form(grid, tile, window, n_text, routes, layout):
    """The layer call against the oracle; the staged calls over tile-ordered copies as well, and core-set rows
    written from the kernel to their tokens equal those unpooled in a pass bit for bit."""
    cfg = LayerConfig(f"forms{grid}", grid, len(routes), 128, "bf16", tile, window, seed=71, n_text=n_text, fixed_routes=routes)
    q, k, v = make_qkv(cfg, DEV, layout)
    want = oracle(cfg, q, k, v, layout)
    plan = vorta.plan_for(cfg, layout=layout)
    r = np.array(routes)
    keep_idx, assign, q_c, k_c, v_c = vorta.vorta_bcs_select_pool(plan, q, k, v, routes)
    q_t, k_t, v_t = (vorta.vorta_reorder_to_tiles(plan, t, routes) for t in (q, k, v))
    for form, halves in FORMS:
        say(f"{cfg.name} {routes} form {form} halves {halves}")
        force_form(plan, form, halves)
        out = torch.full_like(q, float("nan"))
        vorta.vorta_routed_attention_layer(plan, q, k, v, routes, out=out)
        torch.cuda.synchronize()
        close(out, want, layout, f"form {form} halves {halves}")
        again = vorta.vorta_routed_attention_layer(plan, q, k, v, routes)
        assert torch.equal(out, again)
        staged = torch.full_like(q, float("nan"))
        o_t, o_c = torch.empty_like(q_t), torch.empty_like(q_c)
        vorta.vorta_attention_routed(plan, routes, q=q, k=k, v=v, out=staged, q_t=q_t, k_t=k_t, v_t=v_t, o_t=o_t,
                                     q_c=q_c, k_c=k_c, v_c=v_c, o_c=o_c)
        vorta.vorta_scatter_back(plan, routes, o_t, o_c, assign, staged)
        torch.cuda.synchronize()
        close(staged, want, layout, f"staged, form {form} halves {halves}")
        for h in np.nonzero(r != 1)[0]:
            assert torch.equal(by_head(out, layout)[h], by_head(staged, layout)[h])


@pytest.mark.parametrize("mode", [1, 2])
def test_centre_rules_in_every_form(mode):
    cfg = LayerConfig("centres", (8, 9, 10), 3, 128, "bf16", (2, 3, 3), (3, 3, 3), seed=73, n_text=6, fixed_routes=(1, 2, 1))
    q, k, v = make_qkv(cfg, DEV)
    want = oracle(cfg, q, k, v, 1, center_mode=("clamp", "identity", "block")[mode])
    plan = vorta.plan_for(cfg, center_mode=mode)
    for form, halves in FORMS:
        say(f"centre rule {mode} form {form} halves {halves}")
        force_form(plan, form, halves)
        close(vorta.vorta_routed_attention_layer(plan, q, k, v, cfg.fixed_routes), want, 1, f"form {form} halves {halves}")


def test_row_maxima_far_apart_in_every_form():
    """Scores that rise and fall by hundreds of log2 units along the keys: the row reference is raised again and
    again in the middle of the stream, and shares of it vanish from the merge.  A row that few keys
    dominate returns their value rows: half an ulp of the output, and the rounding of P."""
    cfg = LayerConfig("far", (4, 16, 18), 4, 128, "bf16", (2, 8, 6), (3, 3, 3), seed=43, n_text=40, fixed_routes=(0, 1, 2, 1))
    q, k, v = make_qkv(cfg, DEV)
    u = torch.zeros(128, device=DEV)
    u[5] = 1.0
    for height, turns in ((400.0, 25.0), (60.0, 1.5)):
        ramp = torch.sin(torch.linspace(0.0, turns, cfg.n_tokens, device=DEV))[:, None] * height
        kr = (k.float() + ramp * u).to(torch.bfloat16)
        want = oracle(cfg, q, kr, v, 1)
        plan = vorta.plan_for(cfg)
        for form, halves in FORMS:
            say(f"far maxima {height} form {form} halves {halves}")
            force_form(plan, form, halves)
            out = vorta.vorta_routed_attention_layer(plan, q, kr, v, cfg.fixed_routes)
            for h, w in enumerate(want):
                err = np.abs(f64(out[h]) - w)
                assert (err <= np.maximum(2e-2, 2.0 ** -7 * np.abs(w))).all(), f"form {form} halves {halves} head {h}: {err.max():.3e}"


@pytest.mark.parametrize("masked", [-float("inf"), torch.finfo(torch.bfloat16).min], ids=["inf", "lowest"])
def test_rows_whose_first_keys_are_all_masked_in_every_form(masked):
    """Scores of -inf in the first blocks of many rows (see the test over whole layers): they weigh 0."""
    cfg = LayerConfig("masked", (9, 8, 12), 3, 128, "bf16", (3, 6, 4), (3, 3, 3), seed=61, n_text=21, fixed_routes=(0, 1, 1))
    q, k, v = make_qkv(cfg, DEV)
    q[..., 7] = q[..., 7].abs() + 1.5
    k[:, : 6 * 96, 7] = masked
    with np.errstate(all="ignore"):
        want = oracle(cfg, q, k, v, 1)
    plan = vorta.plan_for(cfg)
    for form, halves in FORMS:
        say(f"masked {masked} form {form} halves {halves}")
        force_form(plan, form, halves)
        close(vorta.vorta_routed_attention_layer(plan, q, k, v, cfg.fixed_routes), want, 1, f"form {form} halves {halves}")


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("where", ["k", "v", "q"])
def test_infinities_and_nan_stay_with_the_rows_that_see_them(where, bad, dtype):
    """One token's key, value or query row holds a NaN or an infinity: as in exact arithmetic every row that sees it
    is not finite (of a bad value: in that channel), and all others are what they are without it."""
    cfg = LayerConfig("bad", (9, 8, 12), 3, 128, dtype, (3, 4, 4), (1, 1, 3), seed=67, n_text=10, fixed_routes=(0, 1, 1))
    q, k, v = make_qkv(cfg, DEV)
    token, channel = 500, 9
    if where != "q":
        q[:, :, channel] = q[:, :, channel].abs() + 0.5          # a score of +inf wherever the key is +inf
    want = oracle(cfg, q, k, v, 1)
    {"q": q, "k": k, "v": v}[where][:, token, channel] = bad
    plan = vorta.plan_for(cfg)
    sees = np.ones((3, cfg.n_tokens), dtype=bool)
    for h in (1, 2):
        for i in range(cfg.n_video):
            sees[h, i] = vo.sta_mask_row(i, cfg.grid, cfg.tile, cfg.window)[token]
    if where == "q":
        sees[:] = False
        sees[:, token] = True
    for form, halves in FORMS if dtype == "bf16" else [(0, -1)]:
        say(f"{bad} in {where} {dtype} form {form} halves {halves}")
        force_form(plan, form, halves)
        out = vorta.vorta_routed_attention_layer(plan, q, k, v, cfg.fixed_routes)
        for h in range(3):
            got = f64(out[h])
            hit = ~np.isfinite(got[:, channel]) if where == "v" else ~np.isfinite(got).any(axis=1)
            assert np.array_equal(hit, sees[h]), f"form {form} halves {halves} head {h}"
            if where == "v":
                keep = np.arange(128) != channel
                assert np.abs(got[:, keep] - want[h][:, keep]).max() <= (2e-2 if dtype == "bf16" else 1e-5)
            if not sees[h].all():
                assert np.abs(got[~sees[h]] - want[h][~sees[h]]).max() <= (2e-2 if dtype == "bf16" else 1e-5)


@pytest.mark.parametrize("grid,tile,n_text,rope,layout", [((4, 6, 8), (2, 3, 4), 0, None, 1), ((9, 11, 14), (4, 6, 8), 70, None, 0),
                                                         ((5, 7, 9), (2, 3, 4), 19, (44, 42, 42), 0)])
def test_soft_mixture_in_every_form(grid, tile, n_text, rope, layout):
    cfg = LayerConfig(f"mix{grid}", grid, 3, 128, "bf16", tile, (3, 1, 3), seed=79, n_text=n_text, rope_dims=rope)
    q, k, v = make_qkv(cfg, DEV, layout)
    alpha = np.array([[0.2, 0.5, 0.3], [1.0, 0.0, 0.0], [0.1, 0.1, 0.8]])
    want = vo.soft_mixture_layer(*(f64(by_head(t, layout)) for t in (q, k, v)), alpha, spec_of(cfg))
    plan = vorta.plan_for(cfg, layout=layout)
    for form, halves in FORMS:
        say(f"mixture {grid} form {form} halves {halves}")
        force_form(plan, form, halves)
        close(vorta.vorta_soft_mixture_layer(plan, q, k, v, alpha), list(want), layout, f"form {form} halves {halves}")


@pytest.mark.parametrize("routes", [(1, 0, 2, 1, 1, 1), (1, 1, 1, 1, 1, 1)])
def test_launches_of_many_items_in_every_form(routes):
    """More items than CUs, so that every XCD has some and the half-row items come last; sampled rows."""
    cfg = LayerConfig("many", (18, 24, 40), 6, 128, "bf16", (3, 6, 4), (3, 3, 3), seed=83, n_text=5, fixed_routes=routes)
    q, k, v = make_qkv(cfg, DEV, 0)
    rows = np.unique(np.concatenate([np.arange(0, cfg.n_tokens, 211), np.arange(cfg.n_tokens - 9, cfg.n_tokens)]))
    want = [vo.head_attention(r, f64(q[:, h]), f64(k[:, h]), f64(v[:, h]), spec_of(cfg), rows) for h, r in enumerate(routes)]
    plan = vorta.plan_for(cfg, layout=0)
    first = None
    for form, halves in FORMS + [(PIPE, 131)]:
        say(f"many items {routes} form {form} halves {halves}")
        force_form(plan, form, halves)
        out = torch.full_like(q, float("nan"))
        vorta.vorta_routed_attention_layer(plan, q, k, v, routes, out=out)
        torch.cuda.synchronize()
        assert torch.isfinite(out).all()
        for h, w in enumerate(want):
            assert np.abs(f64(out[torch.as_tensor(rows, device=DEV), h]) - w).max() <= 2e-2, f"form {form} halves {halves} head {h}"
        if form == PIPE:           # halves cut items, not the arithmetic of a row
            first = out if first is None else first
            assert torch.equal(out, first)
