"""The one-pass selection and merge at the edges of its instances (buckets of 12, 16 and 32 tokens, rows of
16 and 32 chunks) against the separate passes, bit for bit, and the oracle's index sets; odd grids, so
that the last bucket of each axis is clipped, and text rows that fill no workgroup."""
import numpy as np
import pytest
import torch

import paper_2505_18809_amd as vorta
from oracle import vorta_oracle as vo
from synth_inputs import LayerConfig, make_qkv
from helpers import f64, select_form

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("layout", [1, 0])
@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("fp32", 64), ("fp32", 128)])
@pytest.mark.parametrize("bucket", [(1, 1, 1), (2, 3, 2), (1, 13, 1), (4, 2, 2), (1, 17, 1), (3, 3, 3), (4, 2, 4), (3, 11, 1)])
def test_one_pass_selection_at_the_edges_of_its_instances(bucket, dtype, d, rope, layout):
    size = int(np.prod(bucket))
    dims = ((44, 42, 42) if d == 128 else (16, 24, 24)) if rope else None
    cfg = LayerConfig(f"bucket{size}", (5, 18, 7), 3, d, dtype, (1, 1, 1), (1, 1, 1), seed=300 + size, n_text=19,
                      fixed_routes=(2, 0, 2), bucket=bucket, keep_num=1, keep_den=2, rope_dims=dims)
    print(cfg.name, bucket, dtype, d, rope, layout, flush=True)
    q, k, v = make_qkv(cfg, DEV, layout)
    plan = vorta.plan_for(cfg, layout=layout)
    keep_idx, assign, q_c, k_c, v_c = vorta.vorta_bcs_select_pool(plan, q, k, v, cfg.fixed_routes)
    ki, asg = vorta.vorta_bcs_build_index(plan, k, cfg.fixed_routes)
    assert torch.equal(keep_idx, ki) and torch.equal(assign, asg)
    for name, got, src, turn in (("q", q_c, q, True), ("k", k_c, k, True), ("v", v_c, v, False)):
        want = vorta.vorta_bcs_pool(plan, src, cfg.fixed_routes, ki, asg, rotate=turn)
        assert torch.equal(got, want), name
    for slot, h in enumerate((0, 2)):
        kh = k[h] if layout == 1 else k[:, h]
        want_ki, want_asg, gap = vo.bcs_select(f64(kh)[:cfg.n_video], cfg.grid, bucket, 1, 2)
        if size > 2:       # two tokens: which of them names the slot is a tie
            assert gap > 1e-9 and np.array_equal(keep_idx[slot].cpu().numpy(), want_ki)
        assert np.array_equal(assign[slot].cpu().numpy(), want_asg)
        assert torch.equal(v_c[slot, plan.n_core:], (v[h] if layout == 1 else v[:, h])[cfg.n_video:])


@pytest.mark.parametrize("apart", [True, False])
@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("bucket,dtype,d", [((2, 3, 2), "bf16", 128), ((4, 2, 2), "bf16", 128), ((3, 3, 3), "bf16", 128),
                                            ((2, 3, 2), "fp32", 64), ((4, 2, 2), "fp32", 64), ((3, 3, 3), "fp32", 64),
                                            ((2, 3, 2), "fp32", 128), ((4, 2, 2), "fp32", 128)])
def test_one_pass_selection_with_a_wavefront_a_tensor_and_with_one_for_all(bucket, dtype, d, rope, apart):
    """Every instance of the one-pass kernel in both its forms: as many heads as still give each tensor of a bucket a wavefront on
    this device, and one more.  36 or 72 buckets a head, the last of each axis clipped."""
    dims = ((44, 42, 42) if d == 128 else (16, 24, 24)) if rope else None
    units = torch.cuda.get_device_properties(0).multi_processor_count

    def config(heads):
        return LayerConfig("pairs", (5, 18, 7), heads, d, dtype, (1, 1, 1), (1, 1, 1), seed=77, n_text=19, fixed_routes=(2,) * heads,
                           bucket=bucket, keep_num=2, keep_den=3, rope_dims=dims)

    def form(heads):
        return select_form(vorta.plan_for(config(heads), layout=0), (2,) * heads, units=units)["apart"] == 1
    heads = next(h for h in range(1, 128) if form(h) and not form(h + 1)) + (not apart)
    assert form(heads) == apart
    cfg = config(heads)
    print(bucket, heads, dtype, d, rope, flush=True)
    q, k, v = make_qkv(cfg, DEV, 0)
    plan = vorta.plan_for(cfg, layout=0)
    keep_idx, assign, q_c, k_c, v_c = vorta.vorta_bcs_select_pool(plan, q, k, v, cfg.fixed_routes)
    ki, asg = vorta.vorta_bcs_build_index(plan, k, cfg.fixed_routes)
    assert torch.equal(keep_idx, ki) and torch.equal(assign, asg)
    for name, got, src, turn in (("q", q_c, q, True), ("k", k_c, k, True), ("v", v_c, v, False)):
        assert torch.equal(got, vorta.vorta_bcs_pool(plan, src, cfg.fixed_routes, ki, asg, rotate=turn)), name


@pytest.mark.parametrize("grid,routes,n_text", [((4, 8, 8), (0, 1, 2), 19), ((5, 9, 7), (1, 2, 1, 0, 2, 2, 1), 3), ((4, 8, 8), (1, 2, 2, 2, 2, 2), 0),
                                                ((3, 6, 2), (0, 1, 2), 70), ((2, 3, 2), (0, 2), 40)])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("fp32", 64), ("fp32", 128)])
@pytest.mark.parametrize("bucket", [(2, 3, 2), (4, 2, 2)])
def test_text_rows_and_turned_rows_behind_the_planes_of_the_three_tensors(bucket, dtype, d, grid, routes, n_text):
    """The buffers that a layer call's selection launch leaves in the workspace, against the separate passes bit for bit, where each
    tensor of a bucket has a wavefront: text and turned rows that fill part of a plane of the grid, one, and several."""
    dims = (44, 42, 42) if d == 128 else (16, 24, 24)
    cfg = LayerConfig("planes", grid, len(routes), d, dtype, (1, 1, 1), (1, 1, 1), seed=91, n_text=n_text, fixed_routes=routes,
                      bucket=bucket, keep_num=1, keep_den=2, rope_dims=dims)
    print(bucket, dtype, d, grid, routes, n_text, flush=True)
    q, k, v = make_qkv(cfg, DEV, 0)
    plan = vorta.plan_for(cfg, layout=0)
    assert select_form(plan, routes, layer=True)["apart"] == 1
    workspace = torch.full((vorta.vorta_workspace_bytes(plan, routes),), 0xA5, dtype=torch.uint8, device=DEV)
    vorta.vorta_routed_attention_layer(plan, q, k, v, routes, workspace=workspace)
    off = [int(o) for o in vorta.vorta_workspace_layout(plan, routes)]

    def buffer(i, like):
        return workspace[off[i]:off[i] + like.numel() * like.element_size()].view(like.dtype).view(like.shape)
    ki, asg = vorta.vorta_bcs_build_index(plan, k, routes)
    assert torch.equal(buffer(8, ki), ki) and torch.equal(buffer(9, asg), asg)
    for i, src, turn in ((4, q, True), (5, k, True), (6, v, False)):
        want = vorta.vorta_bcs_pool(plan, src, routes, ki, asg, rotate=turn)
        assert torch.equal(buffer(i, want), want), i
    heads = [h for h, r in enumerate(routes) if r < 2]
    for i, src in ((10, q), (11, k)):
        want = vorta.vorta_rope_apply(plan, src, routes)
        assert torch.equal(buffer(i, want)[:, heads], want[:, heads]), i


@pytest.mark.parametrize("dims", [(44, 42, 42), (44, 42, 40), (2, 0, 126), (0, 64, 62), (0, 2, 0)])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_rotation_with_spans_that_cover_the_head_and_that_do_not(dims, dtype):
    """Spans that cover the head run without the test for channels past them.  One rounding to the element
    type (8 or 24 significant bits: up to 2^-8 or 2^-24 of a turned value, itself at most |u| + |v|), for bf16
    after one to fp32, and the fp32 table (2^-24 of each product) separate a turned pair from fp64; channels past the spans and text rows keep their bits."""
    cfg = LayerConfig("spans", (5, 6, 7), 2, 128, dtype, (1, 1, 1), (1, 1, 1), seed=41, n_text=5, fixed_routes=(0, 2),
                      bucket=(2, 3, 2), keep_num=1, keep_den=2, rope_dims=dims)
    print(dims, dtype, flush=True)
    q, k, v = make_qkv(cfg, DEV, 1)
    plan = vorta.plan_for(cfg, layout=1)
    got = vorta.vorta_rope_apply(plan, k, cfg.fixed_routes)[0]
    assert torch.equal(got[cfg.n_video:], k[0, cfg.n_video:])
    assert torch.equal(got[:, sum(dims):], k[0, :, sum(dims):])
    tok = np.arange(cfg.n_video)
    F, H, W = cfg.grid
    coords = np.stack([tok // (H * W), tok // W % H, tok % W], axis=1)
    x = f64(k[0])[:cfg.n_video]
    want = vo.rope_rotate(x, coords, dims, cfg.rope_theta)
    size = np.repeat(np.abs(x[:, 0::2]) + np.abs(x[:, 1::2]), 2, axis=1)
    eps = (2.0 ** -8 if dtype == "bf16" else 2.0 ** -24) + 2 * 2.0 ** -24
    assert (np.abs(f64(got)[:cfg.n_video] - want) <= eps * size).all()
    keep_idx, assign, q_c, k_c, v_c = vorta.vorta_bcs_select_pool(plan, q, k, v, cfg.fixed_routes)
    for one, src in ((q_c, q), (k_c, k)):
        assert torch.equal(one, vorta.vorta_bcs_pool(plan, src, cfg.fixed_routes, keep_idx, assign, rotate=True))
