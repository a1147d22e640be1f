"""The one-pass selection and merge at the edges of its instances (buckets of 12, 16 and 32 tokens, rows of
16 and 32 chunks) against the separate passes, bit for bit, and the oracle's index sets; odd grids, so
that the last bucket of each axis is clipped, and text rows that fill no workgroup."""
import numpy as np
import pytest
import torch

import paper_2505_18809_amd as vorta
from oracle import vorta_oracle as vo
from synth_inputs import LayerConfig, make_qkv
from helpers import f64

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
