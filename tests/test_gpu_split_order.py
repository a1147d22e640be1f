"""Split launches of more items than CUs and fewer than twice as many: the items of the first round come in another
order.  Every row of every head against the fp64 oracle, just inside and just outside that range for 256 CUs."""
import numpy as np
import pytest
import torch

import paper_2505_18809_amd as vorta
from oracle import vorta_oracle as vo
from synth_inputs import LayerConfig, make_qkv
from helpers import SPLIT2, f64, force_form, spec_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,heads,items", [((1, 8, 16), 128, 256), ((3, 8, 8), 86, 258), ((5, 8, 8), 102, 510), ((4, 8, 8), 128, 512)])
def test_every_item_is_computed_once(grid, heads, items):
    assert heads * (-(-int(np.prod(grid)) // 64)) == items
    # full heads in front; core-set heads whose tokens are all kept have as many items of the same rows
    routes = tuple([0] * (heads // 3) + [1] * (heads // 3) + [2] * (heads - 2 * (heads // 3)))
    cfg = LayerConfig(f"order{items}", grid, heads, 128, "bf16", (1, 8, 8), (1, 1, 1), seed=83, keep_num=1, keep_den=1,
                      fixed_routes=routes)
    print(cfg.name, flush=True)
    q, k, v = make_qkv(cfg, "cuda")
    out = torch.full_like(q, float("nan"))
    vorta.vorta_routed_attention_layer(force_form(vorta.plan_for(cfg), SPLIT2), q, k, v, routes, out=out)
    torch.cuda.synchronize()
    for h, r in enumerate(routes):
        want = vo.head_attention(r, f64(q[h]), f64(k[h]), f64(v[h]), spec_of(cfg), None)
        err = np.abs(f64(out[h]) - want).max()
        assert err <= 2e-2, f"head {h} route {r}: {err:.3e}"
