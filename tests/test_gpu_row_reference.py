"""Window rows whose weight is nearly all on one late key: probabilities are rounded to bf16 and row sums are not, so that
key's probability has to be exactly 1, which takes its own score for the row reference."""
import numpy as np
import pytest
import torch

import paper_2505_18809_amd as vorta
from oracle import vorta_oracle as vo
from synth_inputs import LayerConfig
from helpers import PIPE, PIPE_WIN_128, SPLIT2, SPLIT4, f64, force_form, spec_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", [SPLIT2, SPLIT4, PIPE, PIPE_WIN_128])
def test_a_late_key_that_dominates_is_not_rounded(form):
    # Key set of the last tiles: 12 x 12 x 12 tokens.  Its first eight keys score 8 a, its last one 12.3 a, with
    # a = 0.9 .. 1.1 by row: 48 to 113 times a key of the first block, 0.8 of the row's weight or more.
    cfg = LayerConfig("late_key", (12, 16, 16), 4, 128, "bf16", (4, 4, 4), (3, 3, 3), seed=97, fixed_routes=(1,) * 4)
    g = torch.Generator().manual_seed(cfg.seed)
    q, k, v = (torch.randn(4, cfg.n_tokens, 128, generator=g) for _ in range(3))
    token = np.arange(cfg.n_tokens).reshape(cfg.grid)
    rows, early, late = token[:, 8:, 8:].reshape(-1), token[0, 4, 4:12], token[-1, -1, -1]
    u = torch.nn.functional.normalize(torch.randn(128, generator=g), dim=0)
    k *= 0.4
    q[:, rows] = (0.9 + 0.2 * torch.rand(4, len(rows), 1, generator=g)) * u * 128 ** 0.5 + 0.5 * q[:, rows]
    k[:, early], k[:, late] = 8.0 * u, 12.3 * u
    v[:, late] = (4 + 4 * torch.rand(4, 128, generator=g)) * torch.randn(4, 128, generator=g).sign()
    q, k, v = (x.to("cuda", torch.bfloat16) for x in (q, k, v))
    out = vorta.vorta_routed_attention_layer(force_form(vorta.plan_for(cfg), form), q, k, v, cfg.fixed_routes)
    torch.cuda.synchronize()
    scale = []
    for h in range(4):
        want = vo.head_attention(1, f64(q[h]), f64(k[h]), f64(v[h]), spec_of(cfg), rows)
        got = f64(out[h])[rows]
        assert np.abs(got - want).max() <= 2.0 ** -8 * np.abs(want).max() + 8e-3     # half a bf16 step and the other keys'
        scale.append((got * want).sum(1) / (want * want).sum(1) - 1)
    # Factor by which a row as a whole is off.  Rounding the output: 2^-9 to 2^-8 of an entry, a half step uniform over its
    # range, mean over 128 entries: 2^-8 * 0.72 / sqrt(3) / sqrt(128) = 1.5e-4 rms; the other keys' probabilities, 0.2 of the
    # weight on eight keys: 0.2 * 1.5e-3 / sqrt(3) / sqrt(8) = 6e-5.  A rounded probability of the late key adds 8e-4.
    rms = np.sqrt(np.mean(np.square(scale)))
    print(f"form {form}: rms {rms:.2e}", flush=True)
    assert rms <= 2.5e-4
