"""The d = 64 key-side backward with 32-row query tiles (grids above its line) against
the same kernel with 64-row tiles (grids below it): one batch row of a large call has
the bits of a call on that row alone, for lengths whose last 64-query tile holds one or
two 32-row tiles, dense, fixed-gate and skipping, recomputing and keeping dS (whose
slots hold 64 queries; its workspace starts as NaN patterns).  Both sum over the queries
in the same order, so nothing may differ."""
import pytest
import torch

import paper_2503_02130_amd as fox
from paper_2503_02130_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# B H ceil(L / 128) workgroups: 520, 525, 546, 600 for the call, at most 45 for one row
@pytest.mark.parametrize("B,H,L", [(65, 8, 33), (35, 5, 289), (26, 7, 352), (24, 5, 577)])
def test_query_tiles_give_the_same_bits(B, H, L):
    d, s = 64, fox.default_scale(64)
    x = inputs.attn_inputs(B, H, L, d, "bf16", ("head_mean_uniform", -2.0, 4.0, 1.0), L, device=DEV)
    bias = fox.fox_fixed_gate_init(H, 2.0, 100.0).to(DEV)
    c = fox.fox_gate_prefix(x["logit"])
    o, lse = fox.fox_attn_fwd(x["q"], x["k"], x["v"], c, s)
    of, lsef = fox.fox_attn_fwd_fixed_gate(x["q"], x["k"], x["v"], bias, s)
    qn, kn = fox.fox_row_norm_max(x["q"]), fox.fox_row_norm_max(x["k"])

    def backwards(b):
        """dk, dv of batch rows b of every backward, and of those keeping dS all outputs
        (the recomputing dQ kernel orders its sums by a rule of its own)."""
        q, k, v, do = (x[n][b].clone() for n in ("q", "k", "v", "do"))
        cc, oo, ll, qq, kk, ofb, lfb = (t[b].clone() for t in (c, o, lse, qn, kn, of, lsef))
        shape = (torch.bfloat16, q.shape[0], H, L, d)

        def nans(size):  # whatever the dQ pass reads must have been written
            return torch.full((size,), 0xFF, dtype=torch.uint8, device=DEV)

        ws = fox.fox_attn_bwd_stored_workspace_bytes(*shape)
        wf = fox.fox_attn_bwd_fixed_gate_stored_workspace_bytes(*shape)
        out = [fox.fox_attn_bwd(q, k, v, cc, oo, ll, do, s)[1:3],
               fox.fox_attn_bwd_stored(q, k, v, cc, oo, ll, do, s, workspace=nans(ws)),
               fox.fox_attn_bwd_skip(q, k, v, cc, oo, ll, do, qq, kk, s)[1:3],
               fox.fox_attn_bwd_skip_stored(q, k, v, cc, oo, ll, do, qq, kk, s,
                                            workspace=nans(ws)),
               fox.fox_attn_bwd_fixed_gate(q, k, v, bias, ofb, lfb, do, s)[1:3],
               fox.fox_attn_bwd_fixed_gate_skip_stored(q, k, v, bias, ofb, lfb, do, qq, kk, s,
                                                       workspace=nans(wf))[:3]]
        return [t for r in out for t in r]

    whole = backwards(slice(0, B))
    for b in (0, B - 1):
        for i, (w, one) in enumerate(zip(whole, backwards(slice(b, b + 1)))):
            assert torch.equal(w[b:b + 1], one), f"L={L} row {b} output {i}"
