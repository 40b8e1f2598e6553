"""The forward's and the recomputing dQ's workgroup order where the second 256 workgroups
run in reverse: 256 workgroups and one more, a second pass that is no multiple of eight,
a full one, the last grid that is reordered (2048) and the first that is not.  A block
computed twice or not at all shows against the skipping kernels, which keep their order and
give the same bits; outputs start as NaN."""
import pytest
import torch

import paper_2503_02130_amd as fox
from paper_2503_02130_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("BH,L", [(256, 128), (257, 65), (90, 300), (261, 200), (171, 380),
                                  (205, 640), (256, 1024), (293, 800)])
def test_paired_order(d, BH, L):
    x = inputs.attn_inputs(1, BH, L, d, "bf16", ("normal", 2.0, 1.0), L + d, device="cuda:0")
    q, k, v = x["q"], x["k"], x["v"]
    do = torch.randn(q.shape, generator=torch.Generator("cuda").manual_seed(L), device=q.device)
    do = do.to(q.dtype)
    c = fox.fox_gate_prefix(x["logit"])
    qn, kn = fox.fox_row_norm_max(q), fox.fox_row_norm_max(k)
    o, lse = torch.full_like(q, float("nan")), torch.full_like(c, float("nan"))
    fox.fox_attn_fwd(q, k, v, c, o=o, lse=lse)
    os_, lses = fox.fox_attn_fwd_skip(q, k, v, c, qn, kn)
    assert torch.equal(o, os_) and torch.equal(lse, lses)
    got = fox.fox_attn_bwd(q, k, v, c, o, lse, do)
    ref = fox.fox_attn_bwd_skip(q, k, v, c, o, lse, do, qn, kn)
    for a, b in zip(got, ref):
        assert torch.isfinite(a).all() and torch.equal(a, b)
