"""The bf16 dQ kernel with the key tiles split over wave groups (short grids with long
rows): one tile below the rule's line and at it (8 key tiles), tile counts with each
remainder over the groups, ragged last tiles that leave waves without queries; prefix
and fixed gates against the fp64 oracle, skipping bit for bit against dense, and
d(log f)_1 = sum of all dc near zero (dc^q and dc^k stay the row and column sums of one
matrix).

Tolerance: the bf16 gradient bar of the parity tests (relative L2 2e-2); the split
changes only the order of fp32 sums."""
import pytest
import torch

import oracle
import paper_2503_02130_amd as fox
from paper_2503_02130_amd import inputs
from test_parity_gpu import check_grad, cpu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L", [448, 449, 512, 575, 577, 641, 1090])
def test_split_dq(d, L):
    B, H = 1, 3
    x = inputs.attn_inputs(B, H, L, d, "bf16", ("head_mean_uniform", -1.0, 5.0, 1.0), 3 * L + d,
                           device=DEV)
    q, k, v, do = x["q"], x["k"], x["v"], x["do"]
    s = fox.default_scale(d)
    xc = cpu(x)
    c = fox.fox_gate_prefix(x["logit"])
    o, lse = fox.fox_attn_fwd(q, k, v, c, s)
    bias = fox.fox_fixed_gate_init(H, 2.0, 400.0)
    g = bias.to(DEV)
    of, lsef = fox.fox_attn_fwd_fixed_gate(q, k, v, g, s)
    got = fox.fox_attn_bwd(q, k, v, c, o, lse, do, s)
    gotf = fox.fox_attn_bwd_fixed_gate(q, k, v, g, of, lsef, do, s)
    qn, kn = fox.fox_row_norm_max(q), fox.fox_row_norm_max(k)
    skip = fox.fox_attn_bwd_skip(q, k, v, c, o, lse, do, qn, kn, s)
    skipf = fox.fox_attn_bwd_fixed_gate_skip(q, k, v, g, of, lsef, do, qn, kn, s)
    torch.cuda.synchronize()
    for a, b in zip((*got, *gotf), (*skip, *skipf)):
        assert torch.equal(a, b)
    ref = oracle.backward(xc["q"], xc["k"], xc["v"], xc["logit"], xc["do"], s)
    for name, a, r in zip(("dQ", "dK", "dV", "dlogf"), got, ref):
        check_grad("bf16", name, a, r, f"L={L}")
    assert float(got[3][..., 0].abs().max()) <= 1e-4 * max(1.0, float(ref[3].abs().max()))
    ref = oracle.backward_fixed_gate(xc["q"], xc["k"], xc["v"], bias, xc["do"], s)
    for name, a, r in zip(("dQ", "dK", "dV"), gotf, ref):
        check_grad("bf16", name, a, r, f"fixed L={L}")
