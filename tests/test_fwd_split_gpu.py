"""The bf16 forward with the keys of a row block split over wave groups (short grids
with long rows), at the edges of that rule and of the tiles: one tile below and at the
splits' limits (12 and 24 key tiles at d = 64, 16 at d = 128), ragged last tiles that
leave waves without queries, odd and even tile counts.  Every form of the kernel:
prefix and fixed gates against the fp64 oracle, the fused output norm and gate against
the standalone one, skipping bit for bit against dense.

Tolerance: the bf16 bars of the parity tests (relative L2 1e-2 on O, max-abs 1e-2 on
LSE); the split changes only the order of fp32 sums."""
import pytest
import torch

import oracle
import paper_2503_02130_amd as fox
from paper_2503_02130_amd import inputs
from test_parity_gpu import check_fwd, cpu, rel_l2

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CASES = ([(64, L) for L in (704, 705, 770, 833, 1472, 1473, 1540, 1601, 1665)] +
         [(128, L) for L in (960, 961, 1025, 1090, 1217)])


@pytest.mark.parametrize("d,L", CASES)
def test_split_forward(d, L):
    B, H = 1, 3
    x = inputs.attn_inputs(B, H, L, d, "bf16", ("head_mean_uniform", -1.0, 5.0, 1.0), 7 * L + d,
                           device=DEV)
    q, k, v = x["q"], x["k"], x["v"]
    s = fox.default_scale(d)
    xc = cpu(x)
    c = fox.fox_gate_prefix(x["logit"])
    o, lse = fox.fox_attn_fwd(q, k, v, c, s)
    bias = fox.fox_fixed_gate_init(H, 2.0, 400.0)
    of, lsef = fox.fox_attn_fwd_fixed_gate(q, k, v, bias.to(DEV), s)
    torch.cuda.synchronize()
    check_fwd("bf16", o, lse, *oracle.forward(xc["q"], xc["k"], xc["v"], xc["logit"], s), f"L={L}")
    check_fwd("bf16", of, lsef, *oracle.forward_fixed_gate(xc["q"], xc["k"], xc["v"], bias, s),
              f"fixed L={L}")
    qn, kn = fox.fox_row_norm_max(q), fox.fox_row_norm_max(k)
    for a, b in ((fox.fox_attn_fwd_skip(q, k, v, c, qn, kn, s), (o, lse)),
                 (fox.fox_attn_fwd_fixed_gate_skip(q, k, v, bias.to(DEV), qn, kn, s), (of, lsef))):
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    wo = 1.0 + 0.1 * torch.randn((H, d), device=DEV, generator=torch.Generator(DEV).manual_seed(L))
    y, op, lsep = fox.fox_attn_fwd_pro(q, k, v, c, x["do"], wo, s)
    assert torch.equal(op, o) and torch.equal(lsep, lse)
    # two bf16 roundings of one fp32 value formed in different orders
    assert rel_l2(y, fox.fox_pro_output_gate(o, x["do"], wo)) <= 1e-3


@pytest.mark.parametrize("d,B,H,L", [(128, 1, 16, 3001), (64, 1, 16, 3001)])
def test_split_skipping_ends_whatever_the_norms_do(d, B, H, L):
    """The norms change in memory while the skipping forward runs: what it then computes is
    nobody's business, but every wave group must leave its tile loop as one (a wave that
    stayed alone would wait for ever), and the next call is right again."""
    x = inputs.attn_inputs(B, H, L, d, "bf16", ("normal", 2.0, 1.0), L, device=DEV)
    q, k, v = x["q"], x["k"], x["v"]
    c = fox.fox_gate_prefix(x["logit"])
    qn, kn = fox.fox_row_norm_max(q), fox.fox_row_norm_max(k)
    moving, other = kn.clone(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for i in range(20):
        with torch.cuda.stream(other):
            for j in range(20):
                moving.fill_(100.0 * (j % 2))
        fox.fox_attn_fwd_skip(q, k, v, c, qn, moving)
    torch.cuda.synchronize()
    for a, b in zip(fox.fox_attn_fwd_skip(q, k, v, c, qn, kn), fox.fox_attn_fwd(q, k, v, c)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("BH,L", [(24, 1500), (32, 1500), (32, 2048)])
def test_pro_split_line(BH, L):
    """fox_attn_fwd_pro at d = 128 on both sides of its own line (288 workgroups of up to 24
    key tiles split; 384 of 24 and 512 of 32 not, where the plain forward splits): o and
    lse agree with fox_attn_fwd's within two bf16 roundings of sums in different orders."""
    x = inputs.attn_inputs(1, BH, L, 128, "bf16", ("normal", 3.0, 1.0), L, device=DEV, grad=True)
    q, k, v, g = x["q"], x["k"], x["v"], x["do"]
    c = fox.fox_gate_prefix(x["logit"])
    wo = torch.ones((BH, 128), device=DEV)
    o, lse = fox.fox_attn_fwd(q, k, v, c)
    y, op, lsep = fox.fox_attn_fwd_pro(q, k, v, c, g, wo)
    assert rel_l2(op, o) <= 1e-3 and float((lsep - lse).abs().max()) <= 1e-4
    assert rel_l2(y, fox.fox_pro_output_gate(op, g, wo)) <= 1e-3
