"""The fp32 kernels at the edges of their tiles and of their split over waves,
against the fp64 oracle: one row, one 32-row tile and its neighbours, fewer and more
tiles than waves, and both splits of the tiles over waves (more than 512 row blocks
take the coarser one), prefix and fixed gates, forward and backward.

Tolerance: the fp32 bars of the parity tests (max-abs 1e-4 on O and LSE, relative L2
1e-4 on gradients).  A sum of d = 128 products and a softmax over L <= 600 keys in
fp32 is within a few 1e-6 of exact at these magnitudes (measured 2e-6 and 4e-6)."""
import pytest
import torch

import oracle
import paper_2503_02130_amd as fox
from paper_2503_02130_amd import inputs
from test_parity_gpu import check_fwd, check_grad, cpu

pytestmark = pytest.mark.gpu

# (B, H, L): 1 to 19 row blocks with the finer split; 35 rows x 17 blocks = 595 and
# 40 x 13 = 520 workgroups with the coarser one
SHAPES = [(1, 2, 1), (1, 2, 32), (1, 3, 33), (2, 1, 64), (1, 2, 130), (1, 1, 257), (1, 1, 600),
          (5, 7, 513), (4, 10, 416)]


@pytest.mark.parametrize("fixed", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,H,L", SHAPES)
def test_f32_forward_backward(B, H, L, d, fixed):
    x = inputs.attn_inputs(B, H, L, d, "f32", ("normal", 2.0, 1.0), 31 * L + d, device="cuda:0")
    s = fox.default_scale(d)
    xc = cpu(x)
    if fixed:
        b = fox.fox_fixed_gate_init(H, 2.0, 64.0)
        g = b.to("cuda:0")
        o, lse = fox.fox_attn_fwd_fixed_gate(x["q"], x["k"], x["v"], g, s)
        got = fox.fox_attn_bwd_fixed_gate(x["q"], x["k"], x["v"], g, o, lse, x["do"], s)[:3]
        O, LSE = oracle.forward_fixed_gate(xc["q"], xc["k"], xc["v"], b, s)
        ref = oracle.backward_fixed_gate(xc["q"], xc["k"], xc["v"], b, xc["do"], s)[:3]
    else:
        c = fox.fox_gate_prefix(x["logit"])
        o, lse = fox.fox_attn_fwd(x["q"], x["k"], x["v"], c, s)
        got = fox.fox_attn_bwd(x["q"], x["k"], x["v"], c, o, lse, x["do"], s)
        O, LSE = oracle.forward(xc["q"], xc["k"], xc["v"], xc["logit"], s)
        ref = oracle.backward(xc["q"], xc["k"], xc["v"], xc["logit"], xc["do"], s)
    torch.cuda.synchronize()
    check_fwd("f32", o, lse, O, LSE, f"L={L}")
    for name, a, r in zip(("dQ", "dK", "dV", "dlogf"), got, ref):
        check_grad("f32", name, a, r, f"L={L}")


@pytest.mark.parametrize("fixed", [False, True])
def test_f32_more_row_blocks_than_workgroups(fixed):
    """Past 2^22 row blocks a workgroup walks several, in the same LDS: B H = 2^21 + 8 rows
    of two blocks, whose last 16 blocks are second ones of their workgroups (two of its
    four waves have no tile there and run ahead of the others).  Rows are independent and
    both calls split the tiles alike, so the rows these blocks belong to must have the bits
    of a call on them alone."""
    BH, L, d = (1 << 21) + 8, 33, 64
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 100 GB of free GPU memory")
    gen = torch.Generator("cuda:0").manual_seed(1)

    def rand(*shape):
        return torch.randn(shape, device="cuda:0", generator=gen)

    x, logit, delta, bias = rand(1, BH, L, d), rand(1, BH, L), rand(1, BH, L), rand(BH)
    tail = slice(BH - 32, BH)
    part = tuple(t[:, tail].clone() for t in (x, logit, delta)) + (bias[tail].clone(),)

    def run(x, logit, delta, bias):
        """The results' last 32 rows; each large one is dropped before the next is made."""
        s, out = fox.default_scale(d), []

        def keep(r):
            out.extend(t[:, -32:].clone() for t in r)

        if fixed:
            o, lse = fox.fox_attn_fwd_fixed_gate(x, x, x, bias, s)
            keep((o, lse))
            keep(fox.fox_attn_bwd_fixed_gate(x, x, x, bias, o, lse, x, s)[:3])
            return out
        c = fox.fox_gate_prefix(logit)
        o, lse = fox.fox_attn_fwd(x, x, x, c, s)
        keep((o, lse))
        del o
        keep(fox.fox_attn_bwd_dkdv(x, x, x, c, lse, x, delta, s))
        keep(fox.fox_attn_bwd_dq(x, x, x, c, lse, x, delta, s))
        return out

    whole = run(x, logit, delta, bias)
    del x, logit, delta
    torch.cuda.empty_cache()
    for i, (w, one) in enumerate(zip(whole, run(*part))):
        assert bool(torch.isfinite(one).all()) and torch.equal(w, one), f"output {i}"
