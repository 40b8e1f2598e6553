"""The decode step at the edges of its split of the keys: one launch without a split (64
KB of keys a head, 256 heads) and just past it, each finer split's limits (768
workgroups, 256 splits of a sequence), against the fp64 oracle; skipping bit for bit
against dense; the allocation-free form bit for bit.

Tolerance: the decode bars of the parity tests (bf16 relative L2 1e-2 on o, fp32 1e-4
max-abs; LSE 1e-2 and, fp32, 1e-4 plus the rounding of the stored prefix values)."""
import pytest
import torch

import oracle
import paper_2503_02130_amd as fox
from paper_2503_02130_amd import inputs
from test_parity_gpu import check_fwd, cpu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CASES = ([("bf16", 128, 1, 3, T) for T in (2, 31, 32, 33, 500, 8192, 8193)] +
         [("bf16", 64, 2, 2, T) for T in (97, 16384, 16385)] +
         [("bf16", 64, 4, 12, 4099), ("bf16", 128, 3, 16, 4096), ("bf16", 128, 3, 16, 4097)] +
         [("f32", 64, 1, 2, 1000), ("f32", 128, 2, 12, 1025)] +
         # direct and, one key or head more, split
         [("bf16", 128, 1, 2, 256), ("bf16", 128, 1, 2, 257), ("bf16", 64, 1, 2, 512),
          ("bf16", 64, 1, 2, 513), ("f32", 128, 1, 2, 128), ("f32", 128, 1, 2, 129),
          ("f32", 64, 2, 2, 255), ("bf16", 128, 16, 16, 40), ("bf16", 128, 257, 1, 40),
         # many heads: one pass of a workgroup's loads is one split, a key more two
         ("bf16", 64, 257, 1, 128), ("bf16", 64, 257, 1, 129), ("f32", 128, 129, 2, 65)])


@pytest.mark.parametrize("dtype,d,B,H,T", CASES)
def test_decode_splits(dtype, d, B, H, T):
    x = inputs.decode_inputs(B, H, T, d, dtype, ("normal", 3.0, 1.0), T + d, device=DEV)
    c0 = torch.zeros((B, H, T), device=DEV)
    c0[..., :T - 1] = fox.fox_gate_prefix(x["cached_logit"])
    c0[..., T - 1] = float("nan")  # written, never read
    args = (x["q"], x["k_cache"], x["v_cache"])
    c, cs, cn = c0.clone(), c0.clone(), c0.clone()
    o, lse = fox.fox_attn_decode(*args, c, x["logit_new"])
    kn = fox.fox_row_norm_max(x["k_cache"])
    os_, lses = fox.fox_attn_decode_skip(*args, cs, x["logit_new"], kn)
    on, lsen = fox.fox_attn_decode_noalloc(*args, cn, x["logit_new"])
    torch.cuda.synchronize()
    for a, b, w in ((os_, lses, cs), (on, lsen, cn)):
        assert torch.equal(a, o) and torch.equal(b, lse) and torch.equal(w, c)
    xc = cpu(x)
    O, LSE, cT = oracle.decode(xc["q"], xc["k_cache"], xc["v_cache"], xc["cached_logit"],
                               xc["logit_new"], fox.default_scale(d))
    check_fwd(dtype, o, lse, O, LSE, f"T={T}", c_abs=float(cT.abs().max()), L=T)
    assert torch.equal(c[..., :T - 1], c0[..., :T - 1])


@pytest.mark.parametrize("B,H,T,Tmax", [(1, 2, 8193, 8193), (1, 3, 500, 9000), (2, 8, 6000, 8192),
                                        (2, 8, 4097, 4097), (1, 16, 47 * 128, 48 * 128),
                                        (8, 16, 7600, 8192)])  # 256 keys a split, and 512
def test_decode_other_workspaces(B, H, T, Tmax):
    """The workspace of 256-key splits alone (coarser splits: the oracle bars; bytes past
    it untouched), and one sized for a longer cache (the same splits, bit for bit)."""
    d = 128
    x = inputs.decode_inputs(B, H, T, d, "bf16", ("normal", 3.0, 1.0), T + H, device=DEV)
    c = torch.zeros((B, H, T), device=DEV)
    c[..., :T - 1] = fox.fox_gate_prefix(x["cached_logit"])
    args = (x["q"], x["k_cache"], x["v_cache"], c, x["logit_new"])
    o, lse = fox.fox_attn_decode(*args)
    need = fox.fox_attn_decode_workspace_bytes(torch.bfloat16, B, H, Tmax, d)
    assert need >= fox.fox_attn_decode_workspace_bytes(torch.bfloat16, B, H, T, d)
    ol, lsel = fox.fox_attn_decode(*args, workspace=torch.empty(need, dtype=torch.uint8,
                                                                device=DEV))
    assert torch.equal(ol, o) and torch.equal(lsel, lse)
    least = B * H * -(-T // 256) * (d + 2) * 4
    room = torch.full((least + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    os_, lses = fox.fox_attn_decode(*args, workspace=room[:least])
    assert bool((room[least:] == 0xA5).all())
    with pytest.raises(fox.FoxError):
        fox.fox_attn_decode(*args, workspace=room[:least - 4])
    xc = cpu(x)
    O, LSE, cT = oracle.decode(xc["q"], xc["k_cache"], xc["v_cache"], xc["cached_logit"],
                               xc["logit_new"], fox.default_scale(d))
    check_fwd("bf16", os_, lses, O, LSE, f"T={T}", c_abs=float(cT.abs().max()), L=T)


@pytest.mark.parametrize("dtype,d,B,H,T", [("bf16", 64, 2, 3, 513), ("bf16", 64, 1, 2, 769),
                                           ("bf16", 128, 1, 3, 321), ("f32", 64, 1, 2, 257),
                                           ("f32", 128, 1, 2, 129), ("bf16", 64, 257, 1, 129)])
def test_fixed_gate_decode_splits(dtype, d, B, H, T):
    """Fixed gates, whose splits keep one pass of a workgroup's loads: last splits of one
    key, against the oracle with the bias as every token's logit; skipping bit for bit."""
    x = inputs.decode_inputs(B, H, T, d, dtype, ("normal", 3.0, 1.0), T + d, device=DEV)
    b = fox.fox_fixed_gate_init(H, 2.0, 400.0) if H > 1 else torch.tensor([3.0])
    args, g = (x["q"], x["k_cache"], x["v_cache"]), b.to(DEV)
    o, lse = fox.fox_attn_decode_fixed_gate(*args, g)
    kn = fox.fox_row_norm_max(x["k_cache"])
    os_, lses = fox.fox_attn_decode_fixed_gate_skip(*args, g, kn)
    assert torch.equal(os_, o) and torch.equal(lses, lse)
    xc = cpu(x)
    O, LSE, cT = oracle.decode(xc["q"], xc["k_cache"], xc["v_cache"],
                               b[None, :, None].expand(B, H, T - 1), b[None].expand(B, H),
                               fox.default_scale(d))
    check_fwd(dtype, o, lse, O, LSE, f"T={T}", c_abs=float(cT.abs().max()), L=T)


def test_decode_rounding():
    """The running sum's rounding, acc <- fma(alpha, acc, rn(p v)) for the first key of a
    pass of the loads and fma(p, v, acc) for the others, checked bit for bit on two passes
    of one lane group: q = 0 and prefix values that make p = 1 and alpha = 2^-x, so that o
    follows from v, alpha and fp32 arithmetic.  alpha itself is the hardware's exponential:
    some value within 2 ulp must explain every element."""
    H, T, d = 768, 128, 64  # no direct launch, one split, two passes of 4 x 16 keys
    g = torch.Generator(DEV).manual_seed(3)
    k = torch.randn((1, H, T, d), device=DEV, generator=g)
    v = torch.zeros_like(k)
    v[:, :, ::16] = torch.randn((1, H, 8, d), device=DEV, generator=g)  # lane group 0's keys
    c = torch.zeros((1, H, T), device=DEV)
    c[..., :64] = 0.4375
    o, _ = fox.fox_attn_decode(torch.zeros((1, H, d), device=DEV), k, v, c,
                               torch.full((1, H), 100.0, device=DEV))
    x = torch.tensor(0.4375) * torch.tensor(1.4426950408889634)  # the score, as the kernel has it
    vs, f32 = v[0, :, ::16].cpu(), torch.float32
    first = ((vs[:, 0] + vs[:, 1]) + vs[:, 2]) + vs[:, 3]
    mismatches = []
    for ulp in range(-2, 3):
        alpha = torch.exp2(-x.double()).to(f32)
        alpha = (alpha.view(torch.int32) + ulp).view(f32)
        acc = (alpha.double() * first.double() + vs[:, 4].double()).to(f32)
        for u in (5, 6, 7):
            acc = acc + vs[:, u]
        l = (alpha.double() * 4 + 1).to(f32) + 1 + 1 + 1
        total = torch.zeros((), dtype=f32)
        for _ in range(16):  # the lane groups' equal sums
            total = total + l
        mismatches.append(int((acc / total != o[0].cpu()).sum()))
    assert min(mismatches) == 0, mismatches
