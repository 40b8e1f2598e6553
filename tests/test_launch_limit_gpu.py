"""The largest accepted count of (batch, head) rows, B H = 2^22: kernels of 1024 threads
pass the 2^32 threads a launch takes there and run in two parts, the second holding the
last row.  Rows are independent, so the last rows must have the bits of a call on them
alone; outputs start as NaN where the caller can bring them."""
import pytest
import torch

import paper_2503_02130_amd as fox

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
N = 1 << 22
B = H = 1 << 11
D = 64


def _randn(*shape, seed, dtype=torch.float32):
    return torch.randn(shape, generator=torch.Generator(DEV).manual_seed(seed), device=DEV,
                       dtype=dtype)


def _nan(*shape, dtype=torch.float32):
    return torch.full(shape, float("nan"), device=DEV, dtype=dtype)


@pytest.mark.parametrize("L", [1, 4])
def test_scans(L):
    x, a, b = (_randn(B, H, L, seed=i) for i in range(3))
    c = fox.fox_gate_prefix(x, c=_nan(B, H, L))
    g, lf = fox.fox_dlogit_from_dc(a, b, x), fox.fox_dlogf_from_dc(a, b)
    last = slice(B - 1, B)
    xs, as_, bs = (t[last].clone() for t in (x, a, b))
    assert torch.equal(c[last], fox.fox_gate_prefix(xs))
    assert torch.equal(g[last], fox.fox_dlogit_from_dc(as_, bs, xs))
    assert torch.equal(lf[last], fox.fox_dlogf_from_dc(as_, bs))
    assert bool(torch.isfinite(c).all())


def test_row_norms():
    x = _randn(B, H, 1, D, seed=4, dtype=torch.bfloat16)
    got = fox.fox_row_norm_max(x)
    assert torch.equal(got[B - 1:], fox.fox_row_norm_max(x[B - 1:].clone()))
    assert float(got.min()) > 0


def test_pro_row_passes():
    bf = torch.bfloat16
    raw = [_randn(B, H, 1, D, seed=i, dtype=bf) for i in range(3)]
    shifts = [_randn(B, H, 1, seed=10 + i) for i in range(2)]
    w = [_randn(H, D, seed=20 + i) for i in range(3)]
    out = [_nan(B, H, 1, D, dtype=bf) for _ in range(4)]
    fox.fox_pro_prologue(*raw, *shifts, *w[:2], q=out[0], k=out[1], v=out[2])
    fox.fox_pro_output_gate(raw[0], raw[1], w[2], y=out[3])
    one = [t[B - 1:].clone() for t in raw + shifts]
    ref = fox.fox_pro_prologue(*one, *w[:2]) + (fox.fox_pro_output_gate(one[0], one[1], w[2]),)
    for o, r in zip(out, ref):
        assert torch.equal(o[B - 1:], r) and bool(torch.isfinite(o).all())


def test_fixed_gate_bias_gradient():
    """One head per (batch, head) row: its bias gradients are 2^22 workgroups."""
    q, k, v, do = (_randn(1, N, 2, D, seed=30 + i, dtype=torch.bfloat16) for i in range(4))
    bias = _randn(N, seed=40)

    def grad(h):
        a = [t[:, h].clone() for t in (q, k, v)]
        o, lse = fox.fox_attn_fwd_fixed_gate(*a, bias[h].clone())
        return fox.fox_attn_bwd_fixed_gate(*a, bias[h].clone(), o, lse, do[:, h].clone())[-1]

    whole = grad(slice(0, N))
    assert torch.equal(whole[N - 64:], grad(slice(N - 64, N)))
    assert bool(torch.isfinite(whole).all()) and int((whole[:64] == 0).sum()) < 8
