"""The Pro prologue's bits do not depend on its launch shape.  The token shift is
fma(m, x_{t-1}, rn((1 - m) x_t)): the value shift is checked against that expression, and
the backward's elementwise gradients of one batch row alone (512 threads a workgroup)
against the same rows in a grid of more than 256 workgroups (256 threads)."""
import pytest
import torch

import paper_2503_02130_amd as fox
from paper_2503_02130_amd import inputs

pytestmark = pytest.mark.gpu
EPS = 1e-6
DEV = "cuda:0"
NAMES = ("q_raw", "k_raw", "v_raw", "k_shift", "v_shift", "wq", "wk")


def _gates(x):
    """sigmoid(v_shift) and 1 - sigmoid(v_shift) as the kernel forms them: the fp32 value
    shift of a row of ones after a row of zeros, and the other way round."""
    B, H, L = x["v_shift"].shape
    t = torch.arange(L, device=DEV)[None, None, :, None].expand(B, H, L, 64)
    z = torch.zeros((B, H, L, 64), device=DEV)
    w = torch.ones((H, 64), device=DEV)

    def shift(v):
        return fox.fox_pro_prologue(z, z, v, x["k_shift"], x["v_shift"], w, w, eps=EPS)[2][..., 0]

    even, odd = (shift((t % 2 == p).float().contiguous()) for p in (0, 1))
    first = torch.arange(L, device=DEV) % 2 == 0  # rows t whose own value is 1 in `even`
    return torch.where(first, odd, even), torch.where(first, even, odd)


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
def test_value_shift_rounding(dtype, d):
    x = inputs.pro_inputs(2, 4, 2001, d, dtype, ("normal", 2.0, 1.0), d, device=DEV)
    v = fox.fox_pro_prologue(*(x[n] for n in NAMES), eps=EPS)[2]
    m, m1 = (t.double()[..., None] for t in _gates(x))
    xv = x["v_raw"].double()
    pv = torch.nn.functional.pad(xv, (0, 0, 1, 0))[:, :, :-1]
    # both products of two fp32 values are exact in 64 bits; the sum's own rounding to 64
    # bits moves an fp32 result with a chance below 2^-27 per element
    ref = (m * pv + (m1 * xv).float().double()).float().to(v.dtype)
    wrong = int((ref != v).sum())
    assert wrong <= (0 if dtype == "bf16" else 1), f"{wrong} of {v.numel()} elements"


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 128])
def test_forward_bits_alone_and_in_a_batch(dtype, d):
    B, H, L = 100, 16, 20  # 1600 workgroups of 256 threads; 16 of 1024 alone
    x = inputs.pro_inputs(B, H, L, d, dtype, ("normal", 2.0, 1.0), 5 * d, device=DEV)

    def outs(b):
        a = [x[n] if n in ("wq", "wk") else x[n][b].clone() for n in NAMES]
        return fox.fox_pro_prologue(*a, eps=EPS) + (
            fox.fox_pro_output_gate(a[0], x["g"][b].clone(), x["wo"], eps=EPS),)

    whole = outs(slice(0, B))
    for b in (0, B - 1):
        for i, (w, one) in enumerate(zip(whole, outs(slice(b, b + 1)))):
            assert torch.equal(w[b:b + 1], one), f"row {b} output {i}"


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 128])
def test_backward_bits_alone_and_in_a_batch(dtype, d):
    B, H, L = 20, 8, 300  # 320 workgroups; 16 alone
    x = inputs.pro_inputs(B, H, L, d, dtype, ("normal", 2.0, 1.0), 3 * d, device=DEV)

    def grads(b):
        a = [x[n] if n in ("wq", "wk") else x[n][b].clone() for n in NAMES]
        g = fox.fox_pro_prologue_bwd(*a, *(x[n][b].clone() for n in ("dq", "dk", "dv")), eps=EPS)
        return [t for t in g if t.shape[0] == a[0].shape[0]]  # without the weights' gradients

    whole = grads(slice(0, B))
    assert len(whole) == 5
    for b in (0, B - 1):
        for i, (w, one) in enumerate(zip(whole, grads(slice(b, b + 1)))):
            assert torch.equal(w[b:b + 1], one), f"row {b} output {i}"
