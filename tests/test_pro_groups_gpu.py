"""The Pro prologue's and output gate's row passes at the edges of their launch shapes:
rows below, at and above one and two passes of a workgroup (L = 1 ... 257), and both
sides of the count of workgroups at which the backward passes change their threads.

Bounds are those of the parity tests: max-abs 1e-4 (fp32) or relative L2 1e-2 (bf16)
forward, relative L2 1e-4 or 2e-2 backward."""
import pytest
import torch

import oracle
import paper_2503_02130_amd as fox
from paper_2503_02130_amd import inputs

pytestmark = pytest.mark.gpu
EPS = 1e-6


def _rel(g, r):
    return float((g.double().cpu() - r).norm() / r.norm().clamp_min(1e-30))


@pytest.mark.parametrize("dtype,d,B,H,L", [
    ("bf16", 128, 1, 2, 33), ("bf16", 64, 1, 3, 255), ("f32", 64, 2, 1, 65),
    ("f32", 128, 16, 16, 31), ("bf16", 64, 16, 16, 129), ("bf16", 128, 16, 8, 257),
    ("bf16", 128, 1, 257, 3), ("f32", 64, 3, 43, 257), ("f32", 128, 2, 129, 17),
    # 768 workgroups of short slices, 1536 of any (output gate, bf16, d = 64): fewer threads
    ("bf16", 64, 8, 96, 80), ("bf16", 64, 8, 96, 128), ("f32", 128, 16, 48, 31),
    ("bf16", 64, 24, 64, 129), ("bf16", 64, 12, 64, 257), ("bf16", 128, 1, 767, 39)])
def test_pro_launch_shapes(dtype, d, B, H, L):
    x = inputs.pro_inputs(B, H, L, d, dtype, ("normal", 2.0, 1.0), L + d, device="cuda:0")
    args = tuple(x[n] for n in ("q_raw", "k_raw", "v_raw", "k_shift", "v_shift", "wq", "wk"))
    fwd = fox.fox_pro_prologue(*args, eps=EPS)
    y = fox.fox_pro_output_gate(fwd[2], x["g"], x["wo"], eps=EPS)
    grads = fox.fox_pro_prologue_bwd(*args, x["dq"], x["dk"], x["dv"], eps=EPS)
    ca = tuple(t.cpu() for t in args)
    ref = oracle.pro_prologue(*ca, EPS) + (
        oracle.output_gate(fwd[2].cpu(), x["g"].cpu(), x["wo"].cpu(), EPS),)
    for g, r in zip(fwd + (y,), ref):
        if dtype == "f32":
            assert float((g.double().cpu() - r).abs().max()) <= 1e-4
        else:
            assert _rel(g, r) <= 1e-2
    refb = oracle.pro_prologue_backward(*ca, EPS, x["dq"].cpu(), x["dk"].cpu(), x["dv"].cpu())
    for g, r in zip(grads, refb):
        assert _rel(g, r) <= (1e-4 if dtype == "f32" else 2e-2)
