"""The row-norm bounds at the edges of a workgroup's rows: one row, 512 and 1024 rows
and their neighbours, few chunks (512 rows each) and many (1024).

Tolerance: the result is the exact maximum enlarged by 2^-10, which covers the fp32
rounding of a sum of at most 128 squares (2^-17 relative)."""
import pytest
import torch

import paper_2503_02130_amd as fox
from paper_2503_02130_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,B,H,L", [
    ("bf16", 128, 1, 1, 1), ("bf16", 64, 1, 2, 511), ("f32", 128, 1, 2, 512),
    ("bf16", 128, 1, 3, 513), ("f32", 64, 2, 3, 1025), ("bf16", 64, 16, 8, 1024),
    ("bf16", 128, 9, 8, 1025), ("f32", 128, 9, 8, 1030),
    # fp32: both sides of its lines, 192 chunks (fewer threads) and, at d = 64, 72 chunks
    ("f32", 64, 1, 191, 1023), ("f32", 64, 3, 64, 1021), ("f32", 128, 2, 96, 1024),
    ("f32", 128, 1, 64, 2049), ("f32", 64, 1, 24, 3072), ("f32", 64, 1, 25, 3001)])
def test_row_norm_chunks(dtype, d, B, H, L):
    x = inputs.attn_inputs(B, H, L, d, dtype, ("normal", 0.0, 1.0), L + d, device="cuda:0")["k"]
    # the largest row of each head at another place: first, last, or between
    rows = torch.arange(B * H, device=x.device).reshape(B, H) * 7919 % L
    rows[0, 0], rows[-1, -1] = 0, L - 1
    x.scatter_(2, rows[..., None, None].expand(B, H, 1, d), 3.0)
    got = fox.fox_row_norm_max(x).double()
    ref = torch.linalg.vector_norm(x.double(), dim=-1).amax(dim=-1)
    assert torch.all(got >= ref) and torch.all(got <= ref * (1 + 2.0 ** -10 + 2.0 ** -16))
