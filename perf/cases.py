"""The workloads whose speed is tracked: what each stands for, how it is prepared,
run and checked.

Every case goes through the package's public entry points the way a program that
uses it does.  The kinds:

  train    gate prefix, forward and backward through autograd (forgetting_attention)
  prefill  gate prefix and forward of a prompt (O and LSE)
  decode   one new token per sequence against a key/value cache
  skip     a training step with exact gate-aware skipping, row norms included
  fixed    forward and backward with fixed per-head gates (ALiBi form)
  pro      the FoX (Pro) layer around the attention, forward and backward
  proj     the forget-gate projection from the layer input, forward and backward

A case is a dict of plain values: kind, dtype, B, H, L (for decode the cache
length), d, and the options of its kind.  `exact` computes the same outputs in
64 bits with plain torch.
"""
import math

import torch

import paper_2503_02130_amd as fox
from paper_2503_02130_amd import inputs

F64 = torch.float64
EPS = 1e-6  # RMSNorm epsilon of the Pro layer

# forget-gate logits as the repository's workloads draw them
GATES = {
    "mixed": ("head_mean_uniform", 0.0, 6.0, 1.0),   # short and long memories side by side
    "n2": ("normal", 2.0, 1.0),
    "n3": ("normal", 3.0, 1.0),
    "split": ("split_heads", (6.0, 1.0), (0.0, math.sqrt(2.0))),
}


def listed():
    return [
        # the long-context training step at the 16k training context, keeping dS
        dict(name="train_16k_d128", kind="train", dtype="bf16", B=2, H=16, L=16384, d=128,
             gate="mixed", keep_ds=True),
        # the 125M-model head shape at a 2k context, the default backward
        dict(name="train_2k_d64", kind="train", dtype="bf16", B=8, H=12, L=2048, d=64,
             gate="n2", keep_ds=False),
        # a small fine-tuning or debugging step in full precision, ragged length
        dict(name="train_f32_1000_d64", kind="train", dtype="f32", B=2, H=12, L=1000, d=64,
             gate="n2", keep_ds=False),
        # length extrapolation: one 64k prompt
        dict(name="prefill_64k_d128", kind="prefill", dtype="bf16", B=1, H=16, L=65536, d=128,
             gate="split"),
        # an ordinary prompt of one request, odd length
        dict(name="prefill_3001_d128", kind="prefill", dtype="bf16", B=1, H=16, L=3001, d=128,
             gate="mixed"),
        # the smallest call: a short full-precision prompt
        dict(name="prefill_f32_256_d64", kind="prefill", dtype="f32", B=1, H=2, L=256, d=64,
             gate="n2"),
        # batched serving: one token for 64 sequences against 32k caches
        dict(name="decode_b64_32k_d128", kind="decode", dtype="bf16", B=64, H=16, L=32768, d=128,
             gate="n3"),
        # interactive serving: one sequence, odd cache length
        dict(name="decode_b1_4097_d128", kind="decode", dtype="bf16", B=1, H=16, L=4097, d=128,
             gate="n3"),
        # the training step with exact skipping
        dict(name="skip_8k_d128", kind="skip", dtype="bf16", B=1, H=16, L=8192, d=128,
             gate="mixed"),
        # fixed gates, ragged length
        dict(name="fixed_1500_d64", kind="fixed", dtype="bf16", B=4, H=12, L=1500, d=64),
        # the FoX (Pro) layer at a 4k context
        dict(name="pro_4k_d128", kind="pro", dtype="bf16", B=2, H=16, L=4096, d=128,
             gate="mixed", keep_ds=True),
        # the forget-gate projection at the long-context training shape
        dict(name="proj_16k_m2048", kind="proj", dtype="bf16", B=2, H=16, L=16384, M=2048),
    ]


def _log_int(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi], odd ones among them."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["train", "train", "train", "prefill", "prefill", "decode", "decode",
                       "skip", "fixed", "pro", "proj"])
    H = rng.choice([1, 2, 4, 8, 12, 16])
    d = rng.choice([64, 128])
    if kind == "decode":
        c = dict(kind=kind, dtype=rng.choice(["bf16", "bf16", "f32"]), B=_log_int(rng, 1, 64), H=H,
                 L=_log_int(rng, 128, 32768), d=d, gate="n3")
        while c["B"] * H * c["L"] * d * (1 if c["dtype"] == "bf16" else 2) > 64 * 16 * 32768 * 128:
            c["L"] = _log_int(rng, 128, 32768)
        return c
    if kind == "proj":
        M = 8 * _log_int(rng, 32, 256)
        return dict(kind=kind, dtype=rng.choice(["bf16", "f32"]), B=_log_int(rng, 1, 4), H=H,
                    L=_log_int(rng, 64, 8192), M=M)
    dtype = "bf16"
    if kind in ("train", "prefill"):
        dtype = rng.choice(["bf16", "bf16", "f32"])
    # (head, pair) products up to the listed ones: 2 x 16 heads at 16k in bf16; the
    # full-precision path is for small work
    pairs = 32 * 16384 ** 2 * 128 if dtype == "bf16" else 24 * 1500 ** 2 * 64
    longest = 16384 if dtype == "bf16" else 2048
    B, L = _log_int(rng, 1, 8), _log_int(rng, 64, longest)
    while B * H * L * L * d > pairs:
        B, L = _log_int(rng, 1, 8), _log_int(rng, 64, longest)
    c = dict(kind=kind, dtype=dtype, B=B, H=H, L=L, d=d)
    if kind != "fixed":
        c["gate"] = rng.choice(["mixed", "n2", "n3"])
    if kind in ("train", "pro"):
        c["keep_ds"] = dtype == "bf16" and rng.choice([True, False])
    return c


def prepare(case, seed):
    kind, dt, dev = case["kind"], case["dtype"], "cuda:0"
    B, H, L = case["B"], case["H"], case["L"]
    gate = GATES.get(case.get("gate"))
    if kind == "proj":
        x = inputs.projection_inputs(B, L, H, case["M"], dt, seed, device=dev)
        for n in ("x", "w_f", "b_f"):
            x[n].requires_grad_(True)
        return dict(kind=kind, **x)
    d = case["d"]
    if kind == "decode":
        x = inputs.decode_inputs(B, H, L, d, dt, gate, seed, device=dev)
        c = torch.zeros((B, H, L), device=dev)
        c[..., : L - 1] = torch.nn.functional.logsigmoid(
            x.pop("cached_logit").to(F64)).cumsum(-1).float()
        # the workspace a serving loop keeps
        ws = torch.empty(max(16, fox.fox_attn_decode_workspace_bytes(x["q"].dtype, B, H, L, d)),
                         device=dev, dtype=torch.uint8)
        return dict(kind=kind, c=c, ws=ws, **x)
    if kind == "pro":
        x = inputs.pro_inputs(B, H, L, d, dt, gate, seed, device=dev)
        for n in ("dq", "dk", "dv"):
            x.pop(n)
        return dict(kind=kind, keep_ds=case["keep_ds"], **x)
    x = inputs.attn_inputs(B, H, L, d, dt, gate or ("constant", 0.0), seed, device=dev,
                           grad=kind != "prefill")
    if kind == "train":
        for n in ("q", "k", "v", "logit"):
            x[n].requires_grad_(True)
        x["keep_ds"] = case["keep_ds"]
    if kind == "fixed":
        x.pop("logit")
        x["bias"] = fox.fox_fixed_gate_init(H, 2.0, 512.0).to(dev)
    return dict(kind=kind, **x)


def run(s):
    kind = s["kind"]
    if kind == "train":
        o = fox.forgetting_attention(s["q"], s["k"], s["v"], s["logit"], keep_ds=s["keep_ds"])
        return [o.detach(), *torch.autograd.grad(o, [s["q"], s["k"], s["v"], s["logit"]], s["do"])]
    if kind == "prefill":
        c = fox.fox_gate_prefix(s["logit"])
        return [c, *fox.fox_attn_fwd(s["q"], s["k"], s["v"], c)]
    if kind == "decode":
        o, lse = fox.fox_attn_decode(s["q"], s["k_cache"], s["v_cache"], s["c"], s["logit_new"],
                                     workspace=s["ws"])
        return [o, lse, s["c"]]
    if kind == "skip":
        c = fox.fox_gate_prefix(s["logit"])
        qn, kn = fox.fox_row_norm_max(s["q"]), fox.fox_row_norm_max(s["k"])
        o, lse = fox.fox_attn_fwd_skip(s["q"], s["k"], s["v"], c, qn, kn)
        return [o, lse, *fox.fox_attn_bwd_skip_stored(s["q"], s["k"], s["v"], c, o, lse, s["do"],
                                                      qn, kn)]
    if kind == "fixed":
        o, lse = fox.fox_attn_fwd_fixed_gate(s["q"], s["k"], s["v"], s["bias"])
        return [o, lse, *fox.fox_attn_bwd_fixed_gate(s["q"], s["k"], s["v"], s["bias"], o, lse,
                                                     s["do"])]
    if kind == "pro":
        q, k, v = fox.fox_pro_prologue(s["q_raw"], s["k_raw"], s["v_raw"], s["k_shift"],
                                       s["v_shift"], s["wq"], s["wk"], eps=EPS)
        c = fox.fox_gate_prefix(s["logit"])
        y, o, lse = fox.fox_attn_fwd_pro(q, k, v, c, s["g"], s["wo"], eps=EPS)
        bwd = fox.fox_attn_bwd_pro_stored if s["keep_ds"] else fox.fox_attn_bwd_pro
        dq, dk, dv, dlf, dg, dwo = bwd(q, k, v, c, o, lse, s["g"], s["wo"], s["dy"], eps=EPS)
        return [y, dlf, dg, dwo,
                *fox.fox_pro_prologue_bwd(s["q_raw"], s["k_raw"], s["v_raw"], s["k_shift"],
                                          s["v_shift"], s["wq"], s["wk"], dq, dk, dv, eps=EPS)]
    logit = fox.forget_gate_logits(s["x"], s["w_f"], s["b_f"])
    return [logit.detach(),
            *torch.autograd.grad(logit, [s["x"], s["w_f"], s["b_f"]], s["d_logit"])]


def work(case):
    """Each input read once and each output written once, in bytes, and the causal
    multiply-adds: 4 d per (query, key) pair forward, 10 d backward."""
    kind, B, H, L = case["kind"], case["B"], case["H"], case["L"]
    es = 2 if case["dtype"] == "bf16" else 4
    n = B * H * L
    if kind == "proj":  # x, w_f, d_logit in; logits, dx, dw_f out
        M = case["M"]
        return dict(bytes=2 * B * L * M * es + 2 * H * M * 4 + 2 * n * 4, flops=6 * n * M)
    d = case["d"]
    pairs = B * H * L * (L + 1) // 2
    if kind == "decode":  # the cache in; q, o and the per-sequence values are small
        return dict(bytes=2 * n * d * es + n * 4 + 2 * B * H * d * es, flops=4 * n * d)
    if kind == "prefill":  # q, k, v, logits in; o, lse, c out
        return dict(bytes=4 * n * d * es + 3 * n * 4, flops=4 * d * pairs)
    # q, k, v, dO in; o, dq, dk, dv out (pro: raw q, k, v, g, dy; y, dg and three
    # gradients); logits in, their gradient out (pro: three of each)
    big, rows = (10, 6) if kind == "pro" else (8, 2)
    return dict(bytes=big * n * d * es + rows * n * 4, flops=14 * d * pairs)


def tolerance(case):
    if case["dtype"] == "f32":
        return dict(rel=TOL_F32[case["kind"]])
    return dict(rel=TOL_BF16[case["kind"]])


# About four times the relative error against `exact` of the worst output (measured:
# bf16 train 3.7e-3, prefill 1.9e-3, decode 1.7e-3, skip 3.9e-3, fixed 5.5e-3, pro
# 5.3e-3, proj 1.7e-3; f32 train 4.6e-6, prefill 2.3e-6, proj 2.5e-6)
TOL_BF16 = dict(train=1.5e-2, prefill=8e-3, decode=8e-3, skip=1.6e-2, fixed=2.2e-2, pro=2.2e-2,
                proj=7e-3)
TOL_F32 = dict(train=2e-5, prefill=1e-5, decode=1e-5, proj=1e-5)


# ------------------------------------------------------------------ 64-bit results
def _attention64(q, k, v, log_f, do=None):
    """One head in 64 bits: o, lse, c and, with do, dq, dk, dv and d(log f);
    a block of query rows at a time."""
    L, d = q.shape
    q, k, v, c = q.to(F64), k.to(F64), v.to(F64), log_f.to(F64).cumsum(0)
    s = 1.0 / math.sqrt(d)
    o, lse = torch.empty_like(q), torch.empty_like(c)
    dq = dk = dv = dlf = None
    if do is not None:
        do = do.to(F64)
        dq, dk, dv, dc = (torch.zeros_like(t) for t in (q, k, v, c))
    rows = max(1, min(L, (1 << 26) // L))
    pos = torch.arange(L, device=q.device)
    for i0 in range(0, L, rows):
        i1 = min(L, i0 + rows)
        S = (q[i0:i1] @ k[:i1].T).mul_(s).add_(c[i0:i1, None]).sub_(c[None, :i1])
        S.masked_fill_(pos[None, :i1] > pos[i0:i1, None], -math.inf)
        lse[i0:i1] = torch.logsumexp(S, 1)
        P = S.sub_(lse[i0:i1, None]).exp_()
        o[i0:i1] = P @ v[:i1]
        if do is not None:
            g = do[i0:i1]
            dv[:i1] += P.T @ g
            dS = P.mul_((g @ v[:i1].T).sub_((g * o[i0:i1]).sum(1, keepdim=True)))
            dq[i0:i1] = (dS @ k[:i1]).mul_(s)
            dk[:i1] += (dS.T @ q[i0:i1]).mul_(s)
            dc[i0:i1] += dS.sum(1)
            dc[:i1] -= dS.sum(0)
    if do is not None:
        dlf = dc.flip(0).cumsum(0).flip(0)
    return o, lse, c, dq, dk, dv, dlf


def _heads64(q, k, v, log_f, do=None):
    """_attention64 over [B, H, ...], each result stacked back to [B, H, ...]."""
    B, H = q.shape[:2]
    out = [_attention64(q[b, h], k[b, h], v[b, h], log_f[b, h],
                        None if do is None else do[b, h]) for b in range(B) for h in range(H)]
    return [None if r[0] is None else torch.stack(r).reshape(B, H, *r[0].shape)
            for r in zip(*out)]


def _rms64(x, w):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * w[None, :, None, :]


def exact(case, seed):
    s = prepare(case, seed)
    s = {n: t.detach() if isinstance(t, torch.Tensor) else t for n, t in s.items()}
    kind = case["kind"]
    logsig = torch.nn.functional.logsigmoid
    if kind == "proj":
        x, w, g = s["x"].to(F64), s["w_f"].to(F64), s["d_logit"].to(F64)
        logit = torch.stack([x[b] @ w.T for b in range(x.shape[0])]).transpose(1, 2)
        dx = torch.stack([g[b].T.contiguous() @ w for b in range(x.shape[0])])
        dw = sum(g[b] @ x[b] for b in range(x.shape[0]))
        return [logit + s["b_f"].to(F64)[None, :, None], dx, dw, g.sum((0, 2))]
    if kind == "decode":
        B, H, d = s["q"].shape
        c = s["c"].to(F64)
        c[..., -1] = (c[..., -2] if c.shape[-1] > 1 else 0.0) + logsig(s["logit_new"].to(F64))
        o, lse = torch.empty((B, H, d), dtype=F64, device=c.device), torch.empty_like(c[..., 0])
        for b in range(B):  # one sequence of the cache in 64 bits at a time
            sc = (s["k_cache"][b].to(F64) * s["q"][b].to(F64)[:, None]).sum(-1) / math.sqrt(d)
            sc += c[b, :, -1:] - c[b]
            lse[b] = torch.logsumexp(sc, -1)
            o[b] = ((sc - lse[b][:, None]).exp()[..., None] * s["v_cache"][b].to(F64)).sum(1)
        return [o, lse, c]
    if kind == "pro":
        a = {n: t.to(F64).requires_grad_(True) for n, t in s.items()
             if n in ("q_raw", "k_raw", "v_raw", "k_shift", "v_shift", "wq", "wk", "wo", "g")}

        def shift(x, z):
            m = torch.sigmoid(z)[..., None]
            return m * torch.nn.functional.pad(x, (0, 0, 1, 0))[:, :, :-1] + (1 - m) * x

        q = _rms64(a["q_raw"], a["wq"])
        k = _rms64(shift(a["k_raw"], a["k_shift"]), a["wk"])
        v = shift(a["v_raw"], a["v_shift"])
        log_f = logsig(s["logit"].to(F64))
        qd, kd, vd = q.detach(), k.detach(), v.detach()
        o = _heads64(qd, kd, vd, log_f)[0].requires_grad_(True)
        y = _rms64(o, a["wo"]) * torch.sigmoid(a["g"])
        do, dg, dwo = torch.autograd.grad(y, [o, a["g"], a["wo"]], s["dy"].to(F64))
        _, _, _, dq, dk, dv, dlf = _heads64(qd, kd, vd, log_f, do)
        names = ("q_raw", "k_raw", "v_raw", "k_shift", "v_shift", "wq", "wk")
        return [y.detach(), dlf, dg, dwo,
                *torch.autograd.grad([q, k, v], [a[n] for n in names], [dq, dk, dv])]
    if kind == "fixed":
        B, H, L, _ = s["q"].shape
        b = s["bias"].to(F64)
        log_f = logsig(b)[None, :, None].expand(B, H, L)
    else:
        log_f = logsig(s["logit"].to(F64))
    o, lse, c, dq, dk, dv, dlf = _heads64(s["q"], s["k"], s["v"], log_f, s.get("do"))
    if kind == "prefill":
        return [c, o, lse]
    if kind == "train":
        return [o, dq, dk, dv, dlf * torch.sigmoid(-s["logit"].to(F64))]
    if kind == "skip":
        return [o, lse, dq, dk, dv, dlf]
    return [o, lse, dq, dk, dv, torch.sigmoid(-b) * dlf.sum((0, 2))]
