"""The attention calls whose speed this framework is judged by, one case each: what a ModernBERT-style classifier (12 heads of
64, every third layer global, the others local with 63 keys to the left and 64 to the right) asks of the library at 512 to 32K
tokens, in both storage types, with the options that such a model uses: sequence lengths, a packed QKV projection read in
place, the operator's additive padding bias, rotary embedding inside the call, and the other head sizes.

A case is a dict of plain values:
  dtype       "fp16" or "bf16"
  batch, heads, max_len, head_dim   tensor extents
  min_len     shortest sequence: the lengths are spread evenly over [min_len, max_len] and dealt to the batch by the seed
              (0: no seq_lens argument, every row is valid)
  window      128: local layer (63 left, 64 right);  -1: global layer
  gain        q and k are gain * N(0, 1)  (1.5: a more peaked softmax)
  lse         the log-sum-exp is asked for
  packed      q, k, v are views of one [batch, len, 3, heads, dim] projection and o is [batch, len, heads, dim]
  bias        padding is an additive key bias of -65504 on the padded keys instead of seq_lens
  rope        q and k are rotated inside the call; a global layer lends the scratch that the library asks for
"""
import math

import torch

import paper_2603_12646_amd as fa

_DT = {"fp16": torch.float16, "bf16": torch.bfloat16}
_FA_DT = {"fp16": fa.FA_DTYPE_F16, "bf16": fa.FA_DTYPE_BF16}
_HEADS = {32: 24, 64: 12, 128: 8}   # hidden size 768 (768, 1024)


def _case(name, dtype, batch, max_len, min_len=0, head_dim=64, window=-1, gain=1.0, lse=True, packed=False, bias=False, rope=False):
    c = dict(dtype=dtype, batch=batch, heads=_HEADS[head_dim], max_len=max_len, head_dim=head_dim, min_len=min_len, window=window,
             gain=gain, lse=lse, packed=packed, bias=bias, rope=rope)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # one request after prompt compression, global layer: latency of a single small call
        _case("request_512", "fp16", 1, 512),
        # the same service's local layers (two of three) on a request of odd length: the smallest call there is
        _case("request_487_local", "fp16", 1, 487, window=128, lse=False),
        # one uncompressed request of ordinary length, padded to 2048
        _case("request_2k", "bf16", 1, 2048, min_len=1900),
        # 32 compressed requests served as one batch, ragged lengths
        _case("batch_32x512", "fp16", 32, 512, min_len=256),
        # a local layer of that batch, straight on the QKV projection's output, as an encoder calls it
        _case("batch_32x512_local_packed", "bf16", 32, 512, min_len=256, window=128, lse=False, packed=True),
        # the paper's operator contract: padding as an additive 1-D bias, no lengths
        _case("bias_8x2048", "fp16", 8, 2048, min_len=1024, bias=True),
        # the headline: an 8K-token global layer, valid length 7900, peaked softmax
        _case("global_8k", "fp16", 1, 8192, min_len=7900, gain=1.5),
        # a local layer of an 8K-token encoder with its rotary embedding, from the packed projection
        _case("local_8k_rope_packed", "bf16", 1, 8192, window=128, lse=False, packed=True, rope=True),
        # the operator's largest head size
        _case("global_8k_d128", "fp16", 1, 8192, min_len=7900, head_dim=128, gain=1.5),
        # three classifier sessions of up to 16K tokens side by side
        _case("sessions_3x16k", "bf16", 3, 16384, min_len=9000),
        # the longest context: one local and one global layer
        _case("local_32k", "bf16", 1, 32768, window=128),
        _case("global_32k", "bf16", 1, 32768),
    ]


def draw(rng):
    """Another call of the same kinds: one to 32 sequences of 128 to 32768 tokens, at most 49152 token rows in all and at most
    the 32K global layer's arithmetic."""
    head_dim = rng.choice([64, 64, 64, 64, 128, 32])
    window = rng.choice([-1, 128])
    while True:
        batch = int(round(math.exp(rng.uniform(0.0, math.log(32.0)))))
        max_len = int(round(math.exp(rng.uniform(math.log(128.0), math.log(32768.0)))))
        # (head_dim 32 does twice the softmax work per flop)
        pairs = batch * _HEADS[head_dim] * max_len * max_len * head_dim * (2 if head_dim == 32 else 1)
        if batch * max_len <= 49152 and (window > 0 or pairs <= 12 * 32768 * 32768 * 64):
            break
    option = rng.choice(["", "", "", "packed", "bias", "rope", "packed rope"])
    min_len = 0
    if "bias" in option or rng.random() < 0.7:
        min_len = max(1, int(max_len * rng.uniform(0.4, 1.0)))
    return _case("", rng.choice(["fp16", "bf16"]), batch, max_len, min_len=min_len, head_dim=head_dim, window=window,
                 gain=rng.choice([1.0, 1.5]), lse=rng.random() < 0.5, packed="packed" in option, bias="bias" in option,
                 rope="rope" in option)


def _lengths(c):
    """Valid lengths before they are dealt to the batch (None: no padding)."""
    if not c["min_len"]:
        return None
    lo, hi, b = c["min_len"], c["max_len"], c["batch"]
    return [lo] if b == 1 else [lo + (hi - lo) * i // (b - 1) for i in range(b)]


def _extents(c):
    return (-1, -1) if c["window"] < 0 else ((c["window"] - 1) // 2, c["window"] // 2)


def prepare(c, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt, B, H, N, D = _DT[c["dtype"]], c["batch"], c["heads"], c["max_len"], c["head_dim"]
    s = {"case": c, "scale": D ** -0.5}
    if c["packed"]:
        qkv = torch.randn((B, N, 3, H, D), generator=g, device="cuda")
        if c["gain"] != 1.0:
            qkv[:, :, :2] *= c["gain"]
        s["qkv"] = qkv.to(dt)
        s["q"], s["k"], s["v"] = s["qkv"][:, :, 0], s["qkv"][:, :, 1], s["qkv"][:, :, 2]
        s["o"] = torch.empty((B, N, H, D), dtype=dt, device="cuda")
        s["in_strides"], s["o_strides"] = (N * 3 * H * D, D, 3 * H * D), (N * H * D, D, H * D)
    else:
        s["q"], s["k"] = ((c["gain"] * torch.randn((B, H, N, D), generator=g, device="cuda")).to(dt) for _ in range(2))
        s["v"] = torch.randn((B, H, N, D), generator=g, device="cuda").to(dt)
        s["o"] = torch.empty((B, H, N, D), dtype=dt, device="cuda")
        s["in_strides"] = s["o_strides"] = None
    s["lse"] = torch.empty((B, H, N), dtype=torch.float32, device="cuda") if c["lse"] else None
    s["lens"] = s["bias"] = s["cos"] = s["sin"] = s["scratch"] = None
    lens = _lengths(c)
    if lens is not None:
        order = torch.randperm(B, generator=g, device="cuda")
        lens = torch.tensor(lens, dtype=torch.int32, device="cuda")[order]
        if c["bias"]:
            padded = torch.arange(N, device="cuda")[None, :] >= lens[:, None]
            s["bias"] = torch.where(padded, torch.tensor(-65504.0, device="cuda"), torch.tensor(0.0, device="cuda")).to(dt)
        else:
            s["lens"] = lens
    if c["rope"]:
        # the rotary base of a local and of a global layer
        base = 10000.0 if c["window"] > 0 else 160000.0
        freq = base ** (-2.0 * torch.arange(D // 2, device="cuda", dtype=torch.float64) / D)
        angle = torch.arange(N, device="cuda", dtype=torch.float64)[:, None] * freq[None, :]
        s["cos"], s["sin"] = angle.cos().float(), angle.sin().float()
        if c["window"] < 0:
            s["scratch"] = torch.empty(fa.fa_rope_scratch_bytes(B, H, N, D), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    c = s["case"]
    if c["packed"] or c["bias"] or c["rope"]:
        left, right = _extents(c)
        scratch = s["scratch"]
        fa.fa_fwd_ex(dtype=_FA_DT[c["dtype"]], q=s["q"], k=s["k"], v=s["v"], o=s["o"], lse=s["lse"], seq_lens=s["lens"],
                     batch=c["batch"], heads=c["heads"], max_len=c["max_len"], head_dim=c["head_dim"], scale=s["scale"],
                     window_left=left, window_right=right, q_strides=s["in_strides"], k_strides=s["in_strides"],
                     v_strides=s["in_strides"], o_strides=s["o_strides"], key_bias=s["bias"], rope_cos=s["cos"],
                     rope_sin=s["sin"], scratch=scratch, scratch_bytes=0 if scratch is None else scratch.numel())
    else:
        fn = fa.fa_fwd if c["dtype"] == "fp16" else fa.fa_fwd_bf16
        fn(s["q"], s["k"], s["v"], s["o"], s["lse"], c["batch"], c["heads"], s["lens"], c["max_len"], c["head_dim"], s["scale"],
           c["window"])
    return {"o": s["o"]} if s["lse"] is None else {"o": s["o"], "lse": s["lse"]}


def _visible(n, c):
    """Number of (query, key) pairs of one sequence of n tokens."""
    left, right = _extents(c)
    if left < 0:
        return n * n
    # row i misses left - i keys before the start and right - (n - 1 - i) keys past the end
    return n * (left + right + 1) - sum(left - i for i in range(min(left, n))) - sum(right - i for i in range(min(right, n)))


def work(c):
    B, H, N, D = c["batch"], c["heads"], c["max_len"], c["head_dim"]
    lens = _lengths(c) if not c["bias"] else None
    rows = B * N if lens is None else sum(lens)
    pairs = B * _visible(N, c) if lens is None else sum(_visible(n, c) for n in lens)
    bytes_ = H * D * 2 * (3 * rows + B * N)            # q, k, v of the valid rows; o of every row
    bytes_ += 4 * B * H * N if c["lse"] else 0
    bytes_ += 2 * B * N if c["bias"] else 0
    bytes_ += 4 * N * D if c["rope"] else 0            # two tables of D / 2 columns
    return {"bytes": bytes_, "flops": 4 * D * H * pairs}


def tolerance(c):
    # o is rounded to 16 bits, and so is every probability before the second product: 11 significand bits (fp16) or 8 (bf16).
    # Measured against exact(): 2.9e-4 and 2.4e-3; four times that
    return {"rel": 1.2e-3} if c["dtype"] == "fp16" else {"rel": 1e-2}


def exact(c, seed):
    s = prepare(c, seed)
    B, H, N, D = c["batch"], c["heads"], c["max_len"], c["head_dim"]
    left, right = _extents(c)
    to_bhnd = (lambda x: x.transpose(1, 2)) if c["packed"] else (lambda x: x)
    lens = [N] * B if s["lens"] is None else s["lens"].tolist()
    o = torch.zeros((B, H, N, D), dtype=torch.float64, device="cuda")
    lse = torch.full((B, H, N), -math.inf, dtype=torch.float64, device="cuda")
    for b in range(B):
        n = lens[b]
        q, k, v = (to_bhnd(s[x])[b, :, :n].double() for x in "qkv")
        if c["rope"]:
            # rotated in pairs (f, f + D/2) and stored in the 16-bit type, as the operator's definition says
            cos, sin, h = s["cos"][:n].double(), s["sin"][:n].double(), D // 2
            q, k = (torch.cat([x[..., :h] * cos - x[..., h:] * sin, x[..., h:] * cos + x[..., :h] * sin], dim=-1)
                    .to(_DT[c["dtype"]]).double() for x in (q, k))
        step = max(64, min(n, (1 << 26) // (H * (n if left < 0 else min(n, 640)))))
        if left >= 0:
            step = min(step, 512)
        for i0 in range(0, n, step):
            i1 = min(n, i0 + step)
            j0, j1 = (0, n) if left < 0 else (max(0, i0 - left), min(n, i1 + right))
            sc = torch.matmul(q[:, i0:i1].contiguous(), k[:, j0:j1].transpose(1, 2).contiguous()) * s["scale"]
            if s["bias"] is not None:
                sc += s["bias"][b, j0:j1].double()
            if left >= 0:
                i, j = torch.arange(i0, i1, device="cuda")[:, None], torch.arange(j0, j1, device="cuda")[None, :]
                sc.masked_fill_((j < i - left) | (j > i + right), -math.inf)
            lse[b, :, i0:i1] = torch.logsumexp(sc, dim=-1)
            o[b, :, i0:i1] = torch.matmul(torch.softmax(sc, dim=-1), v[:, j0:j1].contiguous())
    out = {"o": o.transpose(1, 2).contiguous() if c["packed"] else o}
    return out if s["lse"] is None else {**out, "lse": lse}
