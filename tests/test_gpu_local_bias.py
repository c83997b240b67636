"""GPU parity of the local layers' two-phase kernel with an additive key bias and with a rotation (compile-time variants),
at every head size: tile edges, the merged end blocks, keys excluded for whole windows, negative scale, packed inputs,
and sequence lengths that end inside and at the edges of 32-key blocks.  Against the fp64 oracles with the bounds of the
other parity tests."""
import numpy as np
import pytest
import torch

import paper_2603_12646_amd as fa
from oracle.attention_oracle import attention_oracle, attention_oracle_rows
from workloads import draw, round_to_storage

from tests.gpu_util import FA_DT, check_against, poison, run_ex, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("left,right", [(63, 64), (0, 0), (10, 64), (64, 3)])
def test_two_phase_kernel_with_key_bias(D, dtype, left, right):
    lens = [421, 320, 97, 1]
    B, H, N = len(lens), 2, 421
    rng = np.random.default_rng(D + left)
    _, q, k, v = draw(4000 + D, B, H, N, D, dtype)
    bias = round_to_storage(rng.standard_normal((B, N)).astype(np.float32), dtype)
    bias[rng.random((B, N)) < 0.2] = -np.inf
    bias[0, 100:300] = -np.inf                      # rows around 200 see no key at all
    # the paper's padding value on every second key: beside ordinary keys their probabilities are 0.  (On whole windows it
    # would compare what fp32 cannot hold: a score near -65504 has a spacing of 2^-8, so any fp32 sum of score and bias is up
    # to 2^-9 off and its probability 0.2 %, more than this test's 2e-3 on values up to 4.)
    bias[1, 200::2] = round_to_storage(np.full((1,), -65504.0, dtype=np.float32), dtype)[0]
    bias[1, 201::2] = 0.0
    scale = -(D ** -0.5)
    o_ref, lse_ref = attention_oracle(q, k, v, lens, scale, left, right, key_bias=bias)
    for b, n in enumerate(lens):
        for x in (q, k, v):
            x[b, :, n:] = np.nan
    o, lse = run_ex(q, k, v, lens, dtype, scale, left, right, tuning=fa.FA_TUNE_WIN_TWO_PHASE, key_bias=bias)
    check_against(o, lse, o_ref, lse_ref, lens, dtype, relative=True, label=f"two-phase bias D{D} {left}/{right}")


@pytest.mark.parametrize("D", [32, 64, 128])
def test_two_phase_kernel_with_key_bias_packed_and_many_tiles(D):
    """The library's own choice on a call of more than 384 tiles, read from a packed QKV buffer: the bits of the dense call."""
    B, H, N = 3, 12, 1409
    lens = [1409, 700, 1280]
    _, q, k, v = draw(4100, B, H, N, D, "bf16")
    bias = round_to_storage(np.random.default_rng(2).standard_normal((B, N)).astype(np.float32), "bf16")
    o, lse = run_ex(q, k, v, lens, "bf16", D ** -0.5, 63, 64, key_bias=bias)
    sel = [0, 5, 11]
    o_ref, lse_ref = attention_oracle(q[:, sel], k[:, sel], v[:, sel], lens, D ** -0.5, 63, 64, key_bias=bias)
    check_against(o[:, sel], lse[:, sel], o_ref, lse_ref, lens, "bf16", relative=True, label=f"bias many tiles D{D}")
    packed = torch.stack([to_dev(np.ascontiguousarray(x.transpose(0, 2, 1, 3)), "bf16") for x in (q, k, v)], dim=2)
    st = (N * 3 * H * D, D, 3 * H * D)
    o2 = poison((B, N, H, D), "bf16")
    fa.fa_fwd_ex(dtype=FA_DT["bf16"], q=packed[:, :, 0], k=packed[:, :, 1], v=packed[:, :, 2], o=o2,
                 seq_lens=torch.tensor(lens, dtype=torch.int32, device="cuda"), batch=B, heads=H, max_len=N, head_dim=D,
                 scale=D ** -0.5, window_left=63, window_right=64, q_strides=st, k_strides=st, v_strides=st,
                 o_strides=(N * H * D, D, H * D), key_bias=to_dev(bias, "bf16"))
    torch.cuda.synchronize()
    assert np.array_equal(o2.double().cpu().numpy().transpose(0, 2, 1, 3), o)


@pytest.mark.parametrize("D,rope,N,lens", [(64, True, 6200, [6200, 1000]), (128, True, 6200, [0, 6150]), (32, True, 6200, None),
                                           (32, False, 2100, [2100, 129]), (32, True, 2100, [1, 2000])])
def test_heads_first_order_gives_the_bits_of_the_linear_order(D, rope, N, lens):
    """Calls that hand out the heads of a query tile in a row (a rotation on a long local layer; heads of 32 side by side):
    the same bits as with workgroup ids taken as tile numbers, every padded row zero."""
    B, H = 2, 3
    g = torch.Generator(device="cuda").manual_seed(N + D)
    qkv = torch.randn((B, N, 3, H, D), generator=g, device="cuda").bfloat16()
    ang = torch.arange(N, device="cuda", dtype=torch.float32)[:, None] * 10000.0 ** (-2.0 * torch.arange(D // 2, device="cuda") / D)
    cos, sin = (ang.cos().contiguous(), ang.sin().contiguous()) if rope else (None, None)
    sl = None if lens is None else torch.tensor(lens, dtype=torch.int32, device="cuda")
    st = (N * 3 * H * D, D, 3 * H * D)
    got = []
    for tuning in (0, fa.FA_TUNE_MAP_LINEAR):
        o = poison((B, N, H, D), "bf16")
        lse = torch.full((B, H, N), float("nan"), dtype=torch.float32, device="cuda")
        fa.fa_fwd_ex(dtype=FA_DT["bf16"], q=qkv[:, :, 0], k=qkv[:, :, 1], v=qkv[:, :, 2], o=o, lse=lse, seq_lens=sl, batch=B,
                     heads=H, max_len=N, head_dim=D, scale=D ** -0.5, window_left=63, window_right=64, q_strides=st,
                     k_strides=st, v_strides=st, o_strides=(N * H * D, D, H * D), rope_cos=cos, rope_sin=sin,
                     tuning=tuning | fa.FA_TUNE_WIN_TWO_PHASE)
        torch.cuda.synchronize()
        got.append((o, lse))
    assert not torch.isnan(got[0][0]).any() and torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    for b, n in enumerate(lens or []):
        assert (got[0][0][b, n:] == 0).all() and torch.isneginf(got[0][1][b, :, n:]).all()


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("left,right,N", [(63, 64, 300), (-1, -1, 300), (-1, -1, 5000)])
@pytest.mark.parametrize("dtype,scale", [("fp16", 1e-39), ("fp16", -1e-36), ("bf16", 1e-39), ("bf16", 1e-36)])
def test_key_bias_with_a_tiny_scale(D, left, right, N, dtype, scale):
    """A scale so small that bias / |scale| leaves the range of fp32: the softmax is that of the bias alone."""
    _, q, k, v = draw(4300 + D, 1, 2, N, D, dtype)
    rng = np.random.default_rng(D)
    bias = round_to_storage(rng.standard_normal((1, N)).astype(np.float32), dtype)
    bias[0, rng.random(N) < 0.3] = round_to_storage(np.full((1,), -65504.0, np.float32), dtype)[0]
    o, lse = run_ex(q, k, v, None, dtype, scale, left, right, key_bias=bias)
    rows = np.unique(np.concatenate([np.arange(0, 200), np.arange(N - 70, N)]))
    for h in range(2):
        o_ref, lse_ref = attention_oracle_rows(q, k, v, 0, h, rows, N, scale, left, right, key_bias=bias)
        check_against(o[:, h:h + 1, rows], lse[:, h:h + 1, rows], o_ref[None, None], lse_ref[None, None], None, dtype,
                      relative=True, label=f"tiny scale D{D} h{h}")


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("left,right,N", [(63, 64, 300), (63, 64, 3000), (-1, -1, 300), (-1, -1, 5000)])
@pytest.mark.parametrize("scale", [1.0, 0.75, 0.125])
def test_key_bias_of_the_types_lowest_value(D, left, right, N, scale):
    """bfloat16's lowest finite value as the padding bias, on the first keys (left padding) and scattered ones: those keys
    have weight 0 for every row that sees another."""
    B, H = 1, 12
    _, q, k, v = draw(4400 + D, B, 1, N, D, "bf16", qk_gain=0.3)
    rep = lambda x: np.repeat(x, H, axis=1)
    bias = np.zeros((B, N), np.float32)
    bias[0, :40] = bias[0, 100::3] = torch.finfo(torch.bfloat16).min
    o, lse = run_ex(rep(q), rep(k), rep(v), None, "bf16", scale, left, right, key_bias=bias)
    rows = np.unique(np.concatenate([np.arange(0, 260), np.arange(N - 70, N)]))
    o_ref, lse_ref = attention_oracle_rows(q, k, v, 0, 0, rows, N, scale, left, right, key_bias=bias)
    check_against(o[:, :1, rows], lse[:, :1, rows], o_ref[None, None], lse_ref[None, None], None, "bf16", relative=True,
                  label=f"lowest D{D} {scale}")
    assert (o == o[:, :1]).all()


@pytest.mark.parametrize("tuning", [0, fa.FA_TUNE_BM_128, fa.FA_TUNE_BM_256])
@pytest.mark.parametrize("D,left,right", [(32, 63, 64), (128, 63, 64), (32, -1, -1)])
def test_key_bias_rounds_a_score_once(D, left, right, tuning):
    """The paper's padding value on EVERY key: a score near -65504 is a sum of score and bias that fp32 holds to half a
    spacing, and that one rounding (of bias / scale, by at most d = 2^-24 * 65504 here) is all that may show.  With every
    probability off by at most d + 2^-11 (its own rounding to fp16) relative, o is off by that times the mean distance of
    the values from it (and the numerator alone carries the rounding to fp16, as o does once more)."""
    N = 600
    scale = D ** -0.5
    _, q, k, v = draw(4500 + D, 1, 2, N, D, "fp16", qk_gain=1.7)
    bias = np.full((1, N), -65504.0, np.float32)
    o, lse = run_ex(q, k, v, None, "fp16", scale, left, right, key_bias=bias,
                    tuning=tuning | (0 if left < 0 else fa.FA_TUNE_WIN_TWO_PHASE))
    x = 65504.0 / scale
    d = 0.5 * np.spacing(np.float32(x)) * scale
    assert d <= 2.0 ** -24 * 65504
    o_ref, lse_ref, P = attention_oracle(q, k, v, None, scale, left, right, key_bias=bias, return_p=True)
    spread = np.stack([(P[0, h][:, :, None] * np.abs(v[0, h][None] - o_ref[0, h][:, None])).sum(1) for h in range(2)])[None]
    bound = 1.01 * (d + 2.0 ** -11) * spread + 2.0 ** -10 * np.abs(o_ref) + 2e-5
    worst = (np.abs(o - o_ref) / bound).max()
    assert worst <= 1.0, worst


@pytest.mark.parametrize("tuning", [0, fa.FA_TUNE_BM_128, fa.FA_TUNE_BM_256])
@pytest.mark.parametrize("D,left,right", [(32, 63, 64), (128, 63, 64), (32, -1, -1)])
def test_key_bias_row_sums_are_kept_in_fp32(D, left, right, tuning):
    """lse of fp16 calls with a key bias comes from the probabilities before they are rounded to 16 bits: off by a few
    fp32 spacings, not by the 2^-12 of a rounded probability."""
    N = 600
    _, q, k, v = draw(4600 + D, 1, 2, N, D, "fp16", qk_gain=1.7)
    bias = round_to_storage(np.random.default_rng(D).standard_normal((1, N)).astype(np.float32), "fp16")
    o, lse = run_ex(q, k, v, None, "fp16", D ** -0.5, left, right, key_bias=bias,
                    tuning=tuning | (0 if left < 0 else fa.FA_TUNE_WIN_TWO_PHASE))
    o_ref, lse_ref = attention_oracle(q, k, v, None, D ** -0.5, left, right, key_bias=bias)
    # scores up to 60 carry half an fp32 spacing (2^-19 there) per product step, the sum of up to 600 terms 2^-24 each
    assert np.abs(lse - lse_ref).max() <= 3e-5, np.abs(lse - lse_ref).max()
