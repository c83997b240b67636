"""GPU parity of the split kernel (a workgroup's wavefronts split the keys as well as the rows) in every shape the
library picks by itself, at the edges of its steps: a step is 32 NK keys, so lengths around its multiples, shorter than
one step, one key and none; the ring is refilled where a sequence has more steps than slots.  Against the fp64 oracle
with the bounds of the other parity tests."""
import numpy as np
import pytest
import torch

import paper_2603_12646_amd as fa
from oracle.attention_oracle import attention_oracle, attention_oracle_rows
from workloads import draw, round_to_storage

from tests.gpu_util import FA_DT, check_against, poison, run_ex, to_dev

pytestmark = pytest.mark.gpu

# (head_dim, heads, max_len, lengths, key bias, 16 * NQ + NK): the shape is what the library chooses for the call in either
# type (checked on the CPU).  "long": more steps than two turns of the ring, so that the unrolled part of the loop runs.
CASES = {
    "d64_1x4": (64, 2, 600, [600, 129, 128, 0], False, 0x14),
    "d64_1x4_longest": (64, 4, 639, [639, 512, 513], False, 0x14),
    "d64_1x8": (64, 2, 700, [700, 256, 255, 0], False, 0x18),
    "d64_1x8_long": (64, 1, 1300, [1300, 1024, 513, 31], False, 0x18),
    "d64_2x4": (64, 12, 400, [400, 128], False, 0x24),
    "d64_2x4_long": (64, 4, 2100, [2090], False, 0x24),
    "d64_3x4": (64, 12, 900, [900, 865], False, 0x34),
    "d64_3x4_long": (64, 12, 1500, [1497], False, 0x34),
    "d64_3x4_other": (64, 16, 1290, [97], False, 0x34),
    "d64_2x2_short": (64, 8, 700, [150, 65], False, 0x22),
    "d64_2x2": (64, 35, 500, [500, 333], False, 0x22),
    "d64_2x2_padded": (64, 12, 1200, [1100, 700], False, 0x22),
    "d64_2x2_long": (64, 6, 2210, [2177, 2000], False, 0x22),
    "d128_1x4": (128, 2, 300, [300, 129, 128, 1], False, 0x14),
    "d128_1x4_long": (128, 2, 700, [700, 641], False, 0x14),
    "d128_2x4": (128, 30, 200, [200, 63], False, 0x24),
    "d128_2x4_long": (128, 8, 1400, [1300], False, 0x24),
    "d128_4x2_long": (128, 15, 700, [700, 577], False, 0x42),
    "d32_1x4": (32, 20, 300, [300, 161], False, 0x14),
    "d32_1x4_long": (32, 4, 1400, [1390], False, 0x14),
    "d32_2x2_long": (32, 20, 1010, [1010, 64], False, 0x22),
    "d64_1x8_bias": (64, 2, 600, [600, 256, 255, 1], True, 0x18),
    "d64_1x8_bias_long": (64, 1, 1400, [1400], True, 0x18),
    "d64_2x4_bias": (64, 12, 400, [400, 128], True, 0x24),
    "d64_2x4_bias_long": (64, 4, 1300, [1300, 1200], True, 0x24),
    "d64_3x4_bias": (64, 15, 700, [700, 641], True, 0x34),
    "d64_4x2_bias_long": (64, 24, 600, [600, 577], True, 0x42),
    "d128_1x4_bias": (128, 2, 300, [300, 129, 128, 1], True, 0x14),
    "d128_1x4_bias_long": (128, 2, 700, [700, 641], True, 0x14),
    "d128_2x4_bias": (128, 30, 200, [200, 63], True, 0x24),
    "d128_2x4_bias_long": (128, 8, 1400, [1300], True, 0x24),
    "d128_4x2_bias_long": (128, 15, 700, [700, 577], True, 0x42),
    "d32_1x4_bias": (32, 4, 600, [600, 161], True, 0x14),
    "d32_1x4_bias_long": (32, 2, 1400, [1390], True, 0x14),
    "d32_2x2_bias": (32, 20, 300, [300, 161], True, 0x22),
    "d32_2x2_bias_long": (32, 12, 1200, [1190], True, 0x22),
}


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_split_kernel_shapes(name, dtype):
    D, H, N, lens, biased, _ = CASES[name]
    B = len(lens)
    rng = np.random.default_rng(N + D)
    _, q, k, v = draw(7000 + N, B, H, N, D, dtype)
    bias = None
    if biased:
        # ordinary values, holes, and in the first element a whole first step excluded (its rows see no key until later)
        bias = round_to_storage(rng.standard_normal((B, N)).astype(np.float32), dtype)
        bias[rng.random((B, N)) < 0.2] = -np.inf
        bias[0, :260] = -np.inf
    scale = -(D ** -0.5) if biased else D ** -0.5
    o_ref, lse_ref = attention_oracle(q, k, v, lens, scale, key_bias=bias)
    for b, n in enumerate(lens):   # nothing stored in the padding may show
        for x in (q, k, v):
            x[b, :, n:] = np.nan
    o, lse = run_ex(q, k, v, lens, dtype, scale, key_bias=bias)
    check_against(o, lse, o_ref, lse_ref, lens, dtype, relative=True, label=name)
    o2, lse2 = run_ex(q, k, v, lens, dtype, scale, key_bias=bias, tuning=fa.FA_TUNE_MAP_LINEAR)
    assert np.array_equal(o, o2) and np.array_equal(lse, lse2)


@pytest.mark.parametrize("D", [32, 64, 128])
def test_split_kernel_packed_qkv(D):
    """Read from one [batch, len, 3, heads, dim] buffer, written as [batch, len, heads, dim]: the same bits as dense."""
    B, H, N = 2, 12, 333
    lens = [333, 100]
    _, q, k, v = draw(91, B, H, N, D, "bf16")
    o, lse = run_ex(q, k, v, lens, "bf16", D ** -0.5)
    packed = torch.stack([to_dev(np.ascontiguousarray(x.transpose(0, 2, 1, 3)), "bf16") for x in (q, k, v)], dim=2)
    st = (N * 3 * H * D, D, 3 * H * D)
    o2 = poison((B, N, H, D), "bf16")
    lse2 = torch.full((B, H, N), float("nan"), dtype=torch.float32, device="cuda")
    fa.fa_fwd_ex(dtype=FA_DT["bf16"], q=packed[:, :, 0], k=packed[:, :, 1], v=packed[:, :, 2], o=o2, lse=lse2,
                 seq_lens=torch.tensor(lens, dtype=torch.int32, device="cuda"), batch=B, heads=H, max_len=N, head_dim=D,
                 scale=D ** -0.5, q_strides=st, k_strides=st, v_strides=st, o_strides=(N * H * D, D, H * D))
    torch.cuda.synchronize()
    assert np.array_equal(o2.double().cpu().numpy().transpose(0, 2, 1, 3), o)
    assert np.array_equal(lse2.double().cpu().numpy(), lse)


@pytest.mark.parametrize("tuning", [fa.FA_TUNE_BM_128, fa.FA_TUNE_BM_256])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("N", [1, 33, 64, 65, 129, 640])
def test_key_bias_pipelined_kernel_head_dim_32(N, dtype, tuning):
    """The pipelined global kernel with a key bias at head_dim 32, in both tile shapes, on lengths around its 64-key tiles."""
    B, H, D = 2, 3, 32
    lens = [N, max(1, N - 40)]
    rng = np.random.default_rng(N)
    _, q, k, v = draw(8000 + N, B, H, N, D, dtype)
    bias = round_to_storage(rng.standard_normal((B, N)).astype(np.float32), dtype)
    bias[0, : N // 3] = -np.inf
    o_ref, lse_ref = attention_oracle(q, k, v, lens, 0.2, key_bias=bias)
    for b, n in enumerate(lens):
        for x in (q, k, v):
            x[b, :, n:] = np.nan
    o, lse = run_ex(q, k, v, lens, dtype, 0.2, key_bias=bias, tuning=tuning)
    check_against(o, lse, o_ref, lse_ref, lens, dtype, relative=True, label=f"bias d32 {N}")


# (head_dim, heads, max_len, 16 * NQ + NK): one call per shape the library picks without a key bias, more than one block per
# wavefront; LENGTHS: those that have the shape only where a length is given (the whole tensor here)
LENGTHS = {"d64_1x4"}
SHAPES = {"d64_1x4": (64, 2, 600, 0x14), "d64_1x8_short": (64, 2, 530, 0x18), "d64_1x8": (64, 1, 700, 0x18),
          "d64_2x4": (64, 4, 2100, 0x24), "d64_3x4": (64, 12, 1500, 0x34), "d64_2x2": (64, 12, 2500, 0x22),
          "d128_1x4": (128, 2, 600, 0x14), "d128_2x4": (128, 8, 1500, 0x24), "d128_4x2": (128, 8, 2600, 0x42),
          "d32_1x4": (32, 24, 600, 0x14), "d32_2x2": (32, 24, 1500, 0x22)}


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("name", sorted(SHAPES))
def test_split_kernel_first_block_without_a_finite_score(name, dtype):
    """Keys whose scores are -infinity fill the first block of one wavefront after the other: it takes its reference from a
    later block, and the keys of that block count - also where they are all so far below 0 that they vanish against 0."""
    D, H, N, _ = SHAPES[name]
    _, q, k, v = draw(7200 + N, 1, 1, N, D, dtype)
    rep = lambda x: np.repeat(x, H, axis=1)
    q[..., 0] = 1.0
    k[..., 0] = 0.0
    for g, shift in ((0, 0.0), (1, -40.0), (0, 40.0), (7, -40.0), (2, 0.0)):
        q2, k2 = q.copy(), k.copy()
        q2[..., 1], k2[..., 1] = 40.0, shift          # every score moved by 40 * shift * scale
        k2[..., 32 * g: 32 * g + 32, 0] = -np.inf
        o_ref, lse_ref = attention_oracle(q2, k2, v, None, D ** -0.5)
        o, lse = run_ex(rep(q2), rep(k2), rep(v), [N] if name in LENGTHS else None, dtype, D ** -0.5)
        check_against(o[:, :1], lse[:, :1], o_ref, lse_ref, None, dtype, label=f"{name} block {g} shift {shift}")
        assert (o == o[:, :1]).all() and (lse == lse[:, :1]).all()


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("name", sorted(SHAPES))
def test_split_kernel_merge_of_large_references(name, dtype):
    """Wavefronts whose references are large and differ: scores 1024000 + g / 8 in the blocks of number g mod 8, exact in
    fp32.  The probabilities of a wavefront are formed against its reference times log2(e) ROUNDED to fp32 (spacing 1/8
    here), so the merge has to weigh them against that same number; against the unrounded product a wavefront's share is
    up to 2^(1/16), 4 %, off.  Values are +1 and -1 by g's parity: a share that is off shows in o in full."""
    D, H, N, _ = SHAPES[name]
    g = np.arange(N) // 32 % 8
    q = np.zeros((1, H, N, D), np.float32)
    k = np.zeros((1, H, N, D), np.float32)
    q[..., 0], q[..., 1] = 1024.0, 1.0
    k[..., 0], k[..., 1] = 1000.0, g / 8
    v = np.zeros((1, H, N, D), np.float32)
    v[...] = np.where(g % 2 == 0, 1.0, -1.0)[:, None]
    w = np.exp(g / 8.0)
    want = (w * np.where(g % 2 == 0, 1.0, -1.0)).sum() / w.sum()
    o, lse = run_ex(q, k, v, [N] if name in LENGTHS else None, dtype, 1.0)
    # a probability is rounded to 2^-12 (fp16) or 2^-9 (bf16) of itself, o likewise
    assert np.abs(o - want).max() <= (2.0 ** -11 if dtype == "fp16" else 2.0 ** -8), np.abs(o - want).max()
    assert np.abs(lse - (1024000.0 + np.log(w.sum()))).max() <= 0.5   # eight fp32 spacings there


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("D,H,N,tuning", [(64, 1, 600, fa.FA_TUNE_BM_128), (64, 1, 600, fa.FA_TUNE_BM_256), (64, 12, 6000, 0),
                                          (128, 1, 600, fa.FA_TUNE_BM_128), (128, 1, 600, fa.FA_TUNE_BM_256),
                                          (32, 1, 600, fa.FA_TUNE_BM_128), (32, 1, 600, fa.FA_TUNE_BM_256)])
def test_pipelined_kernel_first_block_without_a_finite_score(D, H, N, tuning, dtype):
    """The same on the kernels that do not split the keys: rows whose scores against the first 32 keys are -infinity take
    their reference from a later block, also where all scores are far below 0 or where those of the second half, or of the
    ragged last tile (whose masked code refreshes by another rule), are higher."""
    _, q, k, v = draw(7300 + N, 1, 1, N, D, dtype)
    rep = lambda x: np.repeat(x, H, axis=1)
    q[..., 0], q[..., 1] = 1.0, 40.0
    k[..., 0], k[..., 1] = 0.0, 0.0
    k[..., :32, 0] = -np.inf
    for first, base, scale in ((N + 1, 0.0, D ** -0.5), (N // 2, 0.0, D ** -0.5), (N - 20, 0.0, D ** -0.5),
                               (N + 1, -40.0, D ** -0.5), (N + 1, 40.0, D ** -0.5), (N // 2, -40.0, 1.0)):
        k2, q2 = k.copy(), q.copy()
        if scale == 1.0:
            q2[..., 2:] *= 0.125                      # (the lowest reference is another one there)
        k2[..., 1] = base                             # every score moved by 40 * base * scale
        k2[..., first:, 1] = 4.0                      # 160 * scale higher from key `first` on
        rows = np.unique(np.concatenate([np.arange(0, 64), np.arange(N - 40, N)]))
        o_ref, lse_ref = attention_oracle_rows(q2, k2, v, 0, 0, rows, N, scale)
        o, lse = run_ex(rep(q2), rep(k2), rep(v), None, dtype, scale, tuning=tuning)
        check_against(o[:, :1, rows], lse[:, :1, rows], o_ref[None, None], lse_ref[None, None], None, dtype,
                      label=f"pipelined D{D} {tuning} from {first} base {base} scale {scale}")
