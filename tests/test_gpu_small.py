"""GPU parity of the small kernel (calls of one round of 32-row workgroups whose wavefronts hold all key blocks) and, where its range
ends, of the kernels beside it, against the fp64 oracle; which call runs which is checked on the CPU: block edges, windows that reach past the tensor or are open on one side, rows that see no key, padding that
holds anything, strided output, and the largest calls that take it beside the first that do not."""
import numpy as np
import pytest
import torch

import paper_2603_12646_amd as fa
from oracle.attention_oracle import attention_oracle
from workloads import draw, round_to_storage

from tests.gpu_util import FA_DT, check_against, poison, run_ex, to_dev

pytestmark = pytest.mark.gpu

# (windows that are open on one side or wider than five blocks for 32 rows run other kernels)
WINDOWS = [(63, 64, [450, 449, 64, 33, 1, 0]), (0, 0, [97, 96, 31]), (128, 0, [300, 129]), (0, 128, [300, 129]), (7, 100, [160, 128, 5]),
           (50, -1, [160, 159, 32]), (-1, 40, [131, 1]), (63, 64, [32]), (63, 64, [20])]


@pytest.mark.parametrize("bias", [False, True])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("left,right,lens", WINDOWS)
def test_windows_and_lengths(D, dtype, left, right, lens, bias):
    B, H, N = len(lens), 3, max(lens)
    _, q, k, v = draw(5000 + D + left, B, H, N, D, dtype)
    kb = None
    if bias:
        rng = np.random.default_rng(D)
        kb = round_to_storage(rng.standard_normal((B, N)).astype(np.float32), dtype)
        kb[rng.random((B, N)) < 0.2] = -np.inf
        kb[0, 20:280] = -np.inf          # whole windows without a key
    scale = -(D ** -0.5)
    o_ref, lse_ref = attention_oracle(q, k, v, lens, scale, left, right, key_bias=kb)
    for b, n in enumerate(lens):
        for x in (q, k, v):
            x[b, :, n:] = np.nan
    o, lse = run_ex(q, k, v, lens, dtype, scale, left, right, key_bias=kb)
    check_against(o, lse, o_ref, lse_ref, lens, dtype, relative=True, label=f"small D{D} {dtype} ({left},{right})")


# Global: four wavefronts with one block each, with two, eight with two (head_dim 128 has no such shape: 257 and 512 run the split kernel);
# lengths at the edges of blocks and of their number
GLOBAL = [[128, 97, 96, 1, 0], [20, 3], [129, 128, 31], [256, 255, 160, 33], [257, 129, 0], [512, 480, 289, 31]]


@pytest.mark.parametrize("bias", [False, True])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("lens", GLOBAL)
def test_global_lengths(D, dtype, lens, bias):
    B, H, N = len(lens), 3, max(lens)
    _, q, k, v = draw(5300 + D + N, B, H, N, D, dtype, qk_gain=1.7)
    kb = None
    if bias:
        rng = np.random.default_rng(D)
        kb = round_to_storage(rng.standard_normal((B, N)).astype(np.float32), dtype)
        kb[rng.random((B, N)) < 0.2] = -np.inf
        kb[0, :70] = -np.inf           # wavefronts without a key that counts
        kb[1, :] = -np.inf             # no key at all
    scale = -(D ** -0.5)
    o_ref, lse_ref = attention_oracle(q, k, v, lens, scale, key_bias=kb)
    for b, n in enumerate(lens):
        for x in (q, k, v):
            x[b, :, n:] = np.nan
    o, lse = run_ex(q, k, v, lens, dtype, scale, key_bias=kb)
    check_against(o, lse, o_ref, lse_ref, lens, dtype, relative=True, label=f"small D{D} {dtype} {lens}")


# (workgroups of one round: the most ids of each shape and head size, and one tile past them)
RANGE = [(64, 16, 1024, 63, 64), (64, 16, 1025, 63, 64), (128, 8, 1024, 63, 64), (128, 8, 1025, 63, 64), (32, 24, 704, 63, 64), (32, 24, 705, 63, 64),
         (32, 24, 1024, 63, 64), (32, 24, 1025, 63, 64), (64, 16, 512, -1, -1), (64, 17, 512, -1, -1), (32, 24, 512, -1, -1), (32, 25, 512, -1, -1),
         (128, 32, 256, -1, -1), (128, 33, 256, -1, -1)]


@pytest.mark.parametrize("D,H,N,left,right", RANGE)
def test_last_call_of_the_range_and_the_next(D, H, N, left, right):
    _, q, k, v = draw(5100 + D, 1, H, N, D, "fp16")
    o, lse = run_ex(q, k, v, None, "fp16", D ** -0.5, left, right)
    sel = [0, H - 1]
    o_ref, lse_ref = attention_oracle(q[:, sel], k[:, sel], v[:, sel], None, D ** -0.5, left, right)
    check_against(o[:, sel], lse[:, sel], o_ref, lse_ref, None, "fp16", relative=True, label=f"small range D{D} N{N}")
    assert np.isfinite(o).all() and np.isfinite(lse).all()


@pytest.mark.parametrize("D", [32, 64, 128])
def test_packed_input_and_output_in_rows_of_heads(D):
    """From a packed QKV buffer, without lse, into [batch, length, heads, D]: the bits of the dense call."""
    B, H, N, lens = 2, 4, 333, [333, 140]
    _, q, k, v = draw(5200 + D, B, H, N, D, "bf16")
    o, _ = run_ex(q, k, v, lens, "bf16", D ** -0.5, 63, 64)
    packed = torch.stack([to_dev(np.ascontiguousarray(x.transpose(0, 2, 1, 3)), "bf16") for x in (q, k, v)], dim=2)
    st = (N * 3 * H * D, D, 3 * H * D)
    o2 = poison((B, N, H, D), "bf16")
    fa.fa_fwd_ex(dtype=FA_DT["bf16"], q=packed[:, :, 0], k=packed[:, :, 1], v=packed[:, :, 2], o=o2,
                 seq_lens=torch.tensor(lens, dtype=torch.int32, device="cuda"), batch=B, heads=H, max_len=N, head_dim=D,
                 scale=D ** -0.5, window_left=63, window_right=64, q_strides=st, k_strides=st, v_strides=st,
                 o_strides=(N * H * D, D, H * D))
    torch.cuda.synchronize()
    assert np.array_equal(o2.double().cpu().numpy().transpose(0, 2, 1, 3), o)
