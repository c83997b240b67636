"""GPU parity of the pipelined global kernel at the edges of its 64-key tiles (one key, one block, a block and one, whole tiles,
one past them) in every shape, with scores that jump at chosen keys, so that references have to be refreshed - in the first
and the second block of a tile, in the first, an inner and the masked last tile, several tiles in a row - and rows whose
first keys are all excluded.  Against the fp64 oracle with the bounds of the other parity tests."""
import numpy as np
import pytest

import paper_2603_12646_amd as fa
from oracle.attention_oracle import attention_oracle, attention_oracle_rows
from workloads import draw, round_to_storage

from tests.gpu_util import check_against, run_ex

pytestmark = pytest.mark.gpu

LENS = [1, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129, 192, 193, 255, 256, 321, 0]
N = 330


def inputs(head_dim, dtype, spikes):
    """Scores of about N(0, 1); key j of `spikes` scores about `spikes[j]` higher with every second query row."""
    _, q, k, v = draw(77, len(LENS), 2, N, head_dim, dtype)
    q[:, :, ::2, 0] = 4.0
    q[:, :, 1::2, 0] = 0.0
    k[:, :, :, 0] = 0.0
    for j, height in spikes.items():
        k[:, :, j, 0] = height * np.sqrt(head_dim) / 4.0
    return q, round_to_storage(k, dtype), v


@pytest.mark.parametrize("spikes", [{}, {40: 30.0}, {70: 14.0, 100: 28.0, 140: 42.0, 200: 300.0}, {5: 60.0, 64: 90.0, 320: 130.0}],
                         ids=["flat", "first_tile", "rising", "last_tile"])
@pytest.mark.parametrize("tuning", [fa.FA_TUNE_BM_128, fa.FA_TUNE_BM_256, fa.FA_TUNE_BM_512], ids=["128", "256", "512"])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("head_dim", [32, 64, 128])
def test_tile_edges_and_refreshes(head_dim, dtype, tuning, spikes):
    q, k, v = inputs(head_dim, dtype, spikes)
    scale = 1.0 / np.sqrt(head_dim)
    o_ref, lse_ref = attention_oracle(q, k, v, LENS, scale, -1, -1)
    o, lse = run_ex(q, k, v, LENS, dtype, scale, tuning=tuning)
    check_against(o, lse, o_ref, lse_ref, LENS, dtype, relative=True)   # (a spiked row is one V row: outputs of up to 4)


@pytest.mark.parametrize("first", [20, 40, 64, 100, 200])
@pytest.mark.parametrize("tuning", [fa.FA_TUNE_BM_128, fa.FA_TUNE_BM_256], ids=["128", "256"])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("head_dim", [32, 64, 128])
def test_bias_excludes_first_keys(head_dim, dtype, tuning, first):
    """No reference until key `first`: in the first or second block of a tile, or after whole excluded tiles."""
    q, k, v = inputs(head_dim, dtype, {150: 40.0})
    bias = np.zeros((len(LENS), N), dtype=np.float32)
    bias[:, :first] = -np.inf
    scale = 1.0 / np.sqrt(head_dim)
    o_ref, lse_ref = attention_oracle(q, k, v, LENS, scale, -1, -1, key_bias=bias)
    o, lse = run_ex(q, k, v, LENS, dtype, scale, tuning=tuning, key_bias=bias)
    check_against(o, lse, o_ref, lse_ref, LENS, dtype, relative=True)


@pytest.mark.parametrize("head_dim,rows", [(32, 128), (64, 256), (128, 128)])
@pytest.mark.parametrize("batch", [2, 3, 33, 64, 65])
def test_ragged_batch_order(batch, head_dim, rows):
    """Sequences taken by falling length (2 to 64 of them, of 640 tokens and more, on more workgroups than one round holds):
    every row of every one, with unsorted, equal, empty and out-of-range lengths.  65: as they come."""
    n, round_tiles = 650, 768 if rows == 128 and head_dim != 128 else 512
    tiles = (n + rows - 1) // rows
    heads = round_tiles // (tiles * batch) + 1
    assert tiles * batch * heads > round_tiles
    lens = np.random.Generator(np.random.PCG64(batch)).integers(-20, n + 20, batch)
    lens[0], lens[-1] = 333, 650
    lens[batch // 2] = lens[0]
    _, q, k, v = draw(5, batch, heads, n, head_dim, "fp16")
    h = sorted({0, heads // 2, heads - 1})          # (the oracle on three heads: all run the same code)
    o_ref, lse_ref = attention_oracle(q[:, h], k[:, h], v[:, h], lens, 0.25, -1, -1)
    o, lse = run_ex(q, k, v, lens, "fp16", 0.25, tuning=fa.FA_TUNE_BM_128 if rows == 128 else fa.FA_TUNE_BM_256)
    assert not np.isnan(o).any() and not np.isnan(lse).any()   # (outputs start as NaN)
    check_against(o[:, h], lse[:, h], o_ref, lse_ref, lens, "fp16", relative=True)


PAD_N, PAD_ENDS = 1100, [1, 64, 65, 300, 576, 588, 640, 1099]


def padded(head_dim, dtype, value):
    _, q, k, v = draw(9, len(PAD_ENDS), 1, PAD_N, head_dim, dtype)
    bias = np.zeros((len(PAD_ENDS), PAD_N), dtype=np.float32)
    for b, end in enumerate(PAD_ENDS):
        bias[b, end:] = value
    return q, k, v, bias


@pytest.mark.parametrize("value", [-65504.0, -np.inf, -750.0])
@pytest.mark.parametrize("tuning", [fa.FA_TUNE_BM_128, fa.FA_TUNE_BM_256], ids=["128", "256"])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("head_dim", [32, 64, 128])
def test_padding_by_bias_leaves_the_call(head_dim, dtype, tuning, value):
    """Tails of keys whose bias makes them count for nothing, fewer and more than the eight tiles from which they are looked
    at; in sequence 3 two keys of the tail count all the same, by their size."""
    q, k, v, bias = padded(head_dim, dtype, round_to_storage(np.float32([value]), dtype)[0])
    scale = 1.0 / np.sqrt(head_dim)
    if value == -750.0:
        q[3, :, :, 0] = 64.0
        k[3, :, [700, 1000], 0] = 900.0 / 64.0 / scale     # 150 above the bias, and above the ordinary keys
    o_ref, lse_ref = attention_oracle(q, round_to_storage(k, dtype), v, None, scale, -1, -1, key_bias=bias)
    o, lse = run_ex(q, round_to_storage(k, dtype), v, None, dtype, scale, tuning=tuning, key_bias=bias)
    check_against(o, lse, o_ref, lse_ref, None, dtype, relative=True)


@pytest.mark.parametrize("head_dim", [32, 64, 128])
def test_padding_by_bias_with_infinite_values(head_dim):
    """A probability of 0 times an infinite V is NaN, in the padding too: such a tail stays in the call."""
    q, k, v, bias = padded(head_dim, "fp16", -65504.0)
    v[3, :, 900, 5] = np.inf
    o, _ = run_ex(q, k, v, None, "fp16", 1.0 / np.sqrt(head_dim), tuning=fa.FA_TUNE_BM_128, key_bias=bias)
    assert np.isnan(o[3, :, :, 5]).all()
    assert np.isfinite(np.delete(o[3], 5, axis=-1)).all() and np.isfinite(np.delete(o, 3, axis=0)).all()


@pytest.mark.parametrize("tuning", [fa.FA_TUNE_BM_128, fa.FA_TUNE_BM_256], ids=["128", "256"])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("head_dim", [32, 64, 128])
def test_padding_by_bias_below_a_length(head_dim, dtype, tuning):
    """A length beside the bias: keys from it on do not exist, whatever q, k, v and the bias hold there, and the padded tail
    ends at it."""
    n, lens, ends = 1300, [1100, 1024, 1217, 1300], [300, 500, 640, 64]
    _, q, k, v = draw(11, len(lens), 1, n, head_dim, dtype)
    bias = np.zeros((len(lens), n), dtype=np.float32)
    for b, (length, end) in enumerate(zip(lens, ends)):
        bias[b, end:length] = -65504.0 if dtype == "fp16" else -65536.0
    o_ref, lse_ref = attention_oracle(q, k, v, lens, 0.125, -1, -1, key_bias=bias)
    for b, length in enumerate(lens):
        q[b, :, length:] = k[b, :, length:] = np.nan
        v[b, :, length:] = np.inf
        bias[b, length:] = np.nan
    o, lse = run_ex(q, k, v, lens, dtype, 0.125, tuning=tuning, key_bias=bias)
    check_against(o, lse, o_ref, lse_ref, lens, dtype, relative=True)


def one_jump_per_row(head_dim, dtype, n, lens, heads, height=20.0):
    """Row i scores `height` higher with one key of tile i % 16 than with the others of N(0, 1): each tile refreshes some rows."""
    _, q, k, v = draw(78, len(lens), heads, n, head_dim, dtype)
    q[..., :16], k[..., :16] = 0.0, 0.0
    for g in range(16):
        q[:, :, g::16, g] = 4.0
        k[:, :, 64 * g + 37 * g % 64, g] = height * np.sqrt(head_dim) / 4.0
    return q, round_to_storage(k, dtype), v


# (head_dim 128 forms its scores in one of two ways, by the number of 128-row tiles: 18 and 360 here)
@pytest.mark.parametrize("head_dim,heads", [(32, 1), (64, 1), (128, 1), (128, 20)])
@pytest.mark.parametrize("tuning", [fa.FA_TUNE_BM_128, fa.FA_TUNE_BM_256, fa.FA_TUNE_BM_384, fa.FA_TUNE_BM_512, fa.FA_TUNE_BM_MIXED],
                         ids=["128", "256", "384", "512", "mixed"])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
def test_refresh_in_every_tile(head_dim, heads, dtype, tuning):
    n, lens = 1100, [1100, 1061]
    if tuning == fa.FA_TUNE_BM_MIXED:
        lens = lens[1:]
    q, k, v = one_jump_per_row(head_dim, dtype, n, lens, heads)
    scale = 1.0 / np.sqrt(head_dim)
    o_ref, lse_ref = attention_oracle(q[:, -1:], k[:, -1:], v[:, -1:], lens, scale, -1, -1)
    o, lse = run_ex(q, k, v, lens, dtype, scale, tuning=tuning)
    check_against(o[:, -1:], lse[:, -1:], o_ref, lse_ref, lens, dtype, relative=True)


@pytest.mark.parametrize("head_dim,heads", [(32, 1), (64, 1), (128, 1), (128, 12)])
@pytest.mark.parametrize("tuning", [fa.FA_TUNE_BM_128, fa.FA_TUNE_BM_256], ids=["128", "256"])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
def test_long_excluded_prefixes(head_dim, heads, dtype, tuning):
    """Sequences whose first keys, up to all of them, are excluded: no key counts for many tiles, then rows take their first
    reference in the middle of a tile, at its edge, in the last tile or never; one of those keys scores far higher."""
    n, first = 900, [0, 33, 64, 500, 511, 640, 863, 864, 899, 900]
    _, q, k, v = draw(79, len(first), heads, n, head_dim, dtype)
    bias = np.zeros((len(first), n), dtype=np.float32)
    for b, j in enumerate(first):
        bias[b, :j] = -np.inf
    q[..., 0], k[..., 0] = 4.0, 0.0
    k[:, :, 870, 0] = 7.0 * np.sqrt(head_dim)
    k = round_to_storage(k, dtype)
    scale = 1.0 / np.sqrt(head_dim)
    o_ref, lse_ref = attention_oracle(q[:, -1:], k[:, -1:], v[:, -1:], None, scale, -1, -1, key_bias=bias)
    o, lse = run_ex(q, k, v, None, dtype, scale, tuning=tuning, key_bias=bias)
    assert (o[-1] == 0).all() and np.isneginf(lse[-1]).all()
    check_against(o[:, -1:], lse[:, -1:], o_ref, lse_ref, None, dtype, relative=True)


@pytest.mark.parametrize("kind", ["zeros", "tail", "tail_and_hole", "tail_and_bias", "first_key_biased"])
@pytest.mark.parametrize("tuning", [fa.FA_TUNE_BM_128, fa.FA_TUNE_BM_256], ids=["128", "256"])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("head_dim", [32, 64, 128])
def test_bias_of_zeros_but_for_padding(head_dim, dtype, tuning, kind):
    """Calls whose bias is zeros and padding run a loop without a bias, others one with; every tile refreshes some rows.  Zeros of
    either sign give the bits of a call without a bias (head_dim 32 sums other values then)."""
    n, ends = 1100, [1100, 1099, 700, 641]
    q, k, v = one_jump_per_row(head_dim, dtype, n, ends, 1)
    bias = np.zeros((len(ends), n), dtype=np.float32)
    bias[:, 1::2] = -0.0
    if kind != "zeros":
        for b, end in enumerate(ends):
            bias[b, end:] = -65504.0
        bias = round_to_storage(bias, dtype)
    if kind == "tail_and_hole":
        bias[:, 300:340] = -np.inf
    if kind == "tail_and_bias":
        bias[:, 600] = 1.5
    if kind == "first_key_biased":
        bias[:, 0] = -2.0
    scale = 1.0 / np.sqrt(head_dim)
    o_ref, lse_ref = attention_oracle(q, k, v, None, scale, -1, -1, key_bias=bias)
    o, lse = run_ex(q, k, v, None, dtype, scale, tuning=tuning, key_bias=bias)
    check_against(o, lse, o_ref, lse_ref, None, dtype, relative=True)
    if kind == "zeros" and head_dim != 32:
        # (head_dim 128 with a bias has 128-row tiles only)
        o0, lse0 = run_ex(q, k, v, None, dtype, scale, tuning=fa.FA_TUNE_BM_128 if head_dim == 128 else tuning)
        assert np.array_equal(o, o0) and np.array_equal(lse, lse0)


FEW_ENDS = [1, 4, 8, 31, 32, 33, 40]


@pytest.mark.parametrize("value", [-65504.0, -np.inf])
@pytest.mark.parametrize("tuning", [fa.FA_TUNE_BM_128, fa.FA_TUNE_BM_256], ids=["128", "256"])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("head_dim", [32, 64, 128])
def test_few_keys_before_padding_by_bias(head_dim, dtype, tuning, value):
    """Sequences of a few keys, the padding behind them scoring far higher but for its bias: a row's reference is one of the keys
    that count, and the bits are the same whatever finite numbers the padding holds."""
    n = 700
    _, q, k, v = draw(83, len(FEW_ENDS), 2, n, head_dim, dtype, qk_gain=1.5)
    bias = np.zeros((len(FEW_ENDS), n), dtype=np.float32)
    for b, end in enumerate(FEW_ENDS):
        bias[b, end:] = value
    bias = round_to_storage(bias, dtype)
    scale = 1.0 / np.sqrt(head_dim)
    want = None
    for k_times, v_times in ((8.0, 1.0), (4.0, 30.0), (1.0, 1.0), (0.0, 0.0)):
        k2, v2 = k.copy(), v.copy()
        for b, end in enumerate(FEW_ENDS):
            k2[b, :, end:] *= k_times
            v2[b, :, end:] *= v_times
        k2, v2 = round_to_storage(k2, dtype), round_to_storage(v2, dtype)
        if want is None:
            o_ref, lse_ref = attention_oracle(q, k2, v2, None, scale, -1, -1, key_bias=bias)
        o, lse = run_ex(q, k2, v2, None, dtype, scale, tuning=tuning, key_bias=bias)
        check_against(o, lse, o_ref, lse_ref, None, dtype, relative=True, label=f"few keys D{head_dim} {dtype} K {k_times}")
        want = want or (o, lse)
        assert np.array_equal(o, want[0]) and np.array_equal(lse, want[1]), k_times


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("head_dim", [32, 64, 128])
@pytest.mark.parametrize("n", [641, 1023, 2049, 4611])
def test_padding_is_found_at_any_alignment_and_step(n, head_dim, dtype):
    """Bias rows of odd length start at odd 16-bit offsets; the padding begins at the edges of every step of the search, alone, with a
    hole or a single bias somewhere before it, or with a last key behind it that counts."""
    ends = sorted({e for s in range(0, n, 512) for e in (s + 1, s + 8, s + 505, s + 512) if e <= n} | {n - 1, n})
    rng = np.random.default_rng(n)
    _, q, k, v = draw(91, len(ends), 1, n, head_dim, dtype, qk_gain=1.5)
    scale = 1.0 / np.sqrt(head_dim)
    rows = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, 6)]))
    for kind in ("padding", "hole", "bias", "last"):
        bias = np.zeros((len(ends), n), dtype=np.float32)
        for b, end in enumerate(ends):
            if kind == "last":
                bias[b, max(0, end - 40):n - 1] = -65504.0
            else:
                bias[b, end:] = -65504.0
            if kind == "hole":
                bias[b, rng.integers(0, end) // 2] = -np.inf if end > 1 else 0.0
            if kind == "bias":
                bias[b, rng.integers(0, end)] = 2.5
        bias = round_to_storage(bias, dtype)
        o, lse = run_ex(q, k, v, None, dtype, scale, tuning=fa.FA_TUNE_BM_128, key_bias=bias)
        for b in range(len(ends)):
            o_ref, lse_ref = attention_oracle_rows(q, k, v, b, 0, rows, n, scale, key_bias=bias)
            check_against(o[b:b + 1, :, rows], lse[b:b + 1, :, rows], o_ref[None, None], lse_ref[None, None], None, dtype, relative=True,
                          label=f"{kind} D{head_dim} {dtype} end {ends[b]} of {n}")
