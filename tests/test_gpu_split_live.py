"""GPU parity of the split kernel whose tile rows follow the length of the one sequence (64, 96 or 128 rows on one workgroup
per compute unit) against the fp64 oracle: the lengths at which the rows change, one key, none, the whole tensor, and lengths
out of range; every row past the sequence is zero."""
import numpy as np
import pytest
import torch

import paper_2603_12646_amd as fa
from oracle.attention_oracle import attention_oracle_rows
from workloads import draw

from tests.gpu_util import LSE_TOL, TOL, run_ex

pytestmark = pytest.mark.gpu


# (heads, max_len, lengths); that these calls run this kernel in either type is checked on the CPU.  12 heads: 21 tiles each, so up
# to 1344, 2016 and 2688 rows; 15 heads: 17 tiles, up to 1088, 1632, 2176
CASES = [(12, 2049, [2049, 2048, 2017, 2016, 1900, 1345, 1344, 700, 31, 1, 0, -5, 4000]), (15, 2160, [2160, 1633, 1632, 1089, 1088, 300])]


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("H,N,lens", CASES)
def test_rows_follow_the_length(H, N, lens, dtype):
    _, q, k, v = draw(8200 + N, 1, H, N, 64, dtype, qk_gain=1.5)
    for n in lens:
        x = [t.copy() for t in (q, k, v)]
        live = min(max(n, 0), N)
        for t in x:
            t[:, :, live:] = np.nan
        o, lse = run_ex(*x, [n], dtype, 0.125)
        assert (o[:, :, live:] == 0).all() and np.isneginf(lse[:, :, live:]).all(), n
        if live == 0:
            continue
        rows = np.unique(np.concatenate([np.arange(0, min(live, 70)), np.arange(max(0, live - 70), live),
                                         np.random.default_rng(n).integers(0, live, 64)]))
        for h in (0, H - 1):
            o_ref, lse_ref = attention_oracle_rows(q, k, v, 0, h, rows, live, 0.125)
            # (rows with a peaked softmax have outputs of 2 and more, which as bf16 numbers are by themselves up to 7.8e-3 off: against
            # their magnitude, as in the other tests)
            assert (np.abs(o[0, h, rows] - o_ref) / np.maximum(1.0, np.abs(o_ref))).max() <= TOL[dtype]["max_abs"], (n, h)
            assert np.abs(lse[0, h, rows] - lse_ref).max() <= LSE_TOL, (n, h)
        assert np.isfinite(o).all() and np.isfinite(lse[:, :, :live]).all()
        if n in (lens[0], lens[4]):   # workgroup ids as they come: the same bits
            o2, lse2 = run_ex(*x, [n], dtype, 0.125, tuning=fa.FA_TUNE_MAP_LINEAR)
            assert np.array_equal(o, o2) and np.array_equal(lse, lse2), n


def test_without_lse_and_a_row_refreshed_late():
    """No lse, and keys of ever higher scores: references taken anew in every shape's steps."""
    H, N = 12, 2048
    _, q, k, v = draw(8300, 1, H, N, 64, "bf16")
    q[..., 0], k[..., 0] = 4.0, 0.0
    for i, j in enumerate(range(50, N, 150)):
        k[:, :, j, 0] = 16.0 * (i + 1)
    for n in (1000, 1990, 2048):
        o, _ = run_ex(q, k, v, [n], "bf16", 0.125, want_lse=False)
        rows = np.arange(0, n, 37)
        o_ref, _ = attention_oracle_rows(q, k, v, 0, 5, rows, n, 0.125)
        # (a row is nearly one V row: its magnitude)
        assert (np.abs(o[0, 5, rows] - o_ref) / np.maximum(1.0, np.abs(o_ref))).max() <= TOL["bf16"]["max_abs"], n
        assert (o[:, :, n:] == 0).all()
