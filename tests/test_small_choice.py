"""The host's choice of the small kernel, of the split kernel whose rows follow the length and of the tile rows of a key bias, walked on the CPU with stub launchers."""
import pathlib
import shutil
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parent.parent

HEAD = r"""
#include <algorithm>
#include <climits>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <initializer_list>
#include "fa.h"
#include "fa_args.h"
static FaKernelArgs last;
static int last_bm;
int fa_launch_f16(const FaKernelArgs& a, int bm, int, int, void*) { last = a; last_bm = bm; return 0; }
int fa_launch_bf16(const FaKernelArgs& a, int bm, int, int, void*) { last = a; last_bm = bm; return 0; }
int fa_launch_rope_rotate(const FaRopeArgs&, int, void*) { return 0; }
int fa_static_scratch(void**) { return 0; }
alignas(16) static char buf[64];
alignas(16) static float table[64];
static fa_params call(int d, int b, int h, int n) {
  fa_params p;
  std::memset(&p, 0, sizeof p);
  p.struct_size = sizeof p;
  p.q = p.k = p.v = p.o = buf;
  p.scale = 0.125f;
  p.window_left = p.window_right = -1;
  p.head_dim = d; p.batch = b; p.heads = h; p.max_len = n;
  return p;
}
#define EXPECT(cond) do { if (!(cond)) { printf("FAILED line %d: %s (d %d b %d h %d n %d window %d %d bias %d: small %x)\n", __LINE__, #cond, \
  p.head_dim, p.batch, p.heads, p.max_len, p.window_left, p.window_right, p.key_bias != nullptr, last.small); return 1; } } while (0)
"""

WINDOWS = HEAD + r"""
// The kernels that local layers have otherwise: two-sided windows of at most five blocks for 32 rows (eight for 128) run kernels that
// sum rounded fp16 probabilities, as the small kernel does; windows past the tensor on both sides run the global kernel, which does too.
int main() {
  long small = 0, calls = 0;
  for (int d : {32, 64, 128})
    for (int biased = 0; biased < 2; ++biased)
      for (int n : {1, 20, 31, 32, 40, 63, 64, 65, 96, 100, 128, 129, 160, 161, 300, 487})
        for (int left : {-1, 0, 7, 31, 50, 63, 64, 96, 127, 128, 129, 200, 1000, INT_MAX})
          for (int right : {-1, 0, 7, 31, 40, 64, 96, 127, 128, 129, 200, 1000, INT_MAX}) {
            if (left < 0 && right < 0) continue;
            fa_params p = call(d, 1, 3, n);
            p.key_bias = biased ? buf : nullptr;
            p.window_left = left; p.window_right = right;
            EXPECT(fa_fwd_ex(&p) == 0);
            ++calls;
            const bool l = left >= 0 && left < n, r = right >= 0 && right < n;   // limits inside the tensor
            const bool held = l && r && (127 + right) / 32 + (left + 31) / 32 + 1 <= 8;
            EXPECT(!last.small || held || (!l && !r));
            EXPECT(!held || last.small == 0x51);   // (three heads: these fit one round)
            small += last.small != 0;
          }
  // heads of K or V that 32-bit offsets do not span: the masked kernel
  for (int which = 0; which < 2; ++which) {
    fa_params p = call(64, 1, 3, 487);
    p.window_left = 63; p.window_right = 64;
    int64_t* st = which ? p.v_strides : p.k_strides;
    st[0] = st[1] = 64;
    st[2] = 4000000;
    EXPECT(fa_fwd_ex(&p) == 0 && last.small == 0x51);
    st[2] = 5000000;
    EXPECT(fa_fwd_ex(&p) == 0 && last.small == 0);
  }
  printf("ok %ld of %ld\n", small, calls);
  return 0;
}
"""

BIAS_ROWS = HEAD + r"""
// 12 heads of 64: the larger tiles where no kind of bias loses by them, in both types
int main() {
  struct { int b, n, rows; } want[] = {{8, 2048, 256}, {16, 1024, 256}, {20, 2100, 256}, {10, 2048, 256}, {1, 16384, 256}, {4, 2500, 256},
                                       {2, 12000, 128}, {12, 1000, 128}, {6, 2048, 128}, {1, 8192, 128}, {9, 1200, 128}};
  for (auto& w : want)
    for (int dtype : {FA_DTYPE_F16, FA_DTYPE_BF16}) {
      fa_params p = call(64, w.b, 12, w.n);
      p.key_bias = buf; p.dtype = dtype;
      EXPECT(fa_fwd_ex(&p) == 0 && last_bm == w.rows);
    }
  printf("ok\n");
  return 0;
}
"""

SHAPES = HEAD + r"""
// What a launch of the small kernel counts on: the shape exists for the head size, no 32-row tile sees more key blocks than it holds
// (counted row by row), the grid is made of 32-row tiles, and the workgroups of one round fit the LDS of 256 units.
int main() {
  long taken = 0;
  for (int d : {32, 64, 128})
    for (int b : {1, 2, 3, 5, 8, 16})
      for (int h : {1, 3, 8, 12, 24, 31})
        for (int n = 1; n < 1500; n += 1 + n / 11)
          for (int w = 0; w < 7; ++w) {
            const int sides[7][2] = {{-1, -1}, {63, 64}, {0, 0}, {128, 0}, {0, 128}, {31, 33}, {5000, 600}};
            fa_params p = call(d, b, h, n);
            p.window_left = sides[w][0]; p.window_right = sides[w][1];
            p.key_bias = w & 1 ? buf : nullptr;
            EXPECT(fa_fwd_ex(&p) == 0);
            if (!last.small) continue;
            ++taken;
            const int s = last.small, nk = s >> 4, nb = s & 15;
            EXPECT(s == 0x51 || s == 0x41 || s == 0x42 || (s == 0x82 && d != 128));
            for (int q0 = 0; q0 < n; q0 += 32) {
              int lo = n, hi = -1;   // keys that a row of the tile sees
              for (int i = q0; i < q0 + 32 && i < n; ++i) {
                lo = std::min(lo, p.window_left < 0 ? 0 : std::max(0, i - p.window_left));
                hi = std::max(hi, p.window_right < 0 ? n - 1 : (int)std::min<long>(n - 1, (long)i + p.window_right));
              }
              EXPECT(hi / 32 - lo / 32 + 1 <= nk * nb);
            }
            EXPECT(last_bm == 32 && last.n_qtiles == (n + 31) / 32 && last.total_tiles == last.n_qtiles * h * b && last.map_xcd);
            EXPECT(!last.heads_first && !last.longest_first && !last.split && !last.live_tiles);
            const long ids = 8L * last.xcd_per * b, block = 32 * d * 2, lds = block + nk * 2 * nb * block + nk * 2 * 64 * 4 + nk * nb * 128;
            EXPECT(ids >= last.total_tiles && ids <= 256 * (160 * 1024 / lds));
          }
  printf("ok %ld\n", taken);
  return taken < 3000;
}
"""

SIZES = HEAD + r"""
// The last call of each shape and head size, of a model's 24, 12 and 8 heads, and the first past it
int main() {
  struct { int d, b, n, window, small; } want[] = {
      {32, 1, 704, 1, 0x51}, {32, 1, 705, 1, 0}, {32, 1, 512, 0, 0x82}, {32, 2, 384, 0, 0}, {32, 4, 256, 0, 0x42}, {32, 5, 256, 0, 0},
      {32, 7, 128, 0, 0x41}, {32, 8, 128, 0, 0}, {64, 1, 1344, 1, 0x51}, {64, 1, 1376, 1, 0}, {64, 1, 512, 0, 0x82}, {64, 1, 513, 0, 0},
      {64, 5, 256, 0, 0x42}, {64, 6, 256, 0, 0}, {64, 16, 128, 0, 0x41}, {64, 17, 128, 0, 0}, {128, 1, 1024, 1, 0x51}, {128, 1, 1025, 1, 0},
      {128, 4, 256, 0, 0x42}, {128, 1, 257, 0, 0}, {128, 16, 128, 0, 0x41}, {128, 17, 128, 0, 0}};
  for (auto& w : want)
    for (int dtype : {FA_DTYPE_F16, FA_DTYPE_BF16})
      for (int lengths = 0; lengths < 2; ++lengths) {
        fa_params p = call(w.d, w.b, 768 / (w.d == 128 ? 96 : w.d), w.n);
        if (w.window) p.window_left = 63, p.window_right = 64;
        p.dtype = dtype;
        p.seq_lens = lengths ? (const int32_t*)table : nullptr;
        EXPECT(fa_fwd_ex(&p) == 0 && last.small == w.small);
      }
  printf("ok\n");
  return 0;
}
"""

LIVE = HEAD + r"""
int main() {
  long taken = 0;
  for (int h = 1; h <= 300; ++h)
    for (int n = 1; n < 40000; n += 1 + n / 50)
      for (int dtype : {FA_DTYPE_F16, FA_DTYPE_BF16}) {
        fa_params p = call(64, 1, h, n);
        p.dtype = dtype;
        p.seq_lens = (const int32_t*)table;
        EXPECT(fa_fwd_ex(&p) == 0);
        const int live = last.live_tiles;
        if (live) {
          // one round, every row of the tensor in a tile of 128 rows, and tiles of 96 rows would not do
          EXPECT(live > 0 && live * h <= 256 && (long)live * 128 >= n && (long)live * 96 < n && n >= 2000);
          ++taken;
          p.batch = 2; EXPECT(fa_fwd_ex(&p) == 0 && !last.live_tiles); p.batch = 1;
          p.seq_lens = nullptr; EXPECT(fa_fwd_ex(&p) == 0 && !last.live_tiles); p.seq_lens = (const int32_t*)table;
          p.key_bias = buf; EXPECT(fa_fwd_ex(&p) == 0 && !last.live_tiles); p.key_bias = nullptr;
          p.rope_cos = p.rope_sin = table; EXPECT(fa_fwd_ex(&p) == 0 && !last.live_tiles); p.rope_cos = p.rope_sin = nullptr;
          p.window_left = 63; p.window_right = 64; EXPECT(fa_fwd_ex(&p) == 0 && !last.live_tiles); p.window_left = p.window_right = -1;
          p.tuning = FA_TUNE_BM_128; EXPECT(fa_fwd_ex(&p) == 0 && !last.live_tiles); p.tuning = 0;
          p.head_dim = 128; EXPECT(fa_fwd_ex(&p) == 0 && !last.live_tiles); p.head_dim = 64;
        }
        // (bf16: the split kernel's own lines have left the call to it)
        const int per = h <= 256 ? 256 / h : 0;
        EXPECT((live != 0) == (per && (n + 127) / 128 <= per && (n + 95) / 96 > per && n >= 2000));
      }
  printf("ok %ld\n", taken);
  return 0;
}
"""


def run(tmp_path, text):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    src, exe, csrc = tmp_path / "driver.cpp", tmp_path / "driver", ROOT / "paper_2603_12646_amd" / "csrc"
    src.write_text(text)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", str(ROOT / "include"),
                    "-I", str(csrc), str(src), str(csrc / "fa_api.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr


def test_local_layers_that_take_the_small_kernel(tmp_path):
    run(tmp_path, WINDOWS)


def test_what_a_launch_of_the_small_kernel_counts_on(tmp_path):
    run(tmp_path, SHAPES)


def test_last_calls_of_the_small_kernel(tmp_path):
    run(tmp_path, SIZES)


def test_tile_rows_of_a_key_bias(tmp_path):
    run(tmp_path, BIAS_ROWS)


def test_rows_by_the_length(tmp_path):
    run(tmp_path, LIVE)
