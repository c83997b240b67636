"""The host's choice of a split-kernel shape, walked on the CPU with stub launchers: a shape is one the kernels exist in,
its grid matches its rows per workgroup and its ids fit the 256 compute units in one round, and calls that the kernel does not
cover (windows, a rotation in the call, a long key bias, forced shapes) never get one.  And the GPU tests of the kernels of small
calls: each of their calls launches the kernel that it is there for."""
import pathlib
import shutil
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parent.parent

DRIVER = r"""
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
#define EXPECT(cond) do { if (!(cond)) { printf("FAILED line %d: %s (d %d b %d h %d n %d bias %d split %x bm %d)\n", __LINE__, #cond, \
  p.head_dim, p.batch, p.heads, p.max_len, p.key_bias != nullptr, last.split, last_bm); return 1; } } while (0)
int main(int argc, char** argv) {
  alignas(16) static char buf[64];
  alignas(16) static float table[64];
  fa_params p;
  std::memset(&p, 0, sizeof p);
  p.struct_size = sizeof p;
  p.q = p.k = p.v = p.o = buf;
  p.scale = 0.125f;
  p.window_left = p.window_right = -1;
  if (argc > 1) {   // the kernels of the calls given as: head_dim batch heads max_len biased bf16 lengths window_left window_right
    for (int i = 1; i + 8 < argc; i += 9) {
      p.head_dim = std::atoi(argv[i]); p.batch = std::atoi(argv[i + 1]); p.heads = std::atoi(argv[i + 2]);
      p.max_len = std::atoi(argv[i + 3]); p.key_bias = std::atoi(argv[i + 4]) ? buf : nullptr;
      p.dtype = std::atoi(argv[i + 5]) ? FA_DTYPE_BF16 : FA_DTYPE_F16;
      p.seq_lens = std::atoi(argv[i + 6]) ? (const int32_t*)table : nullptr;
      p.window_left = std::atoi(argv[i + 7]); p.window_right = std::atoi(argv[i + 8]);
      if (fa_fwd_ex(&p) != 0) return 1;
      if ((last.small != 0) + (last.live_tiles != 0) + (last.split != 0) > 1) return 2;
      if (last.small) printf("small-%x\n", last.small);
      else if (last.live_tiles) printf("live\n");
      else if (last.split) printf("split-%x\n", last.split);
      else printf("other\n");
    }
    return 0;
  }
  long taken = 0, calls = 0;
  for (int d : {32, 64, 128})
    for (int b : {1, 2, 3, 5, 8, 32})
      for (int h : {1, 4, 8, 12, 24, 86})
        for (int n = 1; n < 5000; n += 1 + n / 7)
          for (int biased = 0; biased < 2; ++biased) {
            p.head_dim = d; p.batch = b; p.heads = h; p.max_len = n;
            p.key_bias = biased ? buf : nullptr;
            p.rope_cos = p.rope_sin = nullptr; p.tuning = 0; p.scale = 0.125f;
            p.window_left = p.window_right = -1;
            EXPECT(fa_fwd_ex(&p) == 0);
            ++calls;
            if (last.split) {
              ++taken;
              const int nq = last.split >> 4, s = last.split;
              EXPECT(d == 64 ? (s == 0x18 || s == 0x24 || s == 0x34 || (biased ? s == 0x42 : s == 0x14 || s == 0x22))
                             : (d == 128 ? (s == 0x14 || s == 0x24 || s == 0x42) : (s == 0x14 || s == 0x22)));
              EXPECT(last_bm == 32 * nq && last.n_qtiles == (n + 32 * nq - 1) / (32 * nq));
              // every XCD's eighth of each batch element's tiles, rounded up, is launched: these ids have to fit in one round
              const long ids = 8L * last.xcd_per * b, round = s == 0x22 ? 768 : (d == 32 && !biased ? 512 : 256);
              EXPECT(last.total_tiles == last.n_qtiles * b * h && ids >= last.total_tiles && ids <= round);
              EXPECT(!biased || n <= kSplitBiasKeys);
            }
            p.window_left = 63; p.window_right = 64;
            EXPECT(fa_fwd_ex(&p) == 0 && last.split == 0);
            p.window_left = p.window_right = -1; p.rope_cos = p.rope_sin = table;
            EXPECT(fa_fwd_ex(&p) == 0 && last.split == 0);
            p.rope_cos = p.rope_sin = nullptr; p.tuning = FA_TUNE_BM_128;
            EXPECT(fa_fwd_ex(&p) == 0 && last.split == 0);
            p.tuning = FA_TUNE_V_SCALAR;
            EXPECT(fa_fwd_ex(&p) == 0 && last.split == 0);
            p.tuning = 0; p.scale = 0.0f;
            EXPECT(fa_fwd_ex(&p) == 0 && (!biased || last.split == 0));
          }
  // no shape is there for one size: of one sequence of 1 - 48 heads each is taken for many head counts, and at many lengths (the
  // narrowest, head_dim 64 on four wavefronts of 32 rows, at 513 - 639 tokens where lengths are given: half of them here)
  p.scale = 0.125f; p.batch = 1; p.tuning = 0;
  for (int d : {32, 64, 128})
    for (int biased = 0; biased < 2; ++biased) {
      static int head_counts[256], lengths[256];
      std::memset(head_counts, 0, sizeof head_counts);
      std::memset(lengths, 0, sizeof lengths);
      for (int h = 1; h <= 48; ++h) {
        bool here[256] = {};
        for (int n = 65; n <= kSplitBiasKeys; ++n) {
          p.dtype = n & 1 ? FA_DTYPE_BF16 : FA_DTYPE_F16;
          p.seq_lens = n & 2 ? (const int32_t*)table : nullptr;
          p.head_dim = d; p.heads = h; p.max_len = n; p.key_bias = biased ? buf : nullptr;
          if (fa_fwd_ex(&p) != 0) return 1;
          here[last.split] = true;
          ++lengths[last.split];
        }
        for (int s = 0; s < 256; ++s) head_counts[s] += here[s];
      }
      for (int s = 1; s < 256; ++s)
        if (lengths[s] && (head_counts[s] < 12 || lengths[s] < 50 * head_counts[s])) {
          printf("FAILED head_dim %d bias %d shape %x: %d head counts, %d lengths\n", d, biased, s, head_counts[s], lengths[s]);
          return 1;
        }
    }
  p.scale = 0.125f; p.key_bias = buf; p.batch = 1; p.heads = 1; p.head_dim = 64;
  p.max_len = kSplitBiasKeys; EXPECT(fa_fwd_ex(&p) == 0 && last.split != 0);
  p.max_len = kSplitBiasKeys + 1; EXPECT(fa_fwd_ex(&p) == 0 && last.split == 0);
  printf("ok %ld of %ld\n", taken, calls);
  return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    tmp_path = tmp_path_factory.mktemp("driver")
    src, exe, csrc = tmp_path / "driver.cpp", tmp_path / "driver", ROOT / "paper_2603_12646_amd" / "csrc"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", str(ROOT / "include"),
                    "-I", str(csrc), str(src), str(csrc / "fa_api.cpp"), "-o", str(exe)], check=True)
    return str(exe)


def test_split_shapes_chosen_by_the_host(driver):
    r = subprocess.run([driver], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok "), r.stdout + r.stderr


def kernels(driver, calls):
    """The kernel of each call (head_dim, batch, heads, max_len, biased, bf16, lengths, window_left, window_right)."""
    r = subprocess.run([driver, *[str(int(x)) for c in calls for x in c]], capture_output=True, text=True, check=True)
    got = r.stdout.split()
    assert len(got) == len(calls)
    return got


@pytest.mark.parametrize("bf16", [0, 1])
def test_gpu_cases_run_the_shapes_they_are_named_after(driver, bf16):
    """The calls of the GPU tests of the split kernel launch the shape written beside them, and every shape that any call gets is among
    them."""
    from tests.test_gpu_split import CASES, LENGTHS, SHAPES
    cases = [(name, D, len(lens), H, N, biased, 1, s) for name, (D, H, N, lens, biased, s) in CASES.items()]
    cases += [("shape " + name, D, 1, H, N, False, name in LENGTHS, s) for name, (D, H, N, s) in SHAPES.items()]
    got = kernels(driver, [(D, B, H, N, biased, bf16, lengths, -1, -1) for _, D, B, H, N, biased, lengths, _ in cases])
    assert list(zip([c[0] for c in cases], got)) == [(c[0], f"split-{c[-1]:x}") for c in cases]
    assert {(D, biased, s) for _, D, _, _, _, biased, _, s in cases} == {
        (64, 0, 0x14), (64, 0, 0x18), (64, 0, 0x24), (64, 0, 0x34), (64, 0, 0x22), (128, 0, 0x14), (128, 0, 0x24), (128, 0, 0x42),
        (32, 0, 0x14), (32, 0, 0x22), (64, 1, 0x18), (64, 1, 0x24), (64, 1, 0x34), (64, 1, 0x42), (128, 1, 0x14), (128, 1, 0x24),
        (128, 1, 0x42), (32, 1, 0x14), (32, 1, 0x22)}


@pytest.mark.parametrize("bf16", [0, 1])
def test_gpu_cases_of_the_kernel_whose_rows_follow_the_length(driver, bf16):
    from tests.test_gpu_split_live import CASES
    calls = [(64, 1, H, N, 0, bf16, 1, -1, -1) for H, N, _ in CASES] + [(64, 1, 12, 2048, 0, 1, 1, -1, -1)]
    assert kernels(driver, calls) == ["live"] * len(calls)


@pytest.mark.parametrize("bf16", [0, 1])
def test_gpu_cases_of_the_small_kernel(driver, bf16):
    from tests.test_gpu_small import GLOBAL, RANGE, WINDOWS
    for D in (32, 64, 128):
        for biased in (0, 1):
            got = kernels(driver, [(D, len(lens), 3, max(lens), biased, bf16, 1, left, right) for left, right, lens in WINDOWS])
            # (open on one side, or more than five blocks for 32 rows: the kernels of such windows; six sequences of head_dim 128 are
            # more than one round)
            assert got == ["other" if (left, right) in {(7, 100), (50, -1), (-1, 40)} or (D == 128 and len(lens) == 6) else "small-51"
                           for left, right, lens in WINDOWS]
            got = kernels(driver, [(D, len(lens), 3, max(lens), biased, bf16, 1, -1, -1) for lens in GLOBAL])
            assert got == ["small-41", "small-41", "small-42", "small-42"] + (["split-14"] * 2 if D == 128 else ["small-82"] * 2)
    got = kernels(driver, [(D, 1, H, N, 0, bf16, 0, left, right) for D, H, N, left, right in RANGE])
    for (D, H, N, left, right), kernel in zip(RANGE, got):
        inside = (D, H, N, left) in {(64, 16, 1024, 63), (128, 8, 1024, 63), (32, 24, 704, 63), (64, 16, 512, -1), (32, 24, 512, -1), (128, 32, 256, -1)}
        assert kernel.startswith("small") == inside, (D, H, N, left, kernel)


HEADS_FIRST_DRIVER = r"""
#include <cstdio>
#include <vector>
#include "fa_mix_map.h"
int main() {
  long walks = 0;
  for (int heads : {1, 3, 12, 24, 31})
    for (int tiles = 1; tiles < 60; ++tiles)
      for (int live_tiles = 0; live_tiles <= tiles; live_tiles += 1 + tiles / 9) {
        const int total = heads * tiles, live = heads * live_tiles, per = (total + 7) / 8;
        std::vector<int> seen(total, 0);
        for (int x = 0; x < 8; ++x) {
          int mine = 0;
          for (int jb = 0; jb < per; ++jb) {
            const int u = fa_heads_first_tile(x, jb, per, live, total);
            if (u < -1 || u >= total) { printf("FAILED range %d\n", u); return 1; }
            if (u >= 0) ++seen[u];
            mine += u >= 0 && u < live;
          }
          if (mine > (live + 7) / 8) { printf("FAILED share %d of %d\n", mine, live); return 1; }
        }
        for (int u = 0; u < total; ++u)
          if (seen[u] != 1) { printf("FAILED heads %d tiles %d live %d: tile %d seen %d times\n", heads, tiles, live_tiles, u, seen[u]); return 1; }
        ++walks;
      }
  printf("ok %ld\n", walks);
  return 0;
}
"""


def test_heads_first_order_hands_out_every_tile_once(tmp_path):
    """Every workgroup id of the heads-first order walked on the CPU: each tile once, and no XCD more than its eighth of
    the tiles below the sequence length."""
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(HEADS_FIRST_DRIVER.replace("#include <vector>", "#include <initializer_list>\n#include <vector>"))
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I",
                    str(ROOT / "paper_2603_12646_amd" / "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok "), r.stdout + r.stderr


BIAS_ROPE_DRIVER = r"""
#include <cstdio>
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
int main() {
  alignas(16) static char buf[64];
  alignas(16) static float table[64];
  fa_params p;
  std::memset(&p, 0, sizeof p);
  p.struct_size = sizeof p;
  p.q = p.k = p.v = p.o = buf;
  p.key_bias = buf;
  p.rope_cos = p.rope_sin = table;
  p.scale = 0.125f;
  p.window_left = p.window_right = -1;
  for (int d : {32, 64, 128})
    for (int b : {1, 4})
      for (int h : {1, 24})
        for (int n : {64, 400, 3000, 8192, 40000})
          for (unsigned bm : {FA_TUNE_BM_AUTO, FA_TUNE_BM_128, FA_TUNE_BM_256, FA_TUNE_BM_32, FA_TUNE_BM_384, FA_TUNE_BM_512, FA_TUNE_BM_MIXED}) {
            p.head_dim = d; p.batch = b; p.heads = h; p.max_len = n; p.tuning = bm;
            if (fa_fwd_ex(&p) != 0 || last_bm != 128 || last.split || last.n_qtiles != (n + 127) / 128) {
              printf("FAILED d %d b %d h %d n %d tuning %u: bm %d, %d tiles\n", d, b, h, n, bm, last_bm, last.n_qtiles);
              return 1;
            }
          }
  // a scale by which a bias cannot be divided in fp32: the masked kernel as well, said to the launcher by inv_abs_scale = 0
  p.rope_cos = p.rope_sin = nullptr;
  p.tuning = 0;
  for (int d : {32, 64, 128})
    for (int n : {300, 8192})
      for (float s : {0.0f, 1e-45f, 1e-39f, -1e-36f, 1e-34f, 3e-34f, -0.125f, 8.0f}) {
        p.head_dim = d; p.batch = 1; p.heads = 24; p.max_len = n; p.scale = s;
        const bool divides = s > 2e-34f || s < -2e-34f;
        if (fa_fwd_ex(&p) != 0 || (last.inv_abs_scale > 0.f) != divides || (!divides && (last_bm != 128 || last.split))) {
          printf("FAILED d %d n %d scale %g: bm %d split %x inv %g\n", d, n, s, last_bm, last.split, last.inv_abs_scale);
          return 1;
        }
      }
  printf("ok\n");
  return 0;
}
"""


def test_bias_with_a_rotation_in_the_call_or_a_tiny_scale_keeps_the_masked_kernels_rows(tmp_path):
    """A key bias together with a rotation inside the call, or with a scale that it cannot be divided by, runs the masked
    kernel, whose workgroups hold 128 rows: the grid has to be made of 128-row tiles whatever the size or the forced shape,
    or the rows past the first tiles stay unwritten."""
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    src, exe, csrc = tmp_path / "driver.cpp", tmp_path / "driver", ROOT / "paper_2603_12646_amd" / "csrc"
    src.write_text(BIAS_ROPE_DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", str(ROOT / "include"), "-I", str(csrc), str(src),
                    str(csrc / "fa_api.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
