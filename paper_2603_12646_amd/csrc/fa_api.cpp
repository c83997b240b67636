// Host side of the C boundary declared in include/fa.h: argument validation,
// mapping of the public arguments to the kernel argument block, kernel-shape
// choice.  Nothing here touches device memory; validation failures return before
// any HIP call.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstdint>
#include <cstring>

#include "fa.h"
#include "fa_args.h"
#include "fa_mix_map.h"

namespace {

constexpr float kLog2e = 1.44269504088896340736f;
constexpr float kTauLog2 = 8.0f;  // p = exp2(s*c - m*c) is allowed to reach 2^8 before m is refreshed

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

bool all_zero(const int64_t s[3]) { return s[0] == 0 && s[1] == 0 && s[2] == 0; }

void dense_strides(int64_t out[3], int heads, int max_len, int head_dim) {
  out[2] = head_dim;
  out[1] = (int64_t)max_len * head_dim;
  out[0] = (int64_t)heads * max_len * head_dim;
}

int resolve_strides(const int64_t in[3], int64_t out[3], int heads, int max_len, int head_dim) {
  if (all_zero(in)) {
    dense_strides(out, heads, max_len, head_dim);
    return FA_OK;
  }
  for (int i = 0; i < 3; ++i) {
    if (in[i] % 8 != 0) return FA_ERR_MISALIGNED;
    out[i] = in[i];
  }
  if (in[2] < head_dim) return FA_ERR_BAD_SHAPE;  // rows may not overlap
  if (in[2] > (1 << 24)) return FA_ERR_BAD_SHAPE;  // per-thread tile offsets are 32-bit
  return FA_OK;
}

// The output rows of different (batch, head, row) must not overlap, or workgroups would race
// on them: order the three axes by stride; each stride must cover the extent of the faster
// axes below it (head_dim contiguous elements innermost).  Axes of extent 1 are not stepped.
// Dense, [batch, len, heads, dim] and packed layouts pass; zero, negative or interleaving
// strides do not.
bool output_rows_disjoint(const int64_t st[3], int batch, int heads, int max_len, int head_dim) {
  int64_t stride[3] = {st[0], st[1], st[2]};
  int64_t extent[3] = {batch, heads, max_len};
  for (int i = 0; i < 3; ++i)
    for (int j = i + 1; j < 3; ++j)
      if (stride[j] < stride[i]) {
        int64_t t = stride[i]; stride[i] = stride[j]; stride[j] = t;
        t = extent[i]; extent[i] = extent[j]; extent[j] = t;
      }
  long double covered = head_dim;
  for (int i = 0; i < 3; ++i) {
    if (extent[i] <= 1) continue;
    if (stride[i] <= 0 || (long double)stride[i] < covered) return false;
    covered = (long double)stride[i] * (long double)extent[i];
  }
  return true;
}

// One sequence can take the mixed-shape kernel (it splits the rows between 256-row and 128-row
// workgroups itself, from the sequence length); heads <= 256 keeps the 128-row workgroups left
// over by an odd tile count within the ids the launch reserves for them.
bool mixed_fits(const fa_params& p) {
  const int64_t tiles = ((int64_t)p.max_len + 127) / 128;
  return p.batch == 1 && p.heads <= 256 && tiles * p.heads <= (1 << 20) && fa_mix_ids((int)tiles, p.heads) >= 0;
}

// Relative time of a global layer under a tile shape, from how its workgroups
// fill 256 compute units: full rounds of `slots` workgroups per unit cost slots * blocks each
// (blocks = 32-row query blocks per workgroup), a partly filled last round costs less (its
// workgroups have their SIMDs more to themselves), and `rel` is the shape's cost per block
// relative to the 256-row shape.  Fitted to sweeps of 2K - 32K tokens x 8 - 32 heads of head_dim 64 on MI355X; the callers
// say by `rel` what differs for a bias, a rotation and the other head sizes.
double shape_cost(int64_t workgroups, int slots, int blocks, double rel) {
  const int64_t per_round = 256LL * slots;
  const int64_t full = workgroups / per_round, rest = workgroups % per_round;
  double rounds = (double)full;
  if (rest) {
    const double f = (double)rest / (double)per_round;
    double part = 1.0;
    if (slots == 3) part = f <= 1.0 / 3 ? 0.45 : (f <= 2.0 / 3 ? 0.75 : 1.0);
    if (slots == 2) part = f <= 0.5 ? 0.62 : 1.0;
    rounds += part;
  }
  return rounds * slots * blocks * rel;
}

int choose_bm(const fa_params& p, bool allow_mixed) {
  // Query rows per workgroup (0 = the mixed-shape kernel).  256 (two 32-row blocks per
  // wavefront) halves LDS and L2 traffic per flop and 512 (eight wavefronts on one K/V stage)
  // halves the L2 traffic again, but the larger the tile the coarser the load balance over
  // 256 compute units; local windows (whose key range grows with the tile) take 128.
  const bool windowed = p.window_left >= 0 || p.window_right >= 0;
  if (windowed) return 128;
  const int64_t bh = (int64_t)p.batch * p.heads;
  const bool plain64 = p.head_dim == 64 && !p.key_bias && !p.rope_cos;
  // At head_dim 32 the key-bias variant has four wavefronts per SIMD on 128 rows and two on 256: us, 12 heads, 128 -> 256 rows,
  // 12 x 700 24.2 -> 27.5, 8 x 2048 95 -> 101, 1 x 10000 271 -> 286; nowhere of 40 calls in either type the other way.
  if (p.head_dim == 32 && p.key_bias) return 128;
  if (p.batch > 1 && p.max_len < 2048 && (p.seq_lens || plain64)) {
    // batches of short sequences (ragged lengths leave many tiles empty, which the model
    // below cannot see).  Measured: 768 tiles of 256 rows are 1-5 % faster at 128, 1536 and
    // more 2-7 % faster at 256.
    return (((int64_t)p.max_len + 255) / 256) * bh >= 4 * 256 ? 256 : 128;
  }
  const int64_t w128 = (((int64_t)p.max_len + 127) / 128) * bh;
  const int64_t w256 = (((int64_t)p.max_len + 255) / 256) * bh;
  const int64_t w512 = (((int64_t)p.max_len + 511) / 512) * bh;
  if (w128 <= 512) return 128;                      // at most two 128-row workgroups per unit
  // one sequence: pairs of one 256-row and one 128-row workgroup per unit (up to 768 tiles), or
  // rounds of 256-row pairs with 128-row workgroups on what remains (beyond 1024; between the
  // two a single round of the larger shapes does as well)
  if (allow_mixed && (w128 <= 768 || w128 > 1024) && mixed_fits(p)) return 0;
  // What a block of 128-row workgroups costs more: plain calls, and head_dim 32, 1.08.  A rotation in the call is done once per
  // query tile (us, 12 x 64, 128 -> 256 rows: 7 x 2048 138 -> 118, 12 x 2048 218 -> 193, but 6 x 2048 in a thin second round
  // of the larger ones 105 -> 115).  A key bias is padding as a rule, whose kernels make one pass over it per query tile; other
  // biases, which the host cannot tell from it, gain less by the larger tiles, and the line is where they do not lose: us, 12 x 64,
  // 128 -> 256 rows, padding from the half on, keys 100 - 130 excluded, fp16: 8 x 2048 105 -> 95, 122 -> 117; 16 x 1024 59.1 -> 55.1,
  // 67.4 -> 65.7; 20 x 2100 (1.13 here) 272 -> 246, 328 -> 311; 2 x 12000 (1.16) 742 -> 743, 945 -> 966; 12 x 1000 (1.23) 46.7 -> 51.0, 55 -> 64;
  // bf16: 8 x 2048 99 -> 92, 122 -> 115; 20 x 2100 264 -> 244, 326 -> 312; 2 x 12000 743 -> 729, 956 -> 964; 1 x 16384 521 -> 442, 882 -> 839.
  const double rel = p.head_dim == 32 ? 1.08 : (p.rope_cos ? 1.2 : (p.key_bias ? 1.15 : 1.08));
  const double c128 = shape_cost(w128, 3, 4, rel), c256 = shape_cost(w256, 2, 8, 1.0),
               c512 = shape_cost(w512, 1, 16, 0.98);
  if (c512 < c256 && c512 < c128 && w512 <= 256) return 512;   // 512 only where one round holds the call
  return c256 <= c128 ? 256 : 128;
}

// Shape of the split kernel for a global layer, 16 * NQ + NK (NQ blocks of 32 query rows per workgroup, each shared by
// NK wavefronts that split the keys), or 0 where the other kernels are faster.  A shape is taken only where the call's
// workgroups fit the 256 units in one round - a second, thin round costs as much as the first.  What has to fit are the
// IDS: every XCD takes an eighth of each batch element's tiles, rounded up, so 3 x 12 heads x 197 tokens are 252 tiles of 32
// rows but 264 ids.  The host knows max_len only, not the lengths.  (The small kernel has taken the smallest calls by then: of head
// size 64 those of up to 512 tokens and 256 ids of 32 rows, or 256 tokens and 512.)  All lines below are
// from a sweep of 1 - 16 sequences x 4 - 32 heads x 65 - 4096 tokens, full and at 0.7 and 0.45 of max_len, in both types;
// us per call, the 128 / 256-row kernels -> the shape:
//   head_dim 64   32 rows on eight wavefronts, 4 heads x 1024 13.8 -> 8.0; on four (two workgroups per unit) below 640 tokens where
//                 lengths are given: 540 7.2 (on eight, where every row is there, 6.9).
//                 64 rows: on four wavefronts, three workgroups per unit, 850 12.5 -> 10.4, 1024 13.6 -> 10.9, 1250
//                 16.1 -> 12.4; on eight where the workgroups are short, 2 x 400 7.9 (four: 8.1), 30
//                 heads x 330 7.3 (7.6), or nearly alone, 4 heads x 3500 36.4 -> 23.0 (26.3).
//                 96 rows (bf16): 1440 19.0 -> 17.4, 1750 21.7 -> 18.8, 2 x 880 13.5 -> 13.1; one sequence of 1000 tokens
//                 in a tensor of 2000 loses (12.3 -> 13.0), and of 400 in 880 more (8.9 -> 10.0), where a batch does not.
//                 64 rows, three per unit, beyond 256: where the 128-row kernel fits one round as well it pays for long
//                 sequences, in fp16 from 1000 tokens (15.1 -> 13.8; 2 x 740 12.5 -> 12.1) but in bf16, whose 128-row
//                 kernel spends less on the probabilities, from 2000 (2048 23.4 -> 22.8; 1024 14.1 -> 14.5; 2 x 1200 full
//                 17.1 -> 17.2, ragged 16.5 -> 15.1); where that kernel needs a thin second round, from 480 (3 x 880 20.1 -> 14.7,
//                 2900 49 -> 42; 6 x 400 12.0 -> 12.7).
//                 With a key bias, whose pipelined kernel is slower: 64 rows 600 12.6 -> 9.4, 96 rows 4 x 460 11.7 -> 10.7,
//                 128 rows 2400 43 -> 30, but 4 x 512 10.9 -> 11.5.
//   head_dim 128  32 rows: 512 13.6 -> 8.4;  64 rows: 2048 37 -> 24;  128 rows: 4 x 640
//                 16.8 -> 15.5, 4096 75 -> 65, but 8 x 512 15.6 -> 15.8.  With a bias 16 x 256 13.5 -> 12.3.
//   head_dim 32   32 rows (two workgroups per unit; with a bias one): 12 heads x 1024 11.8 -> 9.4;
//                 64 rows, three per unit, where the 128-row kernel has its thin second round: 1500 22.5 -> 20.7, 2048
//                 29.3 -> 26.7, but 2 x 700 11.9 -> 12.7.  With a bias 12 heads x 600 11.0 -> 7.2 in 32 rows, 1024
//                 15.6 -> 11.9 in 64; 2 x 24 heads x 470 9.7 -> 10.4.
int choose_split(const fa_params& p) {
  auto ids = [&](int rows) { return (((int64_t)p.max_len + rows - 1) / rows * p.heads + 7) / 8 * 8 * p.batch; };
  const int n = p.max_len;
  const bool bias = p.key_bias != nullptr, fp16 = p.dtype == FA_DTYPE_F16, one = p.batch == 1;
  if (n <= 64) return 0;
  if (p.head_dim == 64 && bias) {
    if (ids(64) <= 256) return ids(32) <= 256 ? 0x18 : 0x24;
    if (ids(96) <= 256 && n >= 448) return 0x34;
    if (ids(128) <= 256 && n >= 560) return 0x42;
  } else if (p.head_dim == 64) {
    if (ids(32) <= 256) return p.seq_lens && n < 640 ? 0x14 : 0x18;
    if (ids(64) <= 256) return n >= 1600 || n < 560 ? 0x24 : 0x22;
    if (ids(96) <= 256 && n >= (one ? 1200 : 860)) return 0x34;
    if (ids(128) <= 256) return n >= (fp16 ? (one ? 1000 : 700) : (one ? 2000 : 1100)) ? 0x22 : 0;
    if (ids(64) <= 768 && n >= 480) return 0x22;
  } else if (p.head_dim == 128) {
    if (ids(64) <= 256) return ids(32) <= 256 ? 0x14 : 0x24;
    if (ids(128) <= 256 && n >= (bias ? 256 : 640)) return 0x42;
  } else if (bias) {
    if (ids(64) <= 256) return ids(32) <= 256 ? 0x14 : 0x22;
    if (ids(64) <= 768 && (n >= 520 || (ids(128) > 256 && ids(64) <= 512))) return 0x22;
  } else {
    if (ids(32) <= 512 && n >= 256) return 0x14;
    if (ids(64) > 512 && ids(64) <= 768 && n >= 1000) return 0x22;
  }
  return 0;
}

// Tiles per head of the split kernel whose rows follow the length, or 0.  One sequence whose tensor is too long for one round of
// 96-row workgroups, but not for one of 128-row ones: it goes before the 64-row shape, of which up to two share a unit
// while others have one.  From 2000 tokens on, as that shape in bf16: below (more than 12 heads) full fp16 sequences lose, and bf16
// runs the 128-row kernel.  us, that shape -> it, bf16, fp16:
//   12 heads  1024 of 2048 13.7 -> 11.4, 13.8 -> 11.9; 1331 16.9 -> 12.8, 16.0 -> 13.0; 1638 19.0 -> 16.6, 17.9 -> 16.5; 1904 20.9 -> 18.1, 20.0 -> 18.3; 2048
//             22.2 -> 21.3, 21.1 -> 21.2; 2048 of 2560 22.3 -> 21.3, 21.2 -> 21.1; 2560 27.5 -> 26.6, 27.1 -> 27.0
//   8         960 of 3200 9.9 -> 10.3, 10.3 -> 10.4; 1600 13.3 -> 13.6, 13.9 -> 13.7; 2080 22.6 -> 18.4, 21.1 -> 18.2; 3200 31.3 -> 29.2, 30.2 -> 29.4
//   16        1000 of 2000 14.5 -> 12.0, 13.9 -> 11.9; 1600 18.1 -> 18.6, 17.6 -> 18.5; 2000 23.6 -> 22.6, 23.5 -> 22.9; fp16 1600 of 1600 17.7 -> 18.5
//   2         7763 of 12321 1.6 times as fast, 1.45; 14336 of 14336 1.04, 0.98
int choose_live(const fa_params& p) {
  if (p.head_dim != 64 || p.key_bias || !p.seq_lens || p.batch != 1 || p.heads > 256 || p.max_len < 2000) return 0;
  const int per = 256 / p.heads;
  return (p.max_len + 127) / 128 <= per && (p.max_len + 95) / 96 > per ? per : 0;
}

// Shape of the small kernel, 16 * wavefronts + key blocks of each, or 0: calls whose 32-row workgroups see at most as many key
// blocks as the shape holds, and fit one round of as many workgroups per unit as their LDS allows.  It goes before the kernel
// that the rules above choose.  us, fp16, the kernels before -> it:
//   local   12 x 64 200 tokens 6.7 -> 4.6, 487 6.9 -> 4.7, 690 (264 ids) 6.9 -> 5.0, 1300 (492) 7.05 -> 5.6, but 1600 7.1 -> 7.75; 8 x 128 487
//           8.6 -> 5.9, 1000 (256) 8.7 -> 6.0, but 1300 8.95 -> 10.0; 24 x 32 (in a graph, fp16, bf16) 300 5.5 -> 4.0, 5.5 -> 4.05; 700 (528) 5.6 -> 5.3,
//           5.6 -> 5.3, but 800 (600) 5.2 -> 5.65, 5.1 -> 5.9; 1000 (768) 5.5 -> 5.7, 5.6 -> 6.2.
//   global  12 x 64 110 tokens 4.8 -> 4.3, 16 x 128 (768) 6.7 -> 6.2, 200 5.4 -> 4.8, 5 x 250 (480) 6.55 -> 5.9, but 6 x 250 7.6 -> 8.4; 512 6.3 -> 5.5,
//           but 2 x 384 (288) 7.2 -> 8.9; 8 x 128 110 6.5 -> 5.3, 16 x 128 (512) 8.0 -> 7.4, 256 7.1 -> 5.8, but 5 x 250 (320) 8.4 -> 10.8; 24 x 32 110
//           4.9 -> 3.8, 7 x 110 (672; graph) 4.85 -> 4.7, but bf16 8 x 128 (768) 4.8 -> 4.9; 200 6.2 -> 4.2, 4 x 256 (768) 6.0 -> 5.55, but 5 x 250 6.3 -> 6.6; 512 (384)
//           6.6 -> 6.1, but 2 x 384 (576) 7.0 -> 7.8.
// Windows: those that the resident and two-phase kernels hold (limits on both sides, five blocks for 32 rows), whose sums and
// biased scores are rounded as here, and those that reach past the tensor on both sides.  Wider and one-sided ones stay with the
// kernels whose fp16 row sums are those of unrounded probabilities and whose biased scores are rounded once, and so do heads of K or V
// that 32-bit offsets do not span.
int choose_small(const fa_params& p, const FaKernelArgs& a, bool bias_can_be_divided) {
  if (p.rope_cos || (p.key_bias && !bias_can_be_divided)) return 0;
  const bool windowed = p.window_left >= 0 || p.window_right >= 0;
  const int64_t n = p.max_len, left = p.window_left < 0 || p.window_left >= n ? -1 : p.window_left,
                right = p.window_right < 0 || p.window_right >= n ? -1 : p.window_right;
  const int64_t all = (n + 31) / 32, window = (31 + right) / 32 + (left + 31) / 32 + 1, seen = left >= 0 && window < all ? window : all;
  if ((left < 0) != (right < 0) || (left >= 0 && (window > 5 || (double)n * (double)std::max(a.ks[2], a.vs[2]) * 2.0 >= 4.0e9))) return 0;
  const int64_t ids = (all * p.heads + 7) / 8 * 8 * p.batch;
  const int d = p.head_dim == 32 ? 0 : (p.head_dim == 64 ? 1 : 2);
  // most ids per shape and head size
  static constexpr int k41[3] = {672, 768, 512}, k42[3] = {768, 512, 256}, k51[3] = {528, 512, 256}, k82[3] = {384, 256, 0};
  if (windowed) return seen <= 5 && ids <= k51[d] ? 0x51 : 0;
  if (seen <= 4) return ids <= k41[d] ? 0x41 : 0;
  if (seen <= 8) return ids <= k42[d] ? 0x42 : 0;
  return seen <= 16 && ids <= k82[d] ? 0x82 : 0;
}

}  // namespace

namespace {
// scratch / scratch_bytes: what the call may use (the caller's, or the library's static array);
// static_limit: reject a call that would use more scratch than it has instead of falling back
int fwd_ex_impl(const fa_params* p_in, void* scratch, size_t scratch_bytes, bool static_limit);
}  // namespace

extern "C" int fa_fwd_ex(const fa_params* p) {
  if (!p) return FA_ERR_NULL_POINTER;
  if (p->struct_size != sizeof(fa_params)) return FA_ERR_BAD_STRUCT;
  return fwd_ex_impl(p, p->scratch, p->scratch_bytes, false);
}

extern "C" size_t fa_rope_scratch_bytes(int batch, int heads, int max_len, int head_dim) {
  if (batch <= 0 || heads <= 0 || max_len <= 0 || head_dim <= 0) return 0;
  return (size_t)2 * (size_t)batch * (size_t)heads * (size_t)max_len * (size_t)head_dim * 2u;
}

extern "C" int fa_fwd_ex_static_scratch(const fa_params* p) {
  if (!p) return FA_ERR_NULL_POINTER;
  if (p->struct_size != sizeof(fa_params)) return FA_ERR_BAD_STRUCT;
  // only a rotation on a global layer uses scratch: every other call never touches the array
  const bool uses_scratch = p->rope_cos && p->window_left < 0 && p->window_right < 0;
  void* ptr = nullptr;
  if (uses_scratch) {
    const int rc = fa_static_scratch(&ptr);
    if (rc != 0) return rc;
  }
  return fwd_ex_impl(p, ptr, uses_scratch ? (size_t)FA_STATIC_SCRATCH_BYTES : 0, true);
}

namespace {
int fwd_ex_impl(const fa_params* p_in, void* scratch, size_t scratch_bytes, bool static_limit) {
  fa_params local = *p_in;
  const fa_params* p = &local;
  if (p->dtype != FA_DTYPE_F16 && p->dtype != FA_DTYPE_BF16) return FA_ERR_BAD_DTYPE;
  if (!p->q || !p->k || !p->v || !p->o) return FA_ERR_NULL_POINTER;
  if (p->batch <= 0 || p->heads <= 0 || p->max_len <= 0) return FA_ERR_BAD_SHAPE;
  if (p->head_dim != 32 && p->head_dim != 64 && p->head_dim != 128) return FA_ERR_BAD_HEAD_DIM;
  // the element count must stay inside int64 (before any stride arithmetic is done with it)
  if ((long double)p->batch * p->heads * p->max_len * p->head_dim > 9.0e18L || p->max_len > (1 << 30))
    return FA_ERR_BAD_SHAPE;
  if (!std::isfinite(p->scale)) return FA_ERR_BAD_SCALE;
  if (!aligned16(p->q) || !aligned16(p->k) || !aligned16(p->v) || !aligned16(p->o))
    return FA_ERR_MISALIGNED;
  if (p->lse && (reinterpret_cast<uintptr_t>(p->lse) & 3u)) return FA_ERR_MISALIGNED;
  if (p->key_bias && (reinterpret_cast<uintptr_t>(p->key_bias) & 1u)) return FA_ERR_MISALIGNED;
  if (p->key_bias_stride < 0 || (p->key_bias && p->key_bias_stride != 0 && p->key_bias_stride < p->max_len))
    return FA_ERR_BAD_SHAPE;
  if ((p->rope_cos == nullptr) != (p->rope_sin == nullptr)) return FA_ERR_NULL_POINTER;
  if (p->rope_cos && (!aligned16(p->rope_cos) || !aligned16(p->rope_sin) || p->rope_stride % 4 != 0))
    return FA_ERR_MISALIGNED;
  if (p->rope_stride < 0 || (p->rope_cos && p->rope_stride != 0 && p->rope_stride < p->head_dim / 2))
    return FA_ERR_BAD_SHAPE;
  if (p->tuning & ~0x3337u) return FA_ERR_BAD_TUNING;  // bits of the four fields
  const unsigned t_bm = p->tuning & 0xFu, t_v = p->tuning & 0xF0u, t_map = p->tuning & 0xF00u;
  if (t_bm > FA_TUNE_BM_MIXED || t_v > FA_TUNE_V_SCALAR || t_map > FA_TUNE_MAP_XCD)
    return FA_ERR_BAD_TUNING;

  FaKernelArgs a;
  std::memset(&a, 0, sizeof(a));
  int rc;
  if ((rc = resolve_strides(p->q_strides, a.qs, p->heads, p->max_len, p->head_dim))) return rc;
  if ((rc = resolve_strides(p->k_strides, a.ks, p->heads, p->max_len, p->head_dim))) return rc;
  if ((rc = resolve_strides(p->v_strides, a.vs, p->heads, p->max_len, p->head_dim))) return rc;
  if ((rc = resolve_strides(p->o_strides, a.os, p->heads, p->max_len, p->head_dim))) return rc;
  if (!output_rows_disjoint(a.os, p->batch, p->heads, p->max_len, p->head_dim)) return FA_ERR_BAD_SHAPE;

  FaRopeArgs r;
  bool rotate_first = false;
  // A rotation on a global layer with scratch to spare: q and k are rotated once, ahead of the
  // attention kernel, into dense copies in the scratch; from here on the call is a plain one
  // on those copies (every tile shape is open to it again).
  if (p->rope_cos && p->window_left < 0 && p->window_right < 0) {
    const size_t need = fa_rope_scratch_bytes(p->batch, p->heads, p->max_len, p->head_dim);
    if (scratch && !aligned16(scratch)) return FA_ERR_MISALIGNED;
    if (static_limit && need > scratch_bytes) return FA_ERR_SCRATCH;
    if (scratch && scratch_bytes >= need) {
      rotate_first = true;
      std::memset(&r, 0, sizeof(r));
      r.q = p->q; r.k = p->k;
      r.q_out = scratch;
      r.k_out = static_cast<char*>(scratch) + need / 2;
      std::memcpy(r.qs, a.qs, sizeof r.qs);
      std::memcpy(r.ks, a.ks, sizeof r.ks);
      r.rope_cos = p->rope_cos; r.rope_sin = p->rope_sin;
      r.rope_stride = p->rope_stride ? p->rope_stride : p->head_dim / 2;
      r.batch = p->batch; r.heads = p->heads; r.max_len = p->max_len; r.head_dim = p->head_dim;
      local.q = r.q_out;   // (the rotation is enqueued below, once nothing can be refused any more)
      local.k = r.k_out;
      local.rope_cos = local.rope_sin = nullptr;
      dense_strides(a.qs, p->heads, p->max_len, p->head_dim);
      dense_strides(a.ks, p->heads, p->max_len, p->head_dim);
    }
  }

  // a key bias runs 128-row kernels only unless it can ride on the pipelined global kernel, which has no variant that
  // also rotates (a rotation done ahead of the call is gone from p by now)
  const bool windowed = p->window_left >= 0 || p->window_right >= 0;
  // The pipelined kernels hold a key's bias divided by |scale|.  Below |scale| = 2e-34 that leaves the range of fp32 for
  // biases that 16-bit types can hold (and 0 / |scale| is 0 * infinity); the masked kernel never divides.
  const float inv_abs_scale = p->scale != 0.0f ? 1.0f / std::fabs(p->scale) : 0.0f;
  const bool bias_can_be_divided = p->scale != 0.0f && std::isfinite(65504.0f * inv_abs_scale);
  const bool bias_on_masked_kernel =
      p->key_bias && (windowed || p->rope_cos || !bias_can_be_divided || (p->tuning & 0xF0u) == FA_TUNE_V_SCALAR);
  int bm = 128;
  if (p->head_dim == 64 && !bias_on_masked_kernel) {
    // 384 (12 wavefronts x 32 rows), 512 (8 wavefronts x 64 rows) and the mixed launch exist for
    // global layers without a key bias on the transpose-read path only
    const bool plain = !windowed && !p->key_bias && !p->rope_cos && t_v != FA_TUNE_V_SCALAR;
    bm = choose_bm(*p, plain);
    if (t_bm == FA_TUNE_BM_128) bm = 128;
    if (t_bm == FA_TUNE_BM_256) bm = 256;
    if (t_bm == FA_TUNE_BM_384 && plain) bm = 384;
    if (t_bm == FA_TUNE_BM_512 && plain) bm = 512;
    if (t_bm == FA_TUNE_BM_MIXED && plain && mixed_fits(*p)) bm = 0;
    if (!plain && bm == 512) bm = 256;
  } else if (p->head_dim == 128 && !windowed && !p->key_bias && !p->rope_cos && t_v != FA_TUNE_V_SCALAR) {
    // head_dim 128 global layers: 128 rows on four wavefronts (two workgroups per unit), or 256
    // rows on eight wavefronts sharing one pair of K/V stages (one per unit; 2-3 % faster where
    // its coarser tiles fill the units as well: 8K x 8 heads, 32K x 8 heads)
    const int64_t bh = (int64_t)p->batch * p->heads;
    const int64_t w128 = (((int64_t)p->max_len + 127) / 128) * bh, w256 = (((int64_t)p->max_len + 255) / 256) * bh;
    bm = shape_cost(w256, 1, 8, 1.0) < shape_cost(w128, 2, 4, 1.03) ? 256 : 128;
    // Where one round holds the 128-row workgroups of a batch with lengths they win by the empty tiles: us, 256 -> 128 rows, bf16,
    // 3 x 1500 (1000 -) 39.9 -> 34.0, 2 x 3500 (2000 -) 87 -> 73, but 7 x 1000 (900 -) 33.0 -> 35.4; one sequence, 1 x 8192 (7900) 222 -> 229;
    // full: 3 x 1500 40.3 -> 42.2, 2 x 3000 75.4 -> 79.6.
    if (w128 <= 512 && p->seq_lens && p->batch > 1) bm = 128;
    if (t_bm == FA_TUNE_BM_128) bm = 128;
    if (t_bm == FA_TUNE_BM_256) bm = 256;
  } else if (p->head_dim == 32 && !windowed && !bias_on_masked_kernel && t_v != FA_TUNE_V_SCALAR) {
    // head_dim 32 global layers: the pipelined kernel in its 128- and 256-row shapes, chosen by
    // the same fill model (it matches a sweep of 1K-32K tokens x 8-24 heads to within 1 %)
    bm = choose_bm(*p, false);
    if (bm == 512) bm = 256;
    if (t_bm == FA_TUNE_BM_128) bm = 128;
    if (t_bm == FA_TUNE_BM_256) bm = 256;
  }
  // The kernels of the smallest calls, at most one of them.  Split kernel (a workgroup's wavefronts split the keys as well as the
  // rows): global layers too small for the shapes above to give every SIMD two wavefronts.  Its key bias sits in LDS.
  int small = 0, live = 0, split = 0;
  if (t_bm == FA_TUNE_BM_AUTO && t_v != FA_TUNE_V_SCALAR && (!windowed || (p->tuning & 0xF000u) == 0)) small = choose_small(*p, a, bias_can_be_divided);
  if (small) bm = 32;
  if (!small && !windowed && !p->rope_cos && t_v != FA_TUNE_V_SCALAR && !bias_on_masked_kernel &&
      (!p->key_bias || p->max_len <= kSplitBiasKeys)) {
    if (t_bm == FA_TUNE_BM_AUTO) split = choose_split(*p);
    if (t_bm == FA_TUNE_BM_32 && p->head_dim == 64 && !p->key_bias) split = 0x18;
    if (t_bm == FA_TUNE_BM_AUTO && split) live = choose_live(*p);
    if (live) split = 0;
    if (split) bm = 32 * (split >> 4);
  }
  const int tile_rows = bm == 0 ? 128 : bm;   // (the mixed launch sizes its own grid)
  const int64_t n_qtiles = ((int64_t)p->max_len + tile_rows - 1) / tile_rows;
  const int64_t total = n_qtiles * p->batch * p->heads;
  // the grid must stay inside what the kernels index with
  if (total > 0x7FFFFFF0LL) return FA_ERR_BAD_SHAPE;

  a.q = p->q; a.k = p->k; a.v = p->v; a.o = p->o; a.lse = p->lse; a.seq_lens = p->seq_lens;
  a.batch = p->batch; a.heads = p->heads; a.max_len = p->max_len; a.head_dim = p->head_dim;
  a.key_bias = p->key_bias;
  a.kb_stride = p->key_bias_stride ? p->key_bias_stride : p->max_len;
  // (bfloat16 biases near the type's largest: the factor log2(e), under which they are infinite, before the division)
  a.bias_pre = p->dtype == FA_DTYPE_BF16 && std::fabs(p->scale) > 0.6931f ? kLog2e : 1.0f;
  a.inv_abs_scale = bias_can_be_divided ? inv_abs_scale / a.bias_pre : 0.0f;
  a.rope_cos = p->rope_cos;
  a.rope_sin = p->rope_sin;
  a.rope_stride = p->rope_stride ? p->rope_stride : p->head_dim / 2;
  const float c = std::fabs(p->scale) * kLog2e;
  a.c = c;
  a.negate_q = std::signbit(p->scale) && p->scale != 0.0f ? 1 : 0;
  float tau = c > 0.f ? kTauLog2 / c : FLT_MAX;
  if (!(tau < FLT_MAX)) tau = FLT_MAX;
  a.tau_raw = tau;
  // a window reaching past the sequence on one side is the same as unbounded there
  a.wl = p->window_left < 0 ? -1 : (p->window_left >= p->max_len ? -1 : p->window_left);
  a.wr = p->window_right < 0 ? -1 : (p->window_right >= p->max_len ? -1 : p->window_right);
  a.n_qtiles = (int32_t)n_qtiles;
  a.total_tiles = (int32_t)total;
  // Tiles of one (batch, head) read the same K/V; the XCD-aware order keeps them on one
  // XCD's L2 (measured: 4.6x fewer bytes fetched from the fabric at 8K x 12 heads, same time).
  a.map_xcd = t_map == FA_TUNE_MAP_LINEAR ? 0 : 1;
  // Local layers: the query tiles of one head in a row share the halo of their windows in the XCD's L2.  Two kinds of call
  // gain more from the heads of one query tile in a row, if an XCD's eighth is still several tiles deep: a rotation, whose
  // table rows (as many bytes as K and V) are the same for all heads - measured, us, bf16: head_dim 64 2K 8.7 -> 8.35, 3K
  // 11.4 -> 10.6, 5K 12.6 -> 11.5, 8K 16.3 -> 15.4, 4 x 4000 ragged 26.3 -> 25.1, 8 x 3000 38.2 -> 38.3, but 1K (8 tiles) 7.5 -> 7.7,
  // 16 x 1000 27.8 -> 29.1, 32 x 512 26.4 -> 27.1; 128 1400 (11 tiles) 12.0 -> 11.5, 4 x 1500 18.4 -> 17.7, 8K 26.4 -> 20.4; 32 3K
  // 10.0 -> 9.3, 8K 17.1 -> 16.3 - and heads of 32 side by side in a row, two of which share a 128-byte line: 32K packed 67 -> 53,
  // 2K 7.1 -> 6.8, 32 x 1024 (8 tiles) 51.8 -> 53.1.  (Other calls: 8K head_dim 64 12.7 -> 12.9, 32K 41.9 -> 48.1; a rotation at
  // head_dim 32 on dense tensors with padding, where the padding tiles then all come last: 16000 of 32768 48.5 -> 50.3.)
  a.heads_first = a.map_xcd && windowed && !small &&
                  ((p->rope_cos && n_qtiles >= (p->head_dim == 128 ? 11 : 16) && (p->head_dim != 32 || !p->seq_lens)) || (p->head_dim == 32 && n_qtiles >= 16 && a.ks[1] == 32 && a.ks[2] >= 64));
  // Ragged batches on the pipelined kernel: long sequences first, so that the short tiles fill the last round.  Finding the
  // r-th sequence takes a workgroup 1 us before its first load, which short tiles do not earn back: us, 12 x 64, as they
  // come -> longest first: 12 x 700 (300 -) 20.9 -> 20.1, 16 x 1024 (600 -) 49.1 -> 48.0, 3 x 16K (9000 -) 1476 -> 1465, but
  // 32 x 512 (256 -) 30.9 -> 30.3, (480 -) 36.7 -> 37.7; and where one round holds the call, nothing (6 x 700 8 x 128 23.6 -> 25.4).
  a.longest_first = a.map_xcd && !windowed && p->seq_lens && p->batch > 1 && p->batch <= 64 && p->max_len >= 640 &&
                    total > (bm == 128 && p->head_dim != 128 ? 768 : 512);
  const int64_t per = ((int64_t)p->heads * n_qtiles + 7) / 8;
  if (8 * per * p->batch > 0x7FFFFFF0LL) return FA_ERR_BAD_SHAPE;
  a.xcd_per = (int32_t)per;
  a.split = split;
  a.small = small;
  a.live_tiles = live;
  // (a launch of at most two workgroups per unit has nothing else to hide the read of the sequence length behind)
  a.late_n = total <= 512;
  a.mix_ids_a = bm == 0 ? fa_mix_ids((int)n_qtiles, p->heads) : 0;
  const int v_path = t_v == FA_TUNE_V_SCALAR ? 1 : 0;

  const unsigned t_win = p->tuning & 0xF000u;
  if (t_win > FA_TUNE_WIN_TWO_PHASE) return FA_ERR_BAD_TUNING;
  const int win_kernel = t_win == FA_TUNE_WIN_PIPELINED ? 1 : (t_win == FA_TUNE_WIN_TWO_PHASE ? 2 : 0);
  if (rotate_first) {
    const int rc_rot = fa_launch_rope_rotate(r, p->dtype == FA_DTYPE_BF16, p->stream);
    if (rc_rot != 0) return rc_rot;
  }
  return p->dtype == FA_DTYPE_F16 ? fa_launch_f16(a, bm, v_path, win_kernel, p->stream)
                                  : fa_launch_bf16(a, bm, v_path, win_kernel, p->stream);
}
}  // namespace

static int fwd_simple(int dtype, const void* q, const void* k, const void* v, void* o, float* lse,
                      int batch, int heads, const int32_t* seq_lens, int max_len, int head_dim,
                      float scale, int window, void* stream) {
  if (window == 0) return FA_ERR_BAD_WINDOW;
  fa_params p;
  std::memset(&p, 0, sizeof(p));
  p.struct_size = sizeof(p);
  p.dtype = dtype;
  p.q = q; p.k = k; p.v = v; p.o = o; p.lse = lse; p.seq_lens = seq_lens;
  p.batch = batch; p.heads = heads; p.max_len = max_len; p.head_dim = head_dim;
  p.scale = scale;
  if (window < 0) {
    p.window_left = p.window_right = -1;
  } else {
    p.window_left = (window - 1) / 2;
    p.window_right = window / 2;
  }
  p.stream = stream;
  p.tuning = 0;
  return fa_fwd_ex(&p);
}

extern "C" int fa_fwd(const void* q, const void* k, const void* v, void* o, float* lse, int batch,
                      int heads, const int32_t* seq_lens, int max_len, int head_dim, float scale,
                      int window, void* stream) {
  return fwd_simple(FA_DTYPE_F16, q, k, v, o, lse, batch, heads, seq_lens, max_len, head_dim, scale,
                    window, stream);
}

extern "C" int fa_fwd_bf16(const void* q, const void* k, const void* v, void* o, float* lse,
                           int batch, int heads, const int32_t* seq_lens, int max_len, int head_dim,
                           float scale, int window, void* stream) {
  return fwd_simple(FA_DTYPE_BF16, q, k, v, o, lse, batch, heads, seq_lens, max_len, head_dim, scale,
                    window, stream);
}

extern "C" size_t fa_workspace_bytes(int, int, int, int) { return 0; }

extern "C" const char* fa_strerror(int code) {
  switch (code) {
    case FA_OK: return "success";
    case FA_ERR_NULL_POINTER: return "q, k, v, o or params is NULL";
    case FA_ERR_BAD_SHAPE: return "batch, heads, max_len or a stride is out of range, or output rows overlap";
    case FA_ERR_BAD_HEAD_DIM: return "unsupported head_dim (supported: 32, 64, 128)";
    case FA_ERR_BAD_SCALE: return "scale is not finite";
    case FA_ERR_BAD_WINDOW: return "window must be negative (global) or >= 1 (fa_fwd, fa_fwd_bf16)";
    case FA_ERR_MISALIGNED: return "pointer not 16-byte aligned or stride not a multiple of 8";
    case FA_ERR_BAD_DTYPE: return "dtype must be FA_DTYPE_F16 or FA_DTYPE_BF16";
    case FA_ERR_BAD_STRUCT: return "fa_params.struct_size mismatch";
    case FA_ERR_BAD_TUNING: return "unknown tuning bits";
    case FA_ERR_SCRATCH: return "the call needs more scratch than the library's static array holds";
    default: return code > 0 ? "HIP runtime error" : "unknown error code";
  }
}

extern "C" int fa_version(void) { return FA_VERSION; }
