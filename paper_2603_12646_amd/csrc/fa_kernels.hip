// Flash-attention forward for gfx950 (MI355X): head_dim 64 (also 32 and 128), fp16 / bf16
// storage, fp32 accumulation, key-padding mask by sequence length, optional local window.
//
// The operation is softmax(scale * Q K^T + mask) V per (batch, head), evaluated
// one key block at a time with a running row maximum and row sum so that no
// n x n matrix is ever formed (paper Sec. 2.2; operator attributes scale,
// window_size_left/right and the 1-D padding mask from Sec. 4.1.3 and Eq. 1).
//
// Work decomposition (one workgroup = 4 wavefronts = 256 threads):
//   * a workgroup owns BM = 4*32*NQB query rows of one (batch, head); each
//     wavefront owns NQB blocks of 32 query rows and keeps their Q fragments,
//     running maximum / sum and the head_dim-wide output accumulator in registers;
//   * K and V are streamed through LDS, fetched from HBM/L2 ahead of the arithmetic
//     (in the main kernels with direct global->LDS loads into an unpadded, XOR-swizzled
//     tile; in the reference masked kernel through registers into a padded tile).
//
// Matrix-core mapping (v_mfma_f32_32x32x16_{f16,bf16}, D = A * B + C with
// A: 32 x 16, B: 16 x 32, C: 32 x 32; lane l holds A[l%32][8*(l/32)..+7],
// B[8*(l/32)..+7][l%32] and C[8*(r/4) + 4*(l/32) + r%4][l%32] for r = 0..15):
//   * scores are computed TRANSPOSED, S^T = K * Q^T, so that a lane's 16
//     accumulator values all belong to ONE query (column l%32) and 16 different
//     keys.  Row maxima and sums are then in-lane reductions plus a single
//     exchange between lane l and lane l^32;
//   * the same accumulator registers, rounded to 16 bits and packed, are exactly a
//     B operand of the second product O^T = V^T * P^T once the summation index is
//     ordered as the accumulator orders it (the k index of an MFMA is a dummy
//     index, so any order works if A and B agree).  P never goes through LDS;
//   * the A operand of the second product is V^T: four consecutive keys for one
//     output column d per 64-bit piece.  V sits in LDS as [key][d] (as it is in
//     HBM) and is fetched with the LDS transpose read ds_read_b64_tr_b16.
//
// Softmax (log2 domain, c = scale*log2(e)):  p = exp2(s*c - m*c).  The reference
// maximum m of a row is only refreshed when a block's maximum exceeds it by more
// than a threshold (2^8 in p); rescaling the accumulator is then rare, and the
// result is unchanged because numerator and denominator share the reference.
//
// Kernels:
//   fa_fwd_global_kernel  global layers (no window).  64-key tiles run in a software pipeline over
//       32-key x 32-query units: while the vector ALU turns a unit's scores into probabilities, the
//       matrix cores compute the next unit's scores and accumulate the P.V of the tile before.  The
//       last tile is masked.
//   fa_fwd_window_resident_kernel  local layers whose key range per query tile fits in
//       LDS (the paper's 63/64 window): everything is requested at once, then each
//       wavefront runs the same pipeline over the blocks its queries can see.
//   fa_fwd_small_kernel  the smallest calls, local and global: 32 query rows per workgroup, whose wavefronts hold all key blocks.
//   fa_fwd_window_kernel  wider or one-sided windows: ring of 32-key stages.
//   fa_fwd_split_kernel  global layers with so few query tiles that the kernels above would leave
//       SIMDs with one wavefront or none (a single request, a few short sequences): NQ query
//       blocks per workgroup, each shared by NK wavefronts that split the KEYS and merge their
//       partial results through LDS.
//   fa_fwd_window_twophase_kernel  local layers with a narrow two-sided window: K, then V, through one
//       LDS region; also with a key bias or a rotation.
//   fa_fwd_masked_kernel  general path (register staging, padded tiles, optional 16-bit V
//       reads) for head_dim 32, 64, 128: the production path of wide or one-sided windows of
//       head_dim 32 / 128 and of a key bias outside the pipelined cases; at head_dim 64 also an
//       independent implementation for the tests.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "fa.h"
#include "fa_args.h"
#include "fa_mix_map.h"

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2v __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef short shortx8 __attribute__((ext_vector_type(8)));

constexpr int kD = 64;        // head_dim of the pipelined kernels (the masked kernel takes 32, 64, 128)
constexpr int kBN = 64;       // keys per LDS tile
constexpr int kWaves = 4;
constexpr int kThreads = kWaves * 64;
// Row strides of the PADDED LDS tiles in 16-bit elements, for head_dim D.  K is read with
// 16-byte accesses by 32 rows at once (a row stride of D/2 + 4 dwords puts 16 consecutive
// rows on 16 different 16-byte bank groups for D = 32, 64, 128); V is read by the
// transpose load, 4 rows x 32 bytes per 16 lanes.
constexpr int stride_k(int D) { return D + 8; }
constexpr int stride_v(int D) { return D + 16; }
constexpr float kLn2 = 0.693147180559945309f;
// A lane's 16 probabilities of one block may sum to at most this (against the row's
// current reference) before the reference is refreshed.  2^14 keeps every single p
// inside fp16 range (max 65504) with room to spare and makes refreshes very rare.
constexpr float kPLimit = 16384.f;

struct F16 {
  typedef half8 v8;
  static constexpr bool kSumRounded = true;
  static constexpr bool kWideRange = false;   // its values times any factor below 2^112 are finite fp32 numbers
  static __device__ __forceinline__ floatx16 mfma(v8 a, v8 b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ floatx4 mfma16(v8 a, v8 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ uint32_t pack2(float a, float b) {  // round to nearest even
    half2v h = __builtin_convertvector((floatx2){a, b}, half2v);
    return __builtin_bit_cast(uint32_t, h);
  }
  // acc + lo + hi of a packed pair, accumulated in fp32
  static __device__ __forceinline__ float sum2(uint32_t pk, float acc) {
    return __builtin_amdgcn_fdot2(__builtin_bit_cast(half2v, pk), (half2v){1, 1}, acc, false);
  }
  // lo + hi of a packed pair: the three-operand form with a constant zero addend, so that a
  // chain of sums needs no register zeroed first (the compiler, given the builtin with a zero
  // accumulator, moves 0 into a register and uses the accumulating two-operand form)
  static __device__ __forceinline__ float sum2_first(uint32_t pk) {
    float d;
    asm("v_dot2_f32_f16 %0, %1, %2, 0" : "=v"(d) : "v"(pk), "s"(0x3c003c00u));
    return d;
  }
  static __device__ __forceinline__ float to_float(uint16_t x) { return (float)__builtin_bit_cast(_Float16, x); }
};

struct BF16 {
  typedef bf8 v8;
  static constexpr bool kSumRounded = false;
  static constexpr bool kWideRange = true;
  static __device__ __forceinline__ floatx16 mfma(v8 a, v8 b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ floatx4 mfma16(v8 a, v8 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ uint32_t pack2(float a, float b) {
    bf2v h = __builtin_convertvector((floatx2){a, b}, bf2v);
    return __builtin_bit_cast(uint32_t, h);
  }
  static __device__ __forceinline__ float sum2(uint32_t pk, float acc) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf2v, pk),
                                           (bf2v){(__bf16)1.0f, (__bf16)1.0f}, acc, false);
  }
  static __device__ __forceinline__ float sum2_first(uint32_t pk) { return sum2(pk, 0.f); }  // unused: bf16 sums fp32 values
  static __device__ __forceinline__ float to_float(uint16_t x) { return __builtin_bit_cast(float, (uint32_t)x << 16); }
};

// Exchange between the two lanes (l, l ^ 32) that hold the same query: afterwards
// a = x of the lower lane of the pair and b = x of the upper one, in both lanes.
// v_permlane32_swap exchanges lanes 32..63 of its first register with lanes 0..31 of
// its second.  Written as asm because the compiler folds the builtin's two results
// into one when both inputs are the same value; the s_nop covers the VALU-write ->
// permlane-read hazard the compiler cannot see inside an asm block.  Both registers come into
// the block with a value: one that it merely wrote could still be the destination of a matrix
// product under way, whose late write the compiler only guards against where it sees the other.
__device__ __forceinline__ void swap_halves(float x, float& a, float& b) {
  a = b = x;
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ float max_xor32(float x) {
  float a, b;
  swap_halves(x, a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float sum_xor32(float x) {
  float a, b;
  swap_halves(x, a, b);
  return a + b;
}

// 16 bytes per lane from global memory straight into LDS: lane L's data lands at
// lds_dst + 16*L (lds_dst wavefront-uniform), the global address is gbase (uniform, scalar
// registers) + a per-lane byte offset.  Written as asm: the compiler would make every
// later LDS read wait for such a load (it cannot tell that the stage being filled and the
// stage being read are disjoint), which would serialise the prefetch.  The caller waits
// with wait_direct_loads() before the barrier that publishes the stage.  M0 holds the LDS
// address: M0 is a reserved register for inline asm (the compiler rejects it on a clobber list
// with a warning that such a clobber "may lead to undefined behaviour") and is rewritten by the
// compiler before every use of its own, so nothing of its contents is assumed after the asm.
__device__ __forceinline__ void load16_to_lds(const void* gbase, uint32_t lane_off_bytes, void* lds_dst) {
  typedef __attribute__((address_space(3))) void lds_void;
  const uint32_t l = (uint32_t)(size_t)(lds_void*)lds_dst;
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(l), "v"(lane_off_bytes), "s"(gbase)
               : "memory");
}
// The lane index, formed where it is needed: values derived from it outside the main loop then need no register through it.
// (Only the scalar mask comes out of an asm block: a vector register written in one may still be the destination of a matrix
// product under way, which the compiler waits for where it sees the write.)
__device__ __forceinline__ int lane_now() {
  uint32_t ones;
  asm volatile("s_mov_b32 %0, -1" : "=s"(ones));
  return (int)__builtin_amdgcn_mbcnt_hi(ones, __builtin_amdgcn_mbcnt_lo(ones, 0));
}

// s_waitcnt immediate that waits for vmcnt <= N only (expcnt and lgkmcnt fields at their
// maxima): vmcnt is bits 3:0 plus bits 15:14 of the immediate.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit field");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}
__device__ __forceinline__ void wait_direct_loads() { wait_vmcnt<0>(); }

template <class T>
__device__ __forceinline__ typename T::v8 as_v8(uint4 u) {
  return __builtin_bit_cast(typename T::v8, u);
}

// A operand of S^T = K Q^T for one k-step: K[row l%32][16*ks + 8*(l/32) .. +7]
template <class T, int D = kD>
__device__ __forceinline__ typename T::v8 load_k_frag(const uint16_t* kblk, int l32, int hh, int ks) {
  return as_v8<T>(*(const uint4*)&kblk[l32 * stride_k(D) + ks * 16 + hh * 8]);
}

// A operand of O^T = V^T P^T: column d = 32*db + l%32 of V, summation slots
// (hh, e) = keys 16*ks2 + (e < 4 ? 4*hh + e : 8 + 4*hh + e - 4) of the 32-key block.
// Within 16 lanes, lane p fetches 4 consecutive d of key row p/4; the transpose
// read hands lane i the 4 keys of column i.
template <class T, int D = kD>
__device__ __forceinline__ typename T::v8 load_vt_frag(const uint16_t* vblk, int lane, int ks2, int db) {
  constexpr int SV = stride_v(D);
  const int hh = lane >> 5, p16 = lane & 15;
  const int row = ks2 * 16 + 4 * hh + (p16 >> 2);
  const int col = db * 32 + 16 * ((lane >> 4) & 1) + 4 * (p16 & 3);
  typedef __attribute__((address_space(3))) shortx4 lds_s4;
  const shortx4 x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)&vblk[row * SV + col]);
  const shortx4 x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)&vblk[(row + 8) * SV + col]);
  shortx8 x;
  x[0] = x0[0]; x[1] = x0[1]; x[2] = x0[2]; x[3] = x0[3];
  x[4] = x1[0]; x[5] = x1[1]; x[6] = x1[2]; x[7] = x1[3];
  return __builtin_bit_cast(typename T::v8, x);
}

// Same operand through plain 16-bit LDS reads (slow; kept as an independent path).
template <class T, int D = kD>
__device__ __forceinline__ typename T::v8 load_vt_frag_scalar(const uint16_t* vblk, int lane, int ks2, int db) {
  const int hh = lane >> 5, l32 = lane & 31;
  shortx8 x;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int row = ks2 * 16 + (e < 4 ? 4 * hh + e : 8 + 4 * hh + e - 4);
    x[e] = (short)vblk[row * stride_v(D) + db * 32 + l32];
  }
  return __builtin_bit_cast(typename T::v8, x);
}

// The same two operands from an UNPADDED, swizzled tile (64 halves = 128 bytes per row),
// the layout that direct global->LDS loads produce: 16-byte chunk position c' of row r
// holds logical chunk c' ^ k_swz(r) for K and c' ^ v_swz(r) for V.  LDS has 64 four-byte
// banks, so two consecutive rows cover all banks once and the row's parity already picks
// the half; the swizzles spread what remains.
//   K: the 16-byte operand read of a k-step touches rows 0..15 at one chunk (lanes 0..15)
//      and the neighbouring chunk of the same rows (lanes 32..47): rows of equal parity
//      must land on 8 different chunk positions, whichever 16 lanes are served together.
//   V: a transpose read touches 4 rows x 4 chunks (or 8 rows x 2 chunks) per 32 lanes.
// Measured on gfx950: 246 B/clk per CU for the K reads and 199 B/clk for the V reads,
// the same as conflict-free linear addresses.  kblk / vblk must start at a row that is a
// multiple of 16.
__device__ __forceinline__ int k_swz(int r) { return 2 * ((r >> 1) & 3) + ((r >> 3) & 1); }
__device__ __forceinline__ int v_swz(int r) { return 4 * ((r >> 1) & 1) + 2 * ((r >> 2) & 1); }
// head_dim 128: a 256-byte row covers all 64 banks by itself and has 16 chunk positions.
//   K: rows 0..15 at one chunk need 16 different positions, rows 0..7 at a chunk pair too.
//   V: 4 rows x 4 chunks, or 8 rows x 2 chunks, per 32 lanes.
__device__ __forceinline__ int k_swz128(int r) { return 2 * (r & 7) + ((r >> 3) & 1); }
__device__ __forceinline__ int v_swz128(int r) { return 4 * (r & 3) + 2 * ((r >> 2) & 1); }
// head_dim 32: a 64-byte row has 4 chunk positions and four rows cover the banks once.
//   K: rows r, r+4, r+8, r+12 share their banks, so at one chunk they need four different
//      positions, and rows r, r+4 at a chunk pair (2 ks, 2 ks + 1) two disjoint pairs.
//   V: 4 rows x 4 chunks per 32 lanes is 256 contiguous bytes: no swizzle needed.
__device__ __forceinline__ int k_swz32(int r) { return 2 * ((r >> 2) & 1) + ((r >> 3) & 1); }
template <int D>
__device__ __forceinline__ int k_swz_d(int r) { return D == 128 ? k_swz128(r) : (D == 32 ? k_swz32(r) : k_swz(r)); }
template <int D>
__device__ __forceinline__ int v_swz_d(int r) { return D == 128 ? v_swz128(r) : (D == 32 ? 0 : v_swz(r)); }
// Operand fragments out of a swizzled 32-row block of any head_dim (row = D elements).
template <class T, int D>
__device__ __forceinline__ typename T::v8 load_k_frag_swz_d(const uint16_t* kblk, int l32, int hh, int ks) {
  return as_v8<T>(*(const uint4*)&kblk[l32 * D + (((2 * ks + hh) ^ k_swz_d<D>(l32)) * 8)]);
}
template <class T, int D>
__device__ __forceinline__ typename T::v8 load_vt_frag_swz_d(const uint16_t* vblk, int lane, int ks2, int db) {
  const int hh = lane >> 5, p16 = lane & 15, g = (lane >> 4) & 1;
  const int row = ks2 * 16 + 4 * hh + (p16 >> 2);  // (rows row and row + 8 have the same swizzle)
  const int off = (((4 * db + 2 * g + ((p16 & 3) >> 1)) ^ v_swz_d<D>(row)) * 8) + (p16 & 1) * 4;
  typedef __attribute__((address_space(3))) shortx4 lds_s4;
  const shortx4 x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)&vblk[row * D + off]);
  const shortx4 x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)&vblk[(row + 8) * D + off]);
  shortx8 x;
  x[0] = x0[0]; x[1] = x0[1]; x[2] = x0[2]; x[3] = x0[3];
  x[4] = x1[0]; x[5] = x1[1]; x[6] = x1[2]; x[7] = x1[3];
  return __builtin_bit_cast(typename T::v8, x);
}

// Swizzles of the 16-row operand reads (see k_swz for the tile).  LDS serves a 16-byte read 16 lanes at a time, and not
// consecutive ones: lanes 0-3, 12-15, 20-23, 24-27 first.  Those are rows 0-3 and 12-15 at one chunk and 4-11 at its
// neighbour, so rows 4-11 take the half of the positions that is closed under the step to the neighbour and the others the
// other half (rows that share their banks: all of one parity, all, or every fourth).  With k_swz every such read took two
// turns: a third of the LDS cycles of a 32K call.
template <int D>
__device__ __forceinline__ int k_swz16(int r) {
  const int mid = ((r >> 2) ^ (r >> 3)) & 1, hi = (r >> 3) & 1;
  return D == 128 ? 8 * mid + 4 * hi + (r & 3) : (D == 32 ? 2 * mid + hi : 4 * mid + 2 * hi + ((r >> 1) & 1));
}
// V: a transpose read serves 32 lanes at a time, two groups of 4 rows x 32 bytes, whichever two.
template <int D>
__device__ __forceinline__ int v_swz16(int r) {
  const int mid = ((r >> 2) ^ (r >> 3)) & 1;
  return D == 128 ? 4 * (r & 3) + 2 * mid : (D == 32 ? 2 * mid : 4 * ((r >> 1) & 1) + 2 * mid);
}

// one transposed operand: two reads of 16 lanes x 4 rows each
template <class V8>
__device__ __forceinline__ V8 tr_pair(const uint16_t* at0, const uint16_t* at1) {
  typedef __attribute__((address_space(3))) shortx4 lds_s4;
  const shortx4 x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)at0);
  const shortx4 x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)at1);
  shortx8 x;
  x[0] = x0[0]; x[1] = x0[1]; x[2] = x0[2]; x[3] = x0[3];
  x[4] = x1[0]; x[5] = x1[1]; x[6] = x1[2]; x[7] = x1[3];
  return __builtin_bit_cast(V8, x);
}

template <class T>
__device__ __forceinline__ typename T::v8 load_k_frag_swz(const uint16_t* kblk, int l32, int hh, int ks) {
  return as_v8<T>(*(const uint4*)&kblk[l32 * kD + (((2 * ks + hh) ^ k_swz(l32)) * 8)]);
}
template <class T>
__device__ __forceinline__ typename T::v8 load_vt_frag_swz(const uint16_t* vblk, int lane, int ks2, int db) {
  const int hh = lane >> 5, p16 = lane & 15, g = (lane >> 4) & 1;
  const int row = ks2 * 16 + 4 * hh + (p16 >> 2);
  const int off = (((4 * db + 2 * g + ((p16 & 3) >> 1)) ^ v_swz(row)) * 8) + (p16 & 1) * 4;
  typedef __attribute__((address_space(3))) shortx4 lds_s4;
  const shortx4 x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)&vblk[row * kD + off]);
  const shortx4 x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)&vblk[(row + 8) * kD + off]);
  shortx8 x;
  x[0] = x0[0]; x[1] = x0[1]; x[2] = x0[2]; x[3] = x0[3];
  x[4] = x1[0]; x[5] = x1[1]; x[6] = x1[2]; x[7] = x1[3];
  return __builtin_bit_cast(typename T::v8, x);
}

template <int NQB, int D = kD>
struct RowState {
  floatx16 oacc[NQB][D / 32];  // O^T: [qb][d block], rows d = 32*db + 8*(r/4) + 4*hh + r%4
  float m_ref[NQB];       // reference maximum (raw score units), -inf before the first key
  float mc[NQB];          // m_ref * c, 0 while m_ref = -inf
  float lsum[NQB];        // this lane's share of the row sum
};

// Refresh the reference of rows whose block maximum ran away from it.  Each lane
// decides on its own row's evidence only, so a row's arithmetic never depends on
// which other rows share its wavefront.
template <int NQB, int D>
__device__ __forceinline__ void rescale_rows(RowState<NQB, D>& st, int qb, bool refresh, float tmax, float c) {
  const float m_new = refresh ? tmax : st.m_ref[qb];
  const float mc_new = (m_new == -INFINITY) ? 0.f : m_new * c;
  // nothing has been accumulated while the old reference is -inf: keep 0 * alpha out of
  // reach of an infinite alpha
  const float alpha = (st.m_ref[qb] == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(st.mc[qb] - mc_new);
  st.m_ref[qb] = m_new;
  st.mc[qb] = mc_new;
  st.lsum[qb] *= alpha;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) st.oacc[qb][db][r] *= alpha;
}

// Selection by bit r of a visibility word without a compare: the bit, sign-extended, is an
// all-ones or all-zeros word (one v_bfe_i32), and one more bitwise instruction keeps the value or
// replaces it (a test, a compare and a select would be three).
__device__ __forceinline__ uint32_t bit_to_word(uint32_t vis, int r) { return (uint32_t)__builtin_amdgcn_sbfe((int)vis, r, 1); }
__device__ __forceinline__ float keep_or_zero(float x, uint32_t vis, int r) {
  return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, x) & bit_to_word(vis, r));
}
__device__ __forceinline__ float keep_or_neg_inf(float x, uint32_t vis, int r) {
  const uint32_t m = bit_to_word(vis, r);
  return __builtin_bit_cast(float, (__builtin_bit_cast(uint32_t, x) & m) | (0xFF800000u & ~m));
}

// Probabilities of one 32 x 32 block against the row's current reference, rounded and
// packed as the B operand of the P.V product, plus the lane's share of their row sum.
// fp16: the sum is taken over the ROUNDED probabilities (the numbers the matrix product
// uses), two per v_dot2c instruction.  bf16: the unrounded fp32 values are summed; with
// 8 mantissa bits the rounded sum would cost lse up to ~2e-3 when a row sees only a
// handful of keys.  vis: bit r set = accumulator element r is a visible key.
// SUM32: the unrounded values are summed in fp16 as well.
template <class T, bool MASKED, bool SUM32 = false>
__device__ __forceinline__ void prob_block(const floatx16& sv, float c, float mcq, uint32_t vis,
                                           uint32_t (&pk)[8], float& blk) {
  const float nmc = -mcq;
  float l0 = 0.f, l1 = 0.f;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[2 * r], c, nmc));
    float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[2 * r + 1], c, nmc));
    if (MASKED) {
      e0 = keep_or_zero(e0, vis, 2 * r);
      e1 = keep_or_zero(e1, vis, 2 * r + 1);
    }
    pk[r] = T::pack2(e0, e1);
    if (SUM32 || !T::kSumRounded) {
      l0 += e0;
      l1 += e1;
    }
  }
  if (!SUM32 && T::kSumRounded) {
    l0 = T::sum2_first(pk[0]);
    l1 = T::sum2_first(pk[1]);
#pragma unroll
    for (int r = 2; r < 8; r += 2) {
      l0 = T::sum2(pk[r], l0);
      l1 = T::sum2(pk[r + 1], l1);
    }
  }
  blk = l0 + l1;
}

// Visibility bits of a lane's 16 accumulator elements for the block starting at key kb0:
// bit r is set iff jlo <= kb0 + 8*(r/4) + 4*hh + r%4 <= jhi.  Built from one 32-bit range
// mask (bit k = key kb0 + 4*hh + k visible) whose nibbles 0, 2, 4, 6 are the lane's keys.
__device__ __forceinline__ uint32_t visible_bits(int kb0, int hh, int jlo, int jhi) {
  int lo = jlo - kb0 - 4 * hh, hi = jhi - kb0 - 4 * hh;
  lo = lo < 0 ? 0 : lo;
  hi = hi > 31 ? 31 : hi;
  const bool none = hi < lo;                          // also covers hi < 0 and lo > 31
  const int lo_s = lo > 31 ? 31 : lo, hi_s = hi < 0 ? 0 : hi;  // shift counts stay in 0..31
  const uint32_t m = none ? 0u : ((0xFFFFFFFFu >> (31 - hi_s)) & (0xFFFFFFFFu << lo_s));
  return (m & 0xFu) | ((m >> 4) & 0xF0u) | ((m >> 8) & 0xF00u) | ((m >> 12) & 0xF000u);
}

// One 32-key block, scores to accumulator, with per-element masking if MASKED.
// kblk / vblk: LDS rows of the block; kb0: its first key index; [jlo, jhi] per lane
// is the visible key range of the lane's query.  FRAG selects how operands come out of
// LDS: 0 padded tile + transpose read, 1 padded tile + 16-bit reads, 2 swizzled tile +
// transpose read.
//
// bias2 (optional): 32 floats in LDS, the block's additive key bias times log2(e).  With a
// bias the row state is kept in the log2 domain (m_ref = mc = reference of s*c + bias2).
template <class T, int NQB, bool MASKED, int FRAG, int D>
__device__ __forceinline__ void simple_block(RowState<NQB, D>& st, const typename T::v8 (&qreg)[NQB][D / 16],
                                             const uint16_t* kblk, const uint16_t* vblk, int kb0,
                                             const int (&jlo)[NQB], const int (&jhi)[NQB], int lane,
                                             float c, float tau_raw, const float* bias2 = nullptr) {
  const int l32 = lane & 31, hh = lane >> 5;
  floatx16 sacc[NQB];
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
    for (int r = 0; r < 16; ++r) sacc[qb][r] = 0.f;
  static_assert(FRAG != 2 || D == kD, "swizzled tiles exist for head_dim 64 only");
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) {
    const typename T::v8 ka = FRAG == 2 ? load_k_frag_swz<T>(kblk, l32, hh, ks) : load_k_frag<T, D>(kblk, l32, hh, ks);
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) sacc[qb] = T::mfma(ka, qreg[qb][ks], sacc[qb]);
  }
  uint32_t pk[NQB][8];
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    const uint32_t vis = MASKED ? visible_bits(kb0, hh, jlo[qb], jhi[qb]) : 0xFFFFu;
    float p[16];
    float ls;  // read after a possible rescale of the row state
    if (bias2) {
      // scores in the log2 domain, bias included; the reference lives in the same domain
      float t[16];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 b4 = *(const float4*)&bias2[8 * g + 4 * hh];
        t[4 * g + 0] = __builtin_fmaf(sacc[qb][4 * g + 0], c, b4.x);
        t[4 * g + 1] = __builtin_fmaf(sacc[qb][4 * g + 1], c, b4.y);
        t[4 * g + 2] = __builtin_fmaf(sacc[qb][4 * g + 2], c, b4.z);
        t[4 * g + 3] = __builtin_fmaf(sacc[qb][4 * g + 3], c, b4.w);
      }
      float tmax = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (MASKED) t[r] = keep_or_neg_inf(t[r], vis, r);
        tmax = fmaxf(tmax, t[r]);
      }
      tmax = max_xor32(tmax);
      const bool refresh = (tmax - st.m_ref[qb]) > 8.0f;
      if (__any(refresh)) rescale_rows(st, qb, refresh, tmax, 1.0f);
      const float mcq = st.mc[qb];
      ls = st.lsum[qb];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float e = __builtin_amdgcn_exp2f(t[r] - mcq);
        if (MASKED) e = keep_or_zero(e, vis, r);
        p[r] = e;
        ls += e;
      }
    } else {
      float tmax = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float sv = MASKED ? keep_or_neg_inf(sacc[qb][r], vis, r) : sacc[qb][r];
        tmax = fmaxf(tmax, sv);
      }
      tmax = max_xor32(tmax);
      const bool refresh = (tmax - st.m_ref[qb]) > tau_raw;
      if (__any(refresh)) rescale_rows(st, qb, refresh, tmax, c);
      const float nmc = -st.mc[qb];
      ls = st.lsum[qb];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float e = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[qb][r], c, nmc));
        if (MASKED) e = keep_or_zero(e, vis, r);
        p[r] = e;
        ls += e;
      }
    }
    st.lsum[qb] = ls;
#pragma unroll
    for (int r = 0; r < 8; ++r) pk[qb][r] = T::pack2(p[2 * r], p[2 * r + 1]);
  }
#pragma unroll
  for (int ks2 = 0; ks2 < 2; ++ks2) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db) {
      const typename T::v8 va = FRAG == 2   ? load_vt_frag_swz<T>(vblk, lane, ks2, db)
                                : FRAG == 0 ? load_vt_frag<T, D>(vblk, lane, ks2, db)
                                            : load_vt_frag_scalar<T, D>(vblk, lane, ks2, db);
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) {
        const uint4 pu = make_uint4(pk[qb][ks2 * 4 + 0], pk[qb][ks2 * 4 + 1], pk[qb][ks2 * 4 + 2],
                                    pk[qb][ks2 * 4 + 3]);
        st.oacc[qb][db] = T::mfma(va, as_v8<T>(pu), st.oacc[qb][db]);
      }
    }
  }
}

// A key's bias in raw-score units.  The host sends no call here whose |scale| is too small for this (inv_abs_scale = 0 then).
// bfloat16 holds biases whose product with log2(e) is no finite fp32 number: infinite ones then (a key excluded, as in the
// masked kernel).  A reference of such a bias that is finite while its product with c = |scale| log2(e) is not would turn
// rows into NaN, so where |scale| > ln 2 the factor log2(e) comes first (bias_pre; 1 elsewhere, where the largest fp32
// number times c is finite).  SATURATE: below |scale| = ln 2 a quotient past the largest fp32 number stops there instead of
// excluding the key, as the masked kernel has it: for the head sizes whose biased calls would otherwise run that kernel (it
// takes wavefront 0 of the pipelined kernel 1-3 % of a short call).
template <class T, bool SATURATE>
__device__ __forceinline__ float bias_over_scale(const FaKernelArgs& a, uint16_t bits) {
  const float b = T::to_float(bits);
  if (!T::kWideRange) return b * a.inv_abs_scale;
  const float x = b * a.bias_pre * a.inv_abs_scale;
  if (!SATURATE) return x;
  return __builtin_fabsf(b) <= 2.356e38f ? fminf(fmaxf(x, -3.4028234e38f), 3.4028234e38f) : b * INFINITY;
}

// bias of a 32-key block (32 floats in LDS, raw-score units) added to its scores
__device__ __forceinline__ void add_bias(floatx16& s, const float* bblk, int hh) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const float4 b4 = *(const float4*)&bblk[8 * g + 4 * hh];
    s[4 * g + 0] += b4.x; s[4 * g + 1] += b4.y; s[4 * g + 2] += b4.z; s[4 * g + 3] += b4.w;
  }
}

// One word of every 64 bytes of the argument block, all under way at once: left to itself the compiler loads arguments where
// they are first used, three or four round trips to memory one after the other before a workgroup's first load.  For the kernels
// that one workgroup's latency bounds, us: small kernel, local 487 tokens 4.7 -> 4.4, global 512 5.5 -> 5.4, resident window kernel, 2K
// 7.8 -> 7.4; the split kernel, whose first loads need few of them, 7.0 -> 7.2 (3 x 302), calls of several rounds 0.5 - 1 % slower.
__device__ __forceinline__ void fetch_args() {
  typedef const __attribute__((address_space(4))) uint32_t Word;
  Word* const p = (Word*)__builtin_amdgcn_kernarg_segment_ptr();
  const uint32_t w0 = p[0], w1 = p[16], w2 = p[32], w3 = p[48], w4 = p[64];
  static_assert(sizeof(FaKernelArgs) > 256 && sizeof(FaKernelArgs) <= 320, "five pieces of 64 bytes");
  asm volatile("" : : "s"(w0), "s"(w1), "s"(w2), "s"(w3), "s"(w4));
}

// ---- pieces shared by both kernels ----------------------------------------------------
struct TileCoord {
  int b, h, qt, n, q0;
};

// CLAMP = false leaves tc.n as loaded (the caller clamps it into [0, max_len] when it first
// needs it, so that the wait for the load can come after other work).
// LONGEST_FIRST: the kernel also knows the order of sequences by falling length (a.longest_first).
// HEADS_FIRST: the kernel also knows the heads-first order (a.heads_first); the others keep the query tiles of one head in
// a row, which is an order of the same tiles.
template <int BM, bool CLAMP = true, bool HEADS_FIRST = false, bool LONGEST_FIRST = false>
__device__ __forceinline__ bool locate_tile(const FaKernelArgs& a, TileCoord& tc) {
  if (a.map_xcd) {
    // Workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2.  Tiles of
    // one (batch, head) read the same K/V, so every XCD takes one contiguous eighth of each
    // batch element's (head, query tile) range: K/V re-reads stay in that XCD's L2, and
    // the eighths are equal work whatever the sequence lengths are.
    const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int per = a.xcd_per;                // ceil(heads * n_qtiles / 8)
    tc.b = j / per;
    const int t = x * per + (j - tc.b * per);
    const bool heads_first = HEADS_FIRST && a.heads_first;
    if (tc.b >= a.batch || (!heads_first && t >= a.heads * a.n_qtiles)) return false;
    if (LONGEST_FIRST && a.longest_first) {
      // tc.b is a rank so far: lane l holds sequence l's length; the sequences are taken by eighths of max_len, those of one
      // eighth as they come
      const int lane = threadIdx.x & 63;
      const int len = lane < a.batch ? a.seq_lens[lane] : INT32_MIN;
      uint64_t longer = 0, in = 0;       // sequences above the eighth, sequences of it
#pragma unroll
      for (int e = 7; e >= 0; --e) {
        const uint64_t down = e > 0 ? __ballot(len > (a.max_len >> 3) * e) : __ballot(lane < a.batch);
        if (in == 0 && tc.b < __popcll(down)) in = down & ~longer;
        if (in == 0) longer = down;
      }
      const int at = __builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in, 0));
      const uint64_t mine = __ballot(((in >> lane) & 1) && at == tc.b - __popcll(longer));
      tc.b = __ffsll((unsigned long long)mine) - 1;
    }
    if (heads_first) {
      // all heads of a query tile in a row: the angle tables, or the lines that narrow heads share, are read once per XCD
      int n = a.max_len;
      if (a.seq_lens) {
        n = a.seq_lens[tc.b];
        n = n < 0 ? 0 : (n > a.max_len ? a.max_len : n);
      }
      const int u = fa_heads_first_tile(x, j - tc.b * per, per, (n + BM - 1) / BM * a.heads, a.heads * a.n_qtiles);
      if (u < 0) return false;
      tc.qt = u / a.heads;
      tc.h = u - tc.qt * a.heads;
    } else {
      tc.h = t / a.n_qtiles;
      tc.qt = t - tc.h * a.n_qtiles;
    }
  } else {
    const int tile = blockIdx.x;
    if (tile >= a.total_tiles) return false;
    tc.qt = tile % a.n_qtiles;
    const int bh = tile / a.n_qtiles;
    tc.h = bh % a.heads;
    tc.b = bh / a.heads;
  }
  int n = a.max_len;
  if (a.seq_lens) {
    n = a.seq_lens[tc.b];
    if (CLAMP) n = n < 0 ? 0 : (n > a.max_len ? a.max_len : n);
  }
  tc.n = n;
  tc.q0 = tc.qt * BM;
  return true;
}

// Workgroup entirely in the padding: o = 0, lse = -inf.
template <int BM, int D = kD, int THREADS = kThreads>
__device__ __forceinline__ void zero_fill(const FaKernelArgs& a, const TileCoord& tc, uint16_t* op, float* lsep) {
  const int tid = threadIdx.x, N = a.max_len;
  constexpr int CH = D / 8;  // 16-byte chunks per row
  const int r = tid / CH, c16 = tid % CH;
  for (int row = tc.q0 + r; row < tc.q0 + BM && row < N; row += THREADS / CH)
    *(uint4*)(op + row * a.os[2] + c16 * 8) = make_uint4(0, 0, 0, 0);
  if (lsep)
    for (int row = tc.q0 + tid; row < tc.q0 + BM && row < N; row += THREADS) lsep[row] = -INFINITY;
}

// ---- rotary position embedding (optional) ----------------------------------------------
// Eight pairs (lo[e], hi[e]) = elements (f + e, f + e + head_dim/2) of one row are rotated by
// the row's angles: lo' = lo cos - hi sin, hi' = hi cos + lo sin, in fp32, and rounded to the
// storage type (nearest even).  cs / sn point at the row's table entries f .. f + 7.
template <class T>
__device__ __forceinline__ void rotate8(uint4& lo, uint4& hi, const float* cs, const float* sn) {
  const float4 c0 = *(const float4*)cs, c1 = *(const float4*)(cs + 4);
  const float4 s0 = *(const float4*)sn, s1 = *(const float4*)(sn + 4);
  const float cc[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
  const float ss[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
  const uint32_t lw[4] = {lo.x, lo.y, lo.z, lo.w}, hw[4] = {hi.x, hi.y, hi.z, hi.w};
  uint32_t lo_out[4], hi_out[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    float l[2], h[2], lr[2], hr[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      l[x] = T::to_float((uint16_t)(lw[w] >> (16 * x)));
      h[x] = T::to_float((uint16_t)(hw[w] >> (16 * x)));
      lr[x] = __builtin_fmaf(l[x], cc[2 * w + x], -(h[x] * ss[2 * w + x]));
      hr[x] = __builtin_fmaf(h[x], cc[2 * w + x], l[x] * ss[2 * w + x]);
    }
    lo_out[w] = T::pack2(lr[0], lr[1]);
    hi_out[w] = T::pack2(hr[0], hr[1]);
  }
  lo = make_uint4(lo_out[0], lo_out[1], lo_out[2], lo_out[3]);
  hi = make_uint4(hi_out[0], hi_out[1], hi_out[2], hi_out[3]);
}

// Rotates `rows` rows of K in place in a padded LDS tile (all threads of the workgroup take part; the
// caller puts barriers around the call).  Tile row r is key key0 + r (clamped into the tensor: rows
// outside it are never used unmasked).
template <class T, int D>
__device__ __forceinline__ void rope_rows_in_lds(const FaKernelArgs& a, uint16_t* tile, int stride, int rows, int key0,
                                                 int tid, int nthreads) {
  constexpr int HALF = D / 16;  // 16-byte chunks per half row
  for (int u = tid; u < rows * HALF; u += nthreads) {
    const int r = u / HALF, c = u % HALF;
    const int key = key0 + r < a.max_len ? key0 + r : a.max_len - 1;
    uint4* plo = (uint4*)&tile[r * stride + c * 8];
    uint4* phi = (uint4*)&tile[r * stride + (c + HALF) * 8];
    uint4 lo = *plo, hi = *phi;
    rotate8<T>(lo, hi, a.rope_cos + (int64_t)key * a.rope_stride + 8 * c, a.rope_sin + (int64_t)key * a.rope_stride + 8 * c);
    *plo = lo;
    *phi = hi;
  }
}

// ROPE = false: the kernel is never launched with a rotation (no code for it).
template <class T, int NQB, int KS, bool ROPE = true>
__device__ __forceinline__ void load_q(const FaKernelArgs& a, const uint16_t* qp, int qw0, int lane,
                                       typename T::v8 (&qreg)[NQB][KS]) {
  const int l32 = lane & 31, hh = lane >> 5, N = a.max_len;
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    int row = qw0 + qb * 32 + l32;
    row = row < N ? row : N - 1;
    const uint16_t* src = qp + row * a.qs[2] + hh * 8;
    uint4 u[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) u[ks] = *(const uint4*)(src + ks * 16);
    if (ROPE && a.rope_cos) {
      // the lane holds columns 16 ks + 8 hh + e: chunk ks pairs with chunk ks + KS/2
#pragma unroll
      for (int ks = 0; ks < KS / 2; ++ks) {
        const int64_t t = (int64_t)row * a.rope_stride + 16 * ks + 8 * hh;
        rotate8<T>(u[ks], u[ks + KS / 2], a.rope_cos + t, a.rope_sin + t);
      }
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (a.negate_q) {
        u[ks].x ^= 0x80008000u; u[ks].y ^= 0x80008000u; u[ks].z ^= 0x80008000u; u[ks].w ^= 0x80008000u;
      }
      qreg[qb][ks] = as_v8<T>(u[ks]);
    }
  }
}

template <int NQB, int D>
__device__ __forceinline__ void init_state(RowState<NQB, D>& st) {
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    st.m_ref[qb] = -INFINITY;
    st.mc[qb] = 0.f;
    st.lsum[qb] = 0.f;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) st.oacc[qb][db][r] = 0.f;
  }
}

// Epilogue: o = O / l, cast, store; lse.  A lane holds one output ROW in pieces of four
// columns, so storing from registers would scatter 8-byte pieces over 32 rows per
// instruction.  Each wavefront instead transposes its 32 x 64 block through a private
// LDS patch (rows padded by 16 bytes) and stores whole rows, 16 bytes per lane.
// wave_patch: epi_patch(D) 16-bit elements of LDS owned by this wavefront; the caller has
// made sure (barrier) that nobody still reads tiles from that memory.
constexpr int epi_stride(int D) { return D + 8; }
constexpr int epi_patch(int D) { return 32 * epi_stride(D); }
constexpr int kEpiPatch = epi_patch(kD);

template <class T, int NQB, int D>
__device__ __forceinline__ void epilogue(const FaKernelArgs& a, RowState<NQB, D>& st, uint16_t* op, float* lsep,
                                         int qw0, int n, int lane, uint16_t* wave_patch) {
  constexpr int kEpiStride = epi_stride(D);
  constexpr int CH = D / 8;         // 16-byte chunks per output row
  constexpr int RPP = 64 / CH;      // rows stored per pass
  const int l32 = lane & 31, hh = lane >> 5, N = a.max_len;
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    const int ig = qw0 + qb * 32 + l32;
    const float ltot = sum_xor32(st.lsum[qb]);
    const bool live = (ig < n) && (ltot > 0.f);
    const float inv = live ? 1.0f / ltot : 0.f;
#pragma unroll
    for (int db = 0; db < D / 32; ++db) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        uint2 w;
        w.x = T::pack2(st.oacc[qb][db][4 * g + 0] * inv, st.oacc[qb][db][4 * g + 1] * inv);
        w.y = T::pack2(st.oacc[qb][db][4 * g + 2] * inv, st.oacc[qb][db][4 * g + 3] * inv);
        if (!live) w = make_uint2(0, 0);  // padded rows and rows with no visible key
        *(uint2*)&wave_patch[l32 * kEpiStride + db * 32 + 8 * g + 4 * hh] = w;
      }
    }
    // same wavefront writes and reads the patch: program order is enough
#pragma unroll
    for (int pass = 0; pass < 32 / RPP; ++pass) {
      const int r = pass * RPP + lane / CH;
      const uint4 v = *(const uint4*)&wave_patch[r * kEpiStride + (lane % CH) * 8];
      const int row = qw0 + qb * 32 + r;
      if (row < N) *(uint4*)(op + row * a.os[2] + (lane % CH) * 8) = v;
    }
    if (lsep && hh == 0 && ig < N)
      lsep[ig] = live ? (st.mc[qb] + __builtin_amdgcn_logf(ltot)) * kLn2 : -INFINITY;
  }
}

// One unit of the resident pipelines (head_dim 64, one query block per wavefront, K/V
// blocks as swizzled 32 x 64 tiles in LDS): probabilities of the current block from s_cur;
// meanwhile the matrix cores form the NEXT block's scores (s_nxt, from k_next, started from
// init(s_nxt): zero or a bias) and add the PREVIOUS block's P.V (p_prev, v_prev).
// kb0: first key of the current block; interior: every valid query of the wavefront sees all
// 32 keys, so no mask work; otherwise [jlo, jhi] is the lane's visible key range.
// alive: the lane's query row exists.
template <class T, class Init>
__device__ __forceinline__ void resident_unit(RowState<1>& st, const typename T::v8 (&qreg)[1][4], floatx16& s_cur,
                                              floatx16& s_nxt, typename T::v8 (&p_prev)[2],
                                              typename T::v8 (&p_cur)[2], const uint16_t* k_next,
                                              const uint16_t* v_prev, Init init, int kb0, bool interior, int jlo,
                                              int jhi, bool alive, float c, int lane) {
  const int l32 = lane & 31, hh = lane >> 5;
  typename T::v8 ka[4], va[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) ka[ks] = load_k_frag_swz<T>(k_next, l32, hh, ks);
#pragma unroll
  for (int i = 0; i < 4; ++i) va[i] = load_vt_frag_swz<T>(v_prev, lane, i >> 1, i & 1);
  init(s_nxt);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    s_nxt = T::mfma(ka[ks], qreg[0][ks], s_nxt);
    st.oacc[0][ks & 1] = T::mfma(va[ks], p_prev[ks >> 1], st.oacc[0][ks & 1]);
  }
  uint32_t pk[8];
  float blk;
  uint32_t vis = 0xFFFFu;
  if (!interior) vis = visible_bits(kb0, hh, jlo, jhi);
  // Rows that have not seen a key yet (the wavefront's first block, and the odd row whose
  // window starts a block later) adopt this block's maximum as their reference.  Nothing
  // has been accumulated for such a row, so there is nothing to rescale.
  if (__any(alive && st.m_ref[0] == -INFINITY)) {
    float t0 = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) t0 = fmaxf(t0, keep_or_neg_inf(s_cur[r], vis, r));
    const float tmax = max_xor32(t0);
    if (st.m_ref[0] == -INFINITY) {
      st.m_ref[0] = tmax;
      st.mc[0] = tmax == -INFINITY ? 0.f : tmax * c;
    }
  }
  if (interior) prob_block<T, false>(s_cur, c, st.mc[0], vis, pk, blk);
  else prob_block<T, true>(s_cur, c, st.mc[0], vis, pk, blk);
  // !(blk <= limit) also catches a NaN sum
  const bool trig = alive && !(blk <= kPLimit);
  if (__any(trig)) {
    // a row refreshes iff one of ITS two lanes tripped: no dependence on other rows
    const bool row_trig = sum_xor32(trig ? 1.f : 0.f) > 0.f;
    float t0 = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) t0 = fmaxf(t0, keep_or_neg_inf(s_cur[r], vis, r));
    const float tmax = max_xor32(t0);
    rescale_rows(st, 0, row_trig, tmax, c);
    prob_block<T, true>(s_cur, c, st.mc[0], vis, pk, blk);
  }
  st.lsum[0] += blk;
  p_cur[0] = as_v8<T>(make_uint4(pk[0], pk[1], pk[2], pk[3]));
  p_cur[1] = as_v8<T>(make_uint4(pk[4], pk[5], pk[6], pk[7]));
}

// ======================================================================================
// Masked kernel: windows (and any tile that needs per-element masks)
// ======================================================================================
template <class T, int D, int NQB, bool V_TR, bool BIAS = false>
// (two wavefronts per SIMD asked for where the compiler would otherwise settle for one)
__global__ __launch_bounds__(kThreads, ((D == 128 && !BIAS) || NQB == 2) ? 2 : 1) void fa_fwd_masked_kernel(const FaKernelArgs a) {
  constexpr int BM = kWaves * 32 * NQB;
  constexpr int SK = stride_k(D), SV = stride_v(D);
  static_assert(2 * kBN * SK >= kWaves * epi_patch(D), "the K stages double as the epilogue patches");
  __shared__ __attribute__((aligned(16))) uint16_t lds_k[2][kBN * SK];
  __shared__ __attribute__((aligned(16))) uint16_t lds_v[2][kBN * SV];
  __shared__ __attribute__((aligned(16))) float lds_b[2][BIAS ? kBN : 4];  // key bias * log2(e) of the tile

  TileCoord tc;
  if (!locate_tile<BM>(a, tc)) return;
  const int N = a.max_len, n = tc.n, q0 = tc.q0;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31;

  const uint16_t* qp = (const uint16_t*)a.q + tc.b * a.qs[0] + tc.h * a.qs[1];
  const uint16_t* kp = (const uint16_t*)a.k + tc.b * a.ks[0] + tc.h * a.ks[1];
  const uint16_t* vp = (const uint16_t*)a.v + tc.b * a.vs[0] + tc.h * a.vs[1];
  uint16_t* op = (uint16_t*)a.o + tc.b * a.os[0] + tc.h * a.os[1];
  float* lsep = a.lse ? a.lse + ((int64_t)tc.b * a.heads + tc.h) * N : nullptr;

  if (q0 >= n) {
    zero_fill<BM, D>(a, tc, op, lsep);
    return;
  }

  // key range of this workgroup
  const int q_last = (q0 + BM < n ? q0 + BM : n) - 1;
  int lo = 0, hi = n;
  if (a.wl >= 0) lo = q0 - a.wl > 0 ? q0 - a.wl : 0;
  if (a.wr >= 0) hi = q_last + a.wr + 1 < n ? q_last + a.wr + 1 : n;
  const int t_lo = lo / kBN;
  const int t_hi = (hi + kBN - 1) / kBN;

  // this wavefront's queries
  const int qw0 = q0 + wave * 32 * NQB;
  const int qw_last = (qw0 + 32 * NQB < n ? qw0 + 32 * NQB : n) - 1;  // < qw0: all padding
  const bool wave_has_rows = qw_last >= qw0;

  typename T::v8 qreg[NQB][D / 16];
  load_q<T, NQB>(a, qp, qw0, lane, qreg);
  RowState<NQB, D> st;
  init_state(st);
  int jlo[NQB], jhi[NQB];
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    const int ig = qw0 + qb * 32 + l32;
    jlo[qb] = 0;
    jhi[qb] = n - 1;
    if (a.wl >= 0 && ig - a.wl > jlo[qb]) jlo[qb] = ig - a.wl;
    if (a.wr >= 0 && ig + a.wr < jhi[qb]) jhi[qb] = ig + a.wr;
  }

  // staging: a 64-key tile is 64 rows of D/8 16-byte chunks; thread t moves chunk t % (D/8)
  // of rows t / (D/8) + i * RS, i = 0 .. NST-1 (named registers, not an array: an array
  // captured by the lambdas ends up in scratch memory)
  constexpr int CH = D / 8, RS = kThreads / CH, NST = kBN / RS;  // NST = 1, 2, 4 for D = 32, 64, 128
  const int st_r = tid / CH, st_c = (tid % CH) * 8;
  uint4 kst0, kst1, kst2, kst3, vst0, vst1, vst2, vst3;
  auto fetch_row = [&](int jg, uint4& kk, uint4& vv) {
    const int jc = jg < N ? jg : N - 1;
    kk = *(const uint4*)(kp + jc * a.ks[2] + st_c);
    vv = *(const uint4*)(vp + jc * a.vs[2] + st_c);
    // padded V rows are replaced by zeros: 0 * (whatever is stored there) must be 0
    if (jg >= n) vv = make_uint4(0, 0, 0, 0);
  };
  const uint16_t* bp = BIAS ? (const uint16_t*)a.key_bias + tc.b * a.kb_stride : nullptr;
  float bst = 0.f;  // threads 0..63: the bias of key t*64 + tid
  auto fetch = [&](int t) {
    fetch_row(t * kBN + st_r, kst0, vst0);
    if (NST > 1) fetch_row(t * kBN + RS + st_r, kst1, vst1);
    if (NST > 2) {
      fetch_row(t * kBN + 2 * RS + st_r, kst2, vst2);
      fetch_row(t * kBN + 3 * RS + st_r, kst3, vst3);
    }
    if (BIAS && tid < kBN) {
      const int jg = t * kBN + tid;
      bst = T::to_float(bp[jg < N ? jg : N - 1]) * 1.44269504088896340736f;
    }
  };
  auto stash = [&](int buf) {
    if (BIAS && tid < kBN) lds_b[buf][tid] = bst;
    *(uint4*)&lds_k[buf][st_r * SK + st_c] = kst0;
    *(uint4*)&lds_v[buf][st_r * SV + st_c] = vst0;
    if (NST > 1) {
      *(uint4*)&lds_k[buf][(RS + st_r) * SK + st_c] = kst1;
      *(uint4*)&lds_v[buf][(RS + st_r) * SV + st_c] = vst1;
    }
    if (NST > 2) {
      *(uint4*)&lds_k[buf][(2 * RS + st_r) * SK + st_c] = kst2;
      *(uint4*)&lds_v[buf][(2 * RS + st_r) * SV + st_c] = vst2;
      *(uint4*)&lds_k[buf][(3 * RS + st_r) * SK + st_c] = kst3;
      *(uint4*)&lds_v[buf][(3 * RS + st_r) * SV + st_c] = vst3;
    }
  };

  fetch(t_lo);
  stash(0);
  __syncthreads();
  // rotary embedding: a staged K tile is rotated in place before anybody reads it
  if (a.rope_cos) {
    rope_rows_in_lds<T, D>(a, lds_k[0], SK, kBN, t_lo * kBN, tid, kThreads);
    __syncthreads();
  }

  int buf = 0;
  for (int t = t_lo; t < t_hi; ++t) {
    if (t + 1 < t_hi) fetch(t + 1);
    if (wave_has_rows) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const int kb0 = t * kBN + kb * 32;
        // wavefront-uniform: skip key blocks no query of this wavefront sees
        if (kb0 >= n) continue;
        if (a.wl >= 0 && kb0 + 31 < qw0 - a.wl) continue;
        if (a.wr >= 0 && kb0 > qw_last + a.wr) continue;
        simple_block<T, NQB, true, V_TR ? 0 : 1>(st, qreg, &lds_k[buf][kb * 32 * SK], &lds_v[buf][kb * 32 * SV],
                                                 kb0, jlo, jhi, lane, a.c, a.tau_raw,
                                                 BIAS ? &lds_b[buf][kb * 32] : nullptr);
      }
    }
    if (t + 1 < t_hi) stash(buf ^ 1);
    __syncthreads();
    buf ^= 1;
    if (a.rope_cos && t + 1 < t_hi) {
      rope_rows_in_lds<T, D>(a, lds_k[buf], SK, kBN, (t + 1) * kBN, tid, kThreads);
      __syncthreads();
    }
  }
  // the loop ended with a barrier: the K stages are free
  epilogue<T, NQB>(a, st, op, lsep, qw0, n, lane, &lds_k[0][0] + wave * epi_patch(D));
}

// ======================================================================================
// Window kernel: local layers.  The key range of a 128-row query tile is only a few
// hundred keys, so the work is bound by getting K/V (and Q, O) through HBM once and by
// latency: K/V move in 32-key blocks through a ring of kWinStages LDS stages filled by
// direct global->LDS loads, kWinStages - 1 blocks ahead of the arithmetic (small stages
// keep several workgroups per compute unit AND several blocks per workgroup in flight).
// A wavefront multiplies only the blocks its own 32 queries can see; blocks it sees
// completely skip the mask work.  One barrier per block.
// ======================================================================================
constexpr int kWinStages = 4;
constexpr int kWinBN = 32;  // keys per stage

template <class T>
__global__ __launch_bounds__(kThreads, 2) void fa_fwd_window_kernel(const FaKernelArgs a) {
  constexpr int BM = kWaves * 32;
  // at least the four 32 x 72 epilogue patches must fit in lds_k
  constexpr int kStageElems = kWinBN * kD;
  constexpr int kKElems = kWinStages * kStageElems > kWaves * kEpiPatch ? kWinStages * kStageElems : kWaves * kEpiPatch;
  __shared__ __attribute__((aligned(16))) uint16_t lds_k[kKElems];
  __shared__ __attribute__((aligned(16))) uint16_t lds_v[kWinStages * kStageElems];

  TileCoord tc;
  if (!locate_tile<BM>(a, tc)) return;
  const int N = a.max_len, n = tc.n, q0 = tc.q0;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31;

  const uint16_t* qp = (const uint16_t*)a.q + tc.b * a.qs[0] + tc.h * a.qs[1];
  const uint16_t* kp = (const uint16_t*)a.k + tc.b * a.ks[0] + tc.h * a.ks[1];
  const uint16_t* vp = (const uint16_t*)a.v + tc.b * a.vs[0] + tc.h * a.vs[1];
  uint16_t* op = (uint16_t*)a.o + tc.b * a.os[0] + tc.h * a.os[1];
  float* lsep = a.lse ? a.lse + ((int64_t)tc.b * a.heads + tc.h) * N : nullptr;

  if (q0 >= n) {
    zero_fill<BM>(a, tc, op, lsep);
    return;
  }

  // key range of this workgroup, in 32-key blocks
  const int q_last = (q0 + BM < n ? q0 + BM : n) - 1;
  int lo = 0, hi = n;
  if (a.wl >= 0) lo = q0 - a.wl > 0 ? q0 - a.wl : 0;
  if (a.wr >= 0) hi = q_last + a.wr + 1 < n ? q_last + a.wr + 1 : n;
  const int t_lo = lo / kWinBN;
  const int t_hi = (hi + kWinBN - 1) / kWinBN;

  // Block t goes to stage t % kWinStages.  Wavefront w moves rows 8w..8w+7 of the block
  // (one 1 KB load each for K and V); a lane's row is clamped to the last row of the
  // tensor (rows >= n are masked or zeroed below), so its global offset is a per-lane
  // 32-bit byte offset from the (batch, head) slice.
  const int dl_r = 8 * wave + (lane >> 3);
  const uint32_t kchunk = 2u * (uint32_t)(((lane & 7) ^ k_swz(dl_r)) * 8);
  const uint32_t vchunk = 2u * (uint32_t)(((lane & 7) ^ v_swz(dl_r)) * 8);
  const uint32_t krow_b = 2u * (uint32_t)a.ks[2], vrow_b = 2u * (uint32_t)a.vs[2];
  auto issue_block = [&](int t) {
    const int stage = t % kWinStages;
    const int jg = t * kWinBN + dl_r;
    const uint32_t jc = (uint32_t)(jg < N ? jg : N - 1);
    load16_to_lds(kp, jc * krow_b + kchunk, &lds_k[stage * kStageElems + 8 * wave * kD]);
    load16_to_lds(vp, jc * vrow_b + vchunk, &lds_v[stage * kStageElems + 8 * wave * kD]);
  };
  // After a block has landed: V rows at or beyond n are overwritten with zeros by the
  // lanes that fetched them (0 * whatever is stored in the padding must be 0).
  auto scrub_block = [&](int t) {
    if (t * kWinBN + kWinBN <= n) return;
    if (t * kWinBN + dl_r >= n)
      *(uint4*)&lds_v[(t % kWinStages) * kStageElems + dl_r * kD + (lane & 7) * 8] = make_uint4(0, 0, 0, 0);
  };

  // prologue: kWinStages - 1 blocks in flight before anything else
#pragma unroll
  for (int i = 0; i < kWinStages - 1; ++i)
    if (t_lo + i < t_hi) issue_block(t_lo + i);

  const int qw0 = q0 + wave * 32;
  const int qw_last = (qw0 + 32 < n ? qw0 + 32 : n) - 1;  // < qw0: all padding
  const bool wave_has_rows = qw_last >= qw0;
  typename T::v8 qreg[1][4];
  load_q<T, 1, 4, false>(a, qp, qw0, lane, qreg);
  RowState<1> st;
  init_state(st);
  int jlo[1], jhi[1];
  {
    const int ig = qw0 + l32;
    jlo[0] = 0;
    jhi[0] = n - 1;
    if (a.wl >= 0 && ig - a.wl > jlo[0]) jlo[0] = ig - a.wl;
    if (a.wr >= 0 && ig + a.wr < jhi[0]) jhi[0] = ig + a.wr;
  }

  for (int t = t_lo; t < t_hi; ++t) {
    // Each block is 2 loads per wavefront, and loads complete in order: block t has landed
    // once at most 2 * (number of younger blocks in flight) loads are outstanding.
    const int younger = (t_hi - 1 - t < kWinStages - 2 ? t_hi - 1 - t : kWinStages - 2);
    if (younger >= 2) wait_vmcnt<4>();
    else if (younger == 1) wait_vmcnt<2>();
    else wait_vmcnt<0>();
    scrub_block(t);
    __syncthreads();
    // stage (t-1) % kWinStages is free now: every wavefront finished block t-1 before this barrier
    if (t + kWinStages - 1 < t_hi) issue_block(t + kWinStages - 1);
    const int kb0 = t * kWinBN;
    // wavefront-uniform: skip key blocks no query of this wavefront sees
    if (!wave_has_rows || kb0 >= n) continue;
    if (a.wl >= 0 && kb0 + 31 < qw0 - a.wl) continue;
    if (a.wr >= 0 && kb0 > qw_last + a.wr) continue;
    // blocks every valid query of the wavefront sees completely need no mask work
    const bool interior = kb0 + 32 <= n && (a.wl < 0 || kb0 >= qw_last - a.wl) &&
                          (a.wr < 0 || kb0 + 31 <= qw0 + a.wr);
    const uint16_t* kblk = &lds_k[(t % kWinStages) * kStageElems];
    const uint16_t* vblk = &lds_v[(t % kWinStages) * kStageElems];
    if (interior) simple_block<T, 1, false, 2>(st, qreg, kblk, vblk, kb0, jlo, jhi, lane, a.c, a.tau_raw);
    else simple_block<T, 1, true, 2>(st, qreg, kblk, vblk, kb0, jlo, jhi, lane, a.c, a.tau_raw);
  }
  __syncthreads();  // all blocks consumed: the K stages become the epilogue patches
  epilogue<T, 1>(a, st, op, lsep, qw0, n, lane, lds_k + wave * kEpiPatch);
}

// ======================================================================================
// Resident window kernel: local layers whose whole key range per 128-row query tile fits
// in kResBlocks 32-key blocks of LDS (the paper's 63/64 window needs exactly 8).  All of
// the tile's K/V is requested at once with direct global->LDS loads, one barrier
// publishes it, and then every wavefront runs the same software pipeline as the global
// kernel over just the blocks its own 32 queries can see - next block's scores and the
// previous block's P.V on the matrix cores while the vector ALU forms this block's
// probabilities - with mask work only on the blocks that are cut by the window or the
// sequence end.  No further barriers until the epilogue.
// ======================================================================================
constexpr int kResBlocks = 8;

template <class T, bool BIAS = false>
__global__ __launch_bounds__(kThreads, 2) void fa_fwd_window_resident_kernel(const FaKernelArgs a) {
  constexpr int BM = kWaves * 32;
  constexpr int kBlk = 32 * kD;  // elements per block
  __shared__ __attribute__((aligned(16))) uint16_t lds_k[kResBlocks * kBlk];
  __shared__ __attribute__((aligned(16))) uint16_t lds_v[kResBlocks * kBlk];
  // BIAS: additive key bias / |scale| of every resident key; it enters the scores as the C
  // operand of each block's first MFMA
  __shared__ __attribute__((aligned(16))) float lds_bias[BIAS ? kResBlocks * 32 : 4];

  fetch_args();
  TileCoord tc;
  if (!locate_tile<BM, false>(a, tc)) return;  // tc.n still as loaded: see below
  const int N = a.max_len, q0 = tc.q0;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;

  const uint16_t* qp = (const uint16_t*)a.q + tc.b * a.qs[0] + tc.h * a.qs[1];
  const uint16_t* kp = (const uint16_t*)a.k + tc.b * a.ks[0] + tc.h * a.ks[1];
  const uint16_t* vp = (const uint16_t*)a.v + tc.b * a.vs[0] + tc.h * a.vs[1];
  uint16_t* op = (uint16_t*)a.o + tc.b * a.os[0] + tc.h * a.os[1];
  float* lsep = a.lse ? a.lse + ((int64_t)tc.b * a.heads + tc.h) * N : nullptr;

  // Key blocks this tile can touch, from the tile position and the tensor length alone: the
  // loads below are issued BEFORE the sequence length is looked at, so that the latency of
  // reading it (it sits in device memory) overlaps theirs instead of preceding it - a
  // workgroup that is alone on its compute unit (short sequences) has nothing else to hide
  // it behind.  Block b lives in slot b - b_lo; blocks past the sequence end are fetched and
  // never read.
  const int lo = q0 - a.wl > 0 ? q0 - a.wl : 0;
  const int b_lo = lo >> 5;
  int b_hi_ld = (q0 + BM + a.wr + 31) >> 5;
  b_hi_ld = b_hi_ld < ((N + 31) >> 5) ? b_hi_ld : ((N + 31) >> 5);
  if (b_hi_ld > b_lo + kResBlocks) b_hi_ld = b_lo + kResBlocks;  // never true for the windows the host routes here

  // Wavefront w moves rows 8w..8w+7 of every block (one 1 KB load each for K and V).  A
  // lane's row is clamped to the last row of the tensor (rows >= n are masked or zeroed
  // below), so its global offset is a per-lane 32-bit byte offset from the slice.
  const int dl_r = 8 * wave + (lane >> 3);
  {
    const int b_hi = b_hi_ld;
    const uint32_t kchunk = 2u * (uint32_t)(((lane & 7) ^ k_swz(dl_r)) * 8);
    const uint32_t vchunk = 2u * (uint32_t)(((lane & 7) ^ v_swz(dl_r)) * 8);
    const uint32_t krow_b = 2u * (uint32_t)a.ks[2], vrow_b = 2u * (uint32_t)a.vs[2];
    if (b_hi * 32 <= N) {
      // every row exists: one per-lane offset, the block base advances in scalar registers
      const uint32_t klane = (uint32_t)dl_r * krow_b + kchunk, vlane = (uint32_t)dl_r * vrow_b + vchunk;
      const uint16_t* kg = kp + (int64_t)b_lo * 32 * a.ks[2];
      const uint16_t* vg = vp + (int64_t)b_lo * 32 * a.vs[2];
#pragma unroll
      for (int i = 0; i < kResBlocks; ++i) {
        if (b_lo + i < b_hi) {
          load16_to_lds(kg, klane, &lds_k[i * kBlk + 8 * wave * kD]);
          load16_to_lds(vg, vlane, &lds_v[i * kBlk + 8 * wave * kD]);
          kg += 32 * a.ks[2];
          vg += 32 * a.vs[2];
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < kResBlocks; ++i) {
        if (b_lo + i < b_hi) {
          const int jg = (b_lo + i) * 32 + dl_r;
          const uint32_t jc = (uint32_t)(jg < N ? jg : N - 1);
          load16_to_lds(kp, jc * krow_b + kchunk, &lds_k[i * kBlk + 8 * wave * kD]);
          load16_to_lds(vp, jc * vrow_b + vchunk, &lds_v[i * kBlk + 8 * wave * kD]);
        }
      }
    }
  }

  if (BIAS) {
    // one value per thread: key b_lo*32 + tid (256 resident keys, 256 threads)
    const uint16_t* bp = (const uint16_t*)a.key_bias + tc.b * a.kb_stride;
    const int jg = b_lo * 32 + tid;
    lds_bias[tid] = bias_over_scale<T, false>(a, bp[jg < N ? jg : N - 1]);
  }

  const int qw0 = q0 + wave * 32;
  typename T::v8 qreg[1][4];
  load_q<T, 1, 4, false>(a, qp, qw0, lane, qreg);

  // only now the sequence length
  const int n = tc.n < 0 ? 0 : (tc.n > N ? N : tc.n);
  tc.n = n;
  if (q0 >= n) {
    wait_direct_loads();  // the loads write this workgroup's LDS: they must land before it ends
    zero_fill<BM>(a, tc, op, lsep);
    return;
  }
  const int q_last = (q0 + BM < n ? q0 + BM : n) - 1;
  const int hi = q_last + a.wr + 1 < n ? q_last + a.wr + 1 : n;
  int b_hi = (hi + 31) >> 5;  // blocks [b_lo, b_hi) hold visible keys
  if (b_hi > b_hi_ld) b_hi = b_hi_ld;
  const int qw_last = (qw0 + 32 < n ? qw0 + 32 : n) - 1;  // < qw0: all padding
  const bool wave_has_rows = qw_last >= qw0;
  RowState<1> st;
  init_state(st);
  const int ig = qw0 + l32;
  const bool alive = ig < n;
  int jlo = ig - a.wl > 0 ? ig - a.wl : 0;
  int jhi = ig + a.wr < n - 1 ? ig + a.wr : n - 1;
  const float c = a.c;

  wait_direct_loads();
  // V rows at or beyond n are overwritten with zeros by the lanes that fetched them
  // (0 * whatever is stored in the padding must be 0); only the last block can have any
  {
    const int i = b_hi - 1 - b_lo;
    if ((b_hi - 1) * 32 + dl_r >= n) *(uint4*)&lds_v[i * kBlk + dl_r * kD + (lane & 7) * 8] = make_uint4(0, 0, 0, 0);
  }
  __syncthreads();

  if (wave_has_rows) {
    // blocks this wavefront's queries can see
    int fb = (qw0 - a.wl) >> 5;
    fb = fb < b_lo ? b_lo : fb;
    int lb = (qw_last + a.wr) >> 5;
    lb = lb > b_hi - 1 ? b_hi - 1 : lb;

    floatx16 sA, sB;
    typename T::v8 pA[2], pB[2];
    pA[0] = pA[1] = as_v8<T>(make_uint4(0, 0, 0, 0));
    // accumulator input of a block's score product: its bias, or zero
    auto score_init = [&](floatx16& sv, int slot) {
      if (BIAS) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 b4 = *(const float4*)&lds_bias[slot * 32 + 8 * g + 4 * hh];
          sv[4 * g + 0] = b4.x;
          sv[4 * g + 1] = b4.y;
          sv[4 * g + 2] = b4.z;
          sv[4 * g + 3] = b4.w;
        }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) sv[r] = 0.f;
      }
    };
    score_init(sA, fb - b_lo);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      sA = T::mfma(load_k_frag_swz<T>(&lds_k[(fb - b_lo) * kBlk], l32, hh, ks), qreg[0][ks], sA);

    // One unit of the pipeline: probabilities of block u; scores of block u+1; P.V of
    // block u-1.  At the two ends the neighbour slot is clamped: its product is unused
    // (scores) or multiplied by zero probabilities (P.V).
    auto unit = [&](floatx16& s_cur, floatx16& s_nxt, typename T::v8 (&p_prev)[2], typename T::v8 (&p_cur)[2], int u) {
      const int un = u + 1 > b_hi - 1 ? b_hi - 1 : u + 1;
      const int up = u - 1 < b_lo ? b_lo : u - 1;
      // blocks every valid query of the wavefront sees completely need no mask work
      const int kb0 = u * 32;
      const bool interior = kb0 + 32 <= n && kb0 >= qw_last - a.wl && kb0 + 31 <= qw0 + a.wr;
      resident_unit<T>(st, qreg, s_cur, s_nxt, p_prev, p_cur, &lds_k[(un - b_lo) * kBlk],
                             &lds_v[(up - b_lo) * kBlk], [&](floatx16& sv) { score_init(sv, un - b_lo); }, kb0,
                             interior, jlo, jhi, alive, c, lane);
    };
    auto drain = [&](typename T::v8 (&p_last)[2], int u) {
      const uint16_t* vblk = &lds_v[(u - b_lo) * kBlk];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        st.oacc[0][i & 1] = T::mfma(load_vt_frag_swz<T>(vblk, lane, i >> 1, i & 1), p_last[i >> 1], st.oacc[0][i & 1]);
    };
    int u = fb;
    for (; u + 1 <= lb; u += 2) {
      unit(sA, sB, pA, pB, u);
      unit(sB, sA, pB, pA, u + 1);
    }
    if (u <= lb) {
      unit(sA, sB, pA, pB, u);
      drain(pB, u);
    } else {
      drain(pA, lb);
    }
  }
  __syncthreads();  // all blocks consumed: the K storage becomes the epilogue patches
  epilogue<T, 1>(a, st, op, lsep, qw0, n, lane, lds_k + wave * kEpiPatch);
}

// ======================================================================================
// Two-phase window kernel: local layers of head_dim 64 in which a wavefront's 32 queries see at
// most kTwoPhaseBlocks 32-key blocks (the paper's 63/64 window: five) and a 128-row tile at
// most kResBlocks.  Such a layer is bound by memory traffic (64 flop per byte), and what
// decides its speed is how many workgroups a compute unit holds at once: workgroups load,
// compute and store one after the other, so the more of them are resident, the more of the
// time the memory system has requests in flight.  With K and V both resident in LDS (64 KB,
// the kernel above) that is two workgroups per unit.  Here ONE 32 KB region holds the K
// blocks first and the V blocks afterwards, which allows four workgroups per unit:
//   phase 1: K blocks arrive by direct loads; every wavefront forms the scores of ALL its
//            visible blocks (up to 5 x 16 accumulator registers per lane: a whole window row
//            fits in registers), barrier;
//   phase 2: the V blocks are requested into the same region, and while they travel the
//            wavefront turns its scores into probabilities - an ordinary softmax over the
//            whole row: exact maximum, no running reference, nothing to rescale;
//   phase 3: V has landed (barrier): O^T = sum over blocks of V^T P^T, epilogue.
// No software pipeline inside a wavefront: the four wavefronts a SIMD holds are in different
// phases and fill each other's gaps.  (Touching V's cache lines at the start, so that the
// phase-2 request finds them in cache, measured 8 % slower on a cold cache: not done.)
// ======================================================================================
constexpr int kTwoPhaseBlocks = 5;

// OPT: a rotation (kTwoPhaseRope) or a key bias (kTwoPhaseBias) is a compile-time variant.
//   Rotation: the K blocks are rotated in place in LDS, once for the four wavefronts.  What that costs is the angle
//   tables: 256 bytes per row, as much as its K and V.  So each row's entries are read once per workgroup: a wavefront
//   rotates the K block of its own 32 queries' rows, the same entries rotate those queries, and one block of the halo; four
//   lanes (head_dim 64) read a row side by side, and the queries change into the operand layout, one row per lane, through a
//   small patch.  (Queries rotated where they are used, from table rows of their own, 32 rows per load instruction, took as
//   long as all of K: us, rotated -> this, bf16, packed, 8K 12 x 64 16.8 -> 15.3, 8 x 128 22.6 -> 19.1, 24 x 32 16.9 -> 16.4,
//   487 tokens 8.7 -> 7.6, 32K 12 x 64 64.0 -> 55.6; without a rotation 12.6 at 8K, 42 at 32K.)
//   Bias, head_dim 32 and 128: each key's bias divided by |scale| is added to its block's finished scores, so that a score
//   near -65504 is rounded once, not in every product of the chain, and the row sums are those of the unrounded
//   probabilities, both as in the masked kernel.  head_dim 64: it is the C operand of its block's first score product and
//   fp16 sums are those of the rounded probabilities, both as in the resident kernel (which small calls of this head size
//   run); adding it afterwards does not fit the 128 registers of four wavefronts per SIMD (8K tokens 14 -> 319 us).
enum { kTwoPhasePlain = 0, kTwoPhaseRope = 1, kTwoPhaseBias = 2 };

template <class T, int D, int OPT = kTwoPhasePlain>
__global__ __launch_bounds__(kThreads, D == 128 ? 2 : 4) void fa_fwd_window_twophase_kernel(const FaKernelArgs a) {
  constexpr bool ROPE = OPT == kTwoPhaseRope, BIAS = OPT == kTwoPhaseBias, BIAS_LAST = BIAS && D != 64;
  constexpr int BM = kWaves * 32;
  constexpr int KS = D / 16, DB = D / 32;
  constexpr int kBlk = 32 * D;  // elements per block
  static_assert(kResBlocks * kBlk >= kWaves * epi_patch(D), "the region doubles as the epilogue patches");
  // BIAS: the region is followed by the keys' biases; ROPE: by a patch per wavefront through which rotated Q rows reach the
  // lanes of the operand layout, kQRows at a time (head_dim 64: 40 KB a workgroup, a quarter of the unit's LDS)
  constexpr int kQRows = D == 32 ? 32 : 16;
  __shared__ __attribute__((aligned(16))) uint16_t lds[kResBlocks * kBlk + (BIAS ? kResBlocks * 64 : ROPE ? kWaves * kQRows * D : 0)];
  float* const lds_bias = (float*)(lds + kResBlocks * kBlk);

  TileCoord tc;
  if (!locate_tile<BM, false, ROPE || D == 32>(a, tc)) return;  // tc.n still as loaded: see below
  const int N = a.max_len, q0 = tc.q0;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;

  const uint16_t* qp = (const uint16_t*)a.q + tc.b * a.qs[0] + tc.h * a.qs[1];
  const uint16_t* kp = (const uint16_t*)a.k + tc.b * a.ks[0] + tc.h * a.ks[1];
  const uint16_t* vp = (const uint16_t*)a.v + tc.b * a.vs[0] + tc.h * a.vs[1];
  uint16_t* op = (uint16_t*)a.o + tc.b * a.os[0] + tc.h * a.os[1];
  float* lsep = a.lse ? a.lse + ((int64_t)tc.b * a.heads + tc.h) * N : nullptr;

  // Key blocks this tile can touch, from the tile position and the tensor length alone (the
  // sequence length is looked at only after the loads are on their way).  Block b lives in
  // slot b - b_lo; blocks past the sequence end are fetched and never read.
  const int lo = q0 - a.wl > 0 ? q0 - a.wl : 0;
  const int b_lo = lo >> 5;
  int b_hi_ld = (q0 + BM + a.wr + 31) >> 5;
  b_hi_ld = b_hi_ld < ((N + 31) >> 5) ? b_hi_ld : ((N + 31) >> 5);
  if (b_hi_ld > b_lo + kResBlocks) b_hi_ld = b_lo + kResBlocks;  // never true for the windows the host routes here

  // A direct load moves 1 KB = RPL rows of a block (lane L: row L / CH, chunk position L % CH of
  // the load), so a block is LPB loads; the loads of all blocks, numbered block * LPB + part,
  // are dealt round-robin to the four wavefronts: wavefront w issues loads w, w + 4, w + 8, ...
  //   head_dim 64 (LPB 4): load x of the wavefront is block x, part w;
  //   head_dim 128 (LPB 8): block x / 2, part w + 4 (x % 2);
  //   head_dim 32 (LPB 2): block 2 x + w / 2, part w % 2.
  // So a wavefront has NPART (1 or 2) distinct parts, whose per-lane offsets are computed once,
  // and its blocks advance by a fixed step: the scalar base moves by a 64-bit add per block.
  // A lane's row is clamped to the last row of the tensor where the tile reaches past it (rows
  // >= n are masked or zeroed below); its global offset is then a per-lane 32-bit byte offset
  // from the slice.
  constexpr int CH = D / 8, RPL = 64 / CH, LPB = 32 / RPL;   // D = 32: 4, 16, 2;  64: 8, 8, 4;  128: 16, 4, 8
  constexpr int kLoadsPerWave = kResBlocks * LPB / kWaves;
  constexpr int NPART = LPB > kWaves ? LPB / kWaves : 1;
  constexpr int BSTEP = LPB < kWaves ? kWaves / LPB : 1;     // blocks between consecutive loads of one part
  const int blk0 = LPB < kWaves ? wave / LPB : 0;            // the wavefront's first block
  const bool all_rows_exist = b_hi_ld * 32 <= N;   // workgroup-uniform
  auto request_blocks = [&](const uint16_t* base, int64_t row_elems, bool is_k) {
    const uint32_t row_bytes = 2u * (uint32_t)row_elems;
    int row_of[NPART];            // row within a block that this lane fetches, per part
    uint32_t chunk_bytes[NPART];  // byte offset of its (swizzled) 16-byte chunk within the row
    uint32_t lds_part[NPART];     // element offset of the part within a block's LDS slot
#pragma unroll
    for (int pi = 0; pi < NPART; ++pi) {
      const int part = LPB >= kWaves ? wave + kWaves * pi : wave % LPB;
      row_of[pi] = part * RPL + lane / CH;
      const int swz = is_k ? k_swz_d<D>(row_of[pi]) : v_swz_d<D>(row_of[pi]);
      chunk_bytes[pi] = 2u * (uint32_t)(((lane % CH) ^ swz) * 8);
      lds_part[pi] = (uint32_t)(part * RPL * D);
    }
    if (all_rows_exist) {
      uint32_t lane_off[NPART];
#pragma unroll
      for (int pi = 0; pi < NPART; ++pi) lane_off[pi] = (uint32_t)row_of[pi] * row_bytes + chunk_bytes[pi];
      const int64_t blk_elems = 32 * row_elems;
      const uint16_t* g = base + (int64_t)(b_lo + blk0) * blk_elems;
#pragma unroll
      for (int x = 0; x < kLoadsPerWave; ++x) {
        const int pi = x % NPART;
        const int i = blk0 + (x / NPART) * BSTEP;   // wavefront-uniform
        if (b_lo + i < b_hi_ld) load16_to_lds(g, lane_off[pi], &lds[i * kBlk + lds_part[pi]]);
        if (pi == NPART - 1) g += BSTEP * blk_elems;
      }
    } else {
#pragma unroll
      for (int x = 0; x < kLoadsPerWave; ++x) {
        const int pi = x % NPART;
        const int i = blk0 + (x / NPART) * BSTEP;
        if (b_lo + i < b_hi_ld) {
          const int jg = (b_lo + i) * 32 + row_of[pi];
          const uint32_t jc = (uint32_t)(jg < N ? jg : N - 1);
          load16_to_lds(base, jc * row_bytes + chunk_bytes[pi], &lds[i * kBlk + lds_part[pi]]);
        }
      }
    }
  };
  if (!ROPE) request_blocks(kp, a.ks[2], true);

  const int qw0 = q0 + wave * 32;
  // ROPE: a wavefront fetches two of the region's blocks, the one whose keys are its own 32 queries and one of the four
  // others, and rotates them in place: what it fetched it may read without a barrier.  An item of a lane is a pair of chunks
  // (c, c + HALF) of one row, HALF lanes a row; the angles of the wavefront's own rows rotate its queries as well.
  constexpr int HALF = D / 16, RI = 64 / HALF, NI = 32 / RI;    // lanes per row; rows per item, items per block: D = 32, 64, 128: 32, 1; 16, 2; 8, 4
  const int own_blk = (q0 >> 5) - b_lo + wave;                   // (region-relative; tiles start at multiples of 128)
  const int halo_blk = wave < own_blk - wave ? wave : wave + 4;
  const bool halo_there = b_lo + halo_blk < b_hi_ld;             // wavefront-uniform
  const int rope_c = lane % HALF;
  struct Angles {
    float4 c[2], s[2];
  };
  uint4 q_raw[ROPE ? NI : 1][2];
  Angles t_own[ROPE ? NI : 1], t_halo[ROPE ? NI : 1];
  // the row of item x in a region block (clamped into the tensor: rows outside it are never used unmasked)
  auto item_row = [&](int blk, int x) {
    const int row = 32 * (b_lo + blk) + RI * x + lane / HALF;
    return row < N ? row : N - 1;
  };
  auto load_angles = [&](int blk, int x, Angles& g) {
    const int64_t at = (int64_t)item_row(blk, x) * a.rope_stride + 8 * rope_c;
    const float4 *cs = (const float4*)(a.rope_cos + at), *sn = (const float4*)(a.rope_sin + at);
    g.c[0] = cs[0]; g.c[1] = cs[1]; g.s[0] = sn[0]; g.s[1] = sn[1];
  };
  // item x of a 32-row block in LDS
  auto lo_at = [&](uint16_t* blk, int x) { return (uint4*)&blk[(RI * x + lane / HALF) * D + ((rope_c ^ k_swz_d<D>(RI * x + lane / HALF)) * 8)]; };
  auto hi_at = [&](uint16_t* blk, int x) { return (uint4*)&blk[(RI * x + lane / HALF) * D + (((rope_c + HALF) ^ k_swz_d<D>(RI * x + lane / HALF)) * 8)]; };
  auto rotate_item = [&](uint16_t* blk, int x, const Angles& g) {
    uint4 lo = *lo_at(blk, x), hi = *hi_at(blk, x);
    rotate8<T>(lo, hi, (const float*)g.c, (const float*)g.s);
    *lo_at(blk, x) = lo;
    *hi_at(blk, x) = hi;
  };
  if (ROPE) {
#pragma unroll
    for (int x = 0; x < NI; ++x) {
      const uint16_t* src = qp + item_row(own_blk, x) * a.qs[2] + 8 * rope_c;
      q_raw[x][0] = *(const uint4*)src;
      q_raw[x][1] = *(const uint4*)(src + 8 * HALF);
      load_angles(own_blk, x, t_own[x]);
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int blk = s == 0 ? own_blk : halo_blk, first = 32 * (b_lo + blk);
      if (b_lo + blk < b_hi_ld) {
        const uint16_t* g = kp + (int64_t)first * a.ks[2];
#pragma unroll
        for (int x = 0; x < LPB; ++x) {
          const int r = RPL * x + lane / CH, rc = r < N - 1 - first ? r : N - 1 - first;
          load16_to_lds(g, 2u * ((uint32_t)rc * (uint32_t)a.ks[2] + (uint32_t)(((lane % CH) ^ k_swz_d<D>(r)) * 8)), lds + blk * kBlk + RPL * x * D);
        }
      }
    }
    if (halo_there) {
#pragma unroll
      for (int x = 0; x < NI; ++x) load_angles(halo_blk, x, t_halo[x]);
    }
  }
  uint16_t bias_bits = 0;   // one value per thread: key b_lo*32 + tid (256 keys, 256 threads); used once K has landed
  if (BIAS) {
    const uint16_t* bp = (const uint16_t*)a.key_bias + tc.b * a.kb_stride;
    const int jg = b_lo * 32 + tid;
    bias_bits = bp[jg < N ? jg : N - 1];
  }

  typename T::v8 qreg[1][KS];
  if (!ROPE) load_q<T, 1, KS, false>(a, qp, qw0, lane, qreg);

  // only now the sequence length
  const int n = tc.n < 0 ? 0 : (tc.n > N ? N : tc.n);
  tc.n = n;
  if (q0 >= n) {
    wait_direct_loads();  // the loads write this workgroup's LDS: they must land before it ends
    zero_fill<BM, D>(a, tc, op, lsep);
    return;
  }
  const int q_last = (q0 + BM < n ? q0 + BM : n) - 1;
  const int hi = q_last + a.wr + 1 < n ? q_last + a.wr + 1 : n;
  int b_hi = (hi + 31) >> 5;  // blocks [b_lo, b_hi) hold visible keys
  if (b_hi > b_hi_ld) b_hi = b_hi_ld;
  const int qw_last = (qw0 + 32 < n ? qw0 + 32 : n) - 1;  // < qw0: all padding
  const bool wave_has_rows = qw_last >= qw0;
  const int ig = qw0 + l32;
  const int jlo = ig - a.wl > 0 ? ig - a.wl : 0;
  const int jhi = ig + a.wr < n - 1 ? ig + a.wr : n - 1;
  const float c = a.c;
  // blocks this wavefront's queries can see: fb .. fb + cnt - 1, cnt <= kTwoPhaseBlocks
  int fb = (qw0 - a.wl) >> 5;
  fb = fb < b_lo ? b_lo : fb;
  int lb = (qw_last + a.wr) >> 5;
  lb = lb > b_hi - 1 ? b_hi - 1 : lb;
  int cnt = wave_has_rows ? lb - fb + 1 : 0;
  cnt = cnt > kTwoPhaseBlocks ? kTwoPhaseBlocks : cnt;  // (the host routes no wider window here)

  // ---- phase 1: scores of every visible block
  if (ROPE) {
    uint16_t* const patch = lds + kResBlocks * kBlk + wave * kQRows * D;
    const uint32_t flip = a.negate_q ? 0x80008000u : 0u;
    // queries: rotated, through the patch, into the operand layout (the same wavefront writes and reads it: program order
    // is enough)
#pragma unroll
    for (int half = 0; half < 32 / kQRows; ++half) {
      uint16_t* const rows = patch - half * kQRows * D;   // where row 0 of the block would be
#pragma unroll
      for (int x = 0; x < NI; ++x) {
        if (RI * x / kQRows != half) continue;
        rotate8<T>(q_raw[x][0], q_raw[x][1], (const float*)t_own[x].c, (const float*)t_own[x].s);
        *lo_at(rows, x) = q_raw[x][0];
        *hi_at(rows, x) = q_raw[x][1];
      }
      __builtin_amdgcn_wave_barrier();
      if (l32 / kQRows == half) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          uint4 u = __builtin_bit_cast(uint4, load_k_frag_swz_d<T, D>(rows, l32, hh, ks));
          u.x ^= flip; u.y ^= flip; u.z ^= flip; u.w ^= flip;
          qreg[0][ks] = as_v8<T>(u);
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
    wait_direct_loads();
#pragma unroll
    for (int x = 0; x < NI; ++x) rotate_item(lds + own_blk * kBlk, x, t_own[x]);
    if (halo_there) {
#pragma unroll
      for (int x = 0; x < NI; ++x) rotate_item(lds + halo_blk * kBlk, x, t_halo[x]);
    }
  } else {
    wait_direct_loads();
  }
  if (BIAS) lds_bias[tid] = bias_over_scale<T, BIAS_LAST>(a, bias_bits);
  __syncthreads();
  floatx16 sc[kTwoPhaseBlocks];   // sc[i] is set and used for i < cnt only
#pragma unroll
  for (int i = 0; i < kTwoPhaseBlocks; ++i) {
    if (i < cnt) {
      if (BIAS && !BIAS_LAST) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 b4 = *(const float4*)&lds_bias[(fb + i - b_lo) * 32 + 8 * g + 4 * hh];
          sc[i][4 * g + 0] = b4.x; sc[i][4 * g + 1] = b4.y; sc[i][4 * g + 2] = b4.z; sc[i][4 * g + 3] = b4.w;
        }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[i][r] = 0.f;
      }
      const uint16_t* kblk = &lds[(fb + i - b_lo) * kBlk];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) sc[i] = T::mfma(load_k_frag_swz_d<T, D>(kblk, l32, hh, ks), qreg[0][ks], sc[i]);
      if (BIAS_LAST) add_bias(sc[i], &lds_bias[(fb + i - b_lo) * 32], hh);
    }
  }
  __syncthreads();  // every wavefront has its K fragments out of the region

  // ---- phase 2: request V into the same region; softmax meanwhile
  request_blocks(vp, a.vs[2], false);
  // The paper's window (63 left, 64 right) away from the ends of the sequence: the wavefront's 32
  // queries see five blocks, the middle three completely, and of the outer two query t (0..31)
  // sees keys t+1..31 of the first and keys 0..t of the last: between them exactly one block's
  // worth of keys per query.  The last block's scores are merged into the first's (element by
  // element, the one the query sees), the merged block takes the unmasked path like the middle
  // three, and its probabilities are dealt back to the two blocks for the P.V products.  A
  // masked block costs three times the vector instructions of an unmasked one.
  const bool merged_ends = a.wl == 63 && a.wr == 64 && qw0 >= 64 && qw0 + 96 <= n;   // wavefront-uniform; implies cnt == 5
  if (merged_ends) {
    // accumulator element r is key offset 8 (r / 4) + 4 hh + r % 4 of its block
#pragma unroll
    for (int r = 0; r < 16; ++r) sc[0][r] = 8 * (r >> 2) + (r & 3) <= l32 - 4 * hh ? sc[4][r] : sc[0][r];
  }
  const int cnt2 = merged_ends ? 4 : cnt;   // blocks that go through the softmax
  uint32_t vis[kTwoPhaseBlocks];
  float t0 = -INFINITY;
#pragma unroll
  for (int i = 0; i < kTwoPhaseBlocks; ++i) {
    vis[i] = 0;
    if (i < cnt2) {
      const int kb0 = (fb + i) * 32;
      // blocks every valid query of the wavefront sees completely need no mask work
      const bool interior = (kb0 + 32 <= n && kb0 >= qw_last - a.wl && kb0 + 31 <= qw0 + a.wr) || (i == 0 && merged_ends);
      if (interior) {
        vis[i] = 0xFFFFu;
#pragma unroll
        for (int r = 0; r < 16; r += 2) t0 = fmaxf(fmaxf(t0, sc[i][r]), sc[i][r + 1]);
      } else {
        vis[i] = visible_bits(kb0, hh, jlo, jhi);
#pragma unroll
        for (int r = 0; r < 16; ++r) t0 = fmaxf(t0, keep_or_neg_inf(sc[i][r], vis[i], r));
      }
    }
  }
  RowState<1, D> st;
  init_state(st);
  const float tmax = max_xor32(t0);
  st.m_ref[0] = tmax;
  st.mc[0] = tmax == -INFINITY ? 0.f : tmax * c;   // a row without a visible key: every p is masked to 0
  typename T::v8 pr[kTwoPhaseBlocks][2];
#pragma unroll
  for (int i = 0; i < kTwoPhaseBlocks; ++i) {
    if (i < cnt2) {
      uint32_t pk[8];
      float blk;
      if (vis[i] == 0xFFFFu) prob_block<T, false, BIAS_LAST>(sc[i], c, st.mc[0], vis[i], pk, blk);
      else prob_block<T, true, BIAS_LAST>(sc[i], c, st.mc[0], vis[i], pk, blk);
      st.lsum[0] += blk;
      pr[i][0] = as_v8<T>(make_uint4(pk[0], pk[1], pk[2], pk[3]));
      pr[i][1] = as_v8<T>(make_uint4(pk[4], pk[5], pk[6], pk[7]));
    } else {
      pr[i][0] = pr[i][1] = as_v8<T>(make_uint4(0, 0, 0, 0));
    }
  }
  if (merged_ends) {
    // the merged block's probabilities back to their blocks: pair r holds key offsets k0, k0 + 1
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
      const uint4 u = __builtin_bit_cast(uint4, pr[0][h2]);
      const uint32_t w[4] = {u.x, u.y, u.z, u.w};
      uint32_t first[4], last[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int r = 4 * h2 + x, k0 = 8 * (r >> 1) + 2 * (r & 1), thr = l32 - 4 * hh;
        const uint32_t m = (k0 <= thr ? 0x0000FFFFu : 0u) | (k0 + 1 <= thr ? 0xFFFF0000u : 0u);
        last[x] = w[x] & m;
        first[x] = w[x] & ~m;
      }
      pr[0][h2] = as_v8<T>(make_uint4(first[0], first[1], first[2], first[3]));
      pr[4][h2] = as_v8<T>(make_uint4(last[0], last[1], last[2], last[3]));
    }
  }

  // ---- phase 3: V has landed
  wait_direct_loads();
  // V rows at or beyond n are overwritten with zeros by the lanes that fetched them
  // (0 * whatever is stored in the padding must be 0); only the last block can have any
  {
    const int i = b_hi - 1 - b_lo;
#pragma unroll
    for (int x = 0; x < kLoadsPerWave; ++x) {
      const int j = wave + kWaves * x;
      if (j / LPB == i) {
        const int r = (j % LPB) * RPL + lane / CH;
        if ((b_hi - 1) * 32 + r >= n) *(uint4*)&lds[i * kBlk + r * D + (lane % CH) * 8] = make_uint4(0, 0, 0, 0);
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kTwoPhaseBlocks; ++i) {
    if (i < cnt) {
      const uint16_t* vblk = &lds[(fb + i - b_lo) * kBlk];
#pragma unroll
      for (int ks2 = 0; ks2 < 2; ++ks2)
#pragma unroll
        for (int db = 0; db < DB; ++db)
          st.oacc[0][db] = T::mfma(load_vt_frag_swz_d<T, D>(vblk, lane, ks2, db), pr[i][ks2], st.oacc[0][db]);
    }
  }
  __syncthreads();  // all blocks consumed: the region becomes the epilogue patches
  epilogue<T, 1, D>(a, st, op, lsep, qw0, n, lane, lds + wave * epi_patch(D));
}

// ======================================================================================
// Split kernel: global layers whose query tiles alone would leave SIMDs with one wavefront or
// none (a single request, a few short sequences).  A workgroup is NQ x NK wavefronts: NQ query
// blocks of 32 rows, each shared by NK wavefronts that split the KEYS: in step i wavefront
// (qb, g) takes the 32-key block i NK + g, so the NK NQ wavefronts read one contiguous super
// tile of 32 NK keys, staged once in LDS for all of them.
//
// What bounds such a call is latency, not a unit's throughput: a lone wavefront per SIMD pays
// its LDS and memory round trips in full (one 2K-token request: 0.29 - 0.32 us per 32 x 32 unit at one
// wavefront per SIMD, 0.245 at two; the bare instruction mix takes 0.22 - 0.24).  Hence
//   * everything is fetched by direct loads in an order the waits can count on (Q, K0, K1, then
//     pairs (K of step t + 2, V of step t)), so the first product waits for Q and K0 only, and
//     loads run P - 2 steps ahead of their use (double steps, below, wait for all that the two before
//     requested); a call with at most P steps requests everything up front;
//   * the requests are issued before the sequence length is looked at (late_n), where the launch
//     is so small that no other workgroup hides that read;
//   * the steady part of the loop is unrolled over the ring and free of branches (0.30 us per unit at one
//     wavefront per SIMD against 0.52 for the general step, whose ~100 scalar instructions a lone wavefront pays); with four
//     ring slots two steps share a barrier, but at head_dim 128, which has no registers for it (twelve wavefronts, us: 1500 tokens
//     15.7 -> 15.1, 2 x 950 13.5 -> 13.2, 1900 18.9 -> 18.5);
//   * the ragged last block is a masked step like any other: nothing is staged a second time;
//   * the NK partial (reference, sum, accumulator) states are merged through LDS with the
//     split / merge identity of the online softmax, every wavefront finishing 1/NK of the output
//     columns.
// Measured, fp16, 12 x 64, us per call against the 128-row kernel: 1024 tokens 14.7 -> 10.9, 2000 25.0 -> 21.0, 3072 48.3 -> 43.7; 8 x 128,
// 2048 tokens 39 -> 24.  (As a function of its own, which the kernel below shares, the body of a shape is scheduled otherwise: 64 rows on
// four wavefronts, 1000 tokens, as a kernel -> so, bf16 10.9 -> 11.2, fp16 11.3 -> 11.1.)
// ======================================================================================
template <class T, int D, bool BIAS>
struct SplitWave {
  static constexpr int KS = D / 16, DB = D / 32;
  // head_dim 32 with a bias: the bias is added to finished scores and row sums are unrounded, as in the masked kernel
  // (head_dim 64 / 128: the bias is the C operand, as in the pipelined kernel)
  static constexpr bool BIAS_LAST = BIAS && D == 32, BIAS_FIRST = BIAS && !BIAS_LAST;
  RowState<1, D> st;
  typename T::v8 q[KS];
  uint32_t kfo[KS], vfo[DB];   // per-lane operand offsets (16-bit elements) into a swizzled 32-row block
  // A block sum above this refreshes the row's reference: kPLimit, or -1 while the row has none (its blocks so far held
  // no score above -infinity), so that the first block with a score always sets it.  A register in place of a constant:
  // the test costs what it did without.
  float sum_limit;

  __device__ __forceinline__ void set_limit() { sum_limit = st.m_ref[0] == -INFINITY ? -1.f : kPLimit; }
  __device__ __forceinline__ void init(int lane) {
    init_state(st);
    set_limit();
    const int l32 = lane & 31, hh = lane >> 5, p16 = lane & 15, gg = (lane >> 4) & 1, row = 4 * hh + (p16 >> 2);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kfo[ks] = l32 * D + (((2 * ks + hh) ^ k_swz_d<D>(l32)) * 8);
#pragma unroll
    for (int db = 0; db < DB; ++db)
      vfo[db] = row * D + (((4 * db + 2 * gg + ((p16 & 3) >> 1)) ^ v_swz_d<D>(row)) * 8) + (p16 & 1) * 4;
  }
  __device__ __forceinline__ typename T::v8 k_frag(const uint16_t* kblk, int ks) const {
    return as_v8<T>(*(const uint4*)&kblk[kfo[ks]]);
  }
  __device__ __forceinline__ typename T::v8 vt_frag(const uint16_t* vblk, int ks2, int db) const {
    typedef __attribute__((address_space(3))) shortx4 lds_s4;
    const shortx4 x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)&vblk[vfo[db] + ks2 * 16 * D]);
    const shortx4 x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)&vblk[vfo[db] + (ks2 * 16 + 8) * D]);
    shortx8 x;
    x[0] = x0[0]; x[1] = x0[1]; x[2] = x0[2]; x[3] = x0[3];
    x[4] = x1[0]; x[5] = x1[1]; x[6] = x1[2]; x[7] = x1[3];
    return __builtin_bit_cast(typename T::v8, x);
  }

  // scores of a block on top of `s` (zero, or the block's bias)
  __device__ __forceinline__ void scores(floatx16& s, const uint16_t* kblk, const float* bblk, int lane) {
    const int hh = lane >> 5;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 b4 = BIAS_FIRST ? *(const float4*)&bblk[8 * g + 4 * hh] : make_float4(0.f, 0.f, 0.f, 0.f);
      s[4 * g + 0] = b4.x; s[4 * g + 1] = b4.y; s[4 * g + 2] = b4.z; s[4 * g + 3] = b4.w;
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) s = T::mfma(k_frag(kblk, ks), q[ks], s);
    if (BIAS_LAST) add_bias(s, bblk, hh);
  }
  __device__ __forceinline__ void accumulate(const typename T::v8 (&p)[2], const uint16_t* vblk) {
#pragma unroll
    for (int ks2 = 0; ks2 < 2; ++ks2)
#pragma unroll
      for (int db = 0; db < DB; ++db)
        st.oacc[0][db] = T::mfma(vt_frag(vblk, ks2, db), p[ks2], st.oacc[0][db]);
  }
  // first reference of the rows: the maximum of the wavefront's first block
  __device__ __forceinline__ void prime(const floatx16& s, uint32_t vis, float c) {
    float t0 = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) t0 = fmaxf(t0, keep_or_neg_inf(s[r], vis, r));
    st.m_ref[0] = max_xor32(t0);
    st.mc[0] = st.m_ref[0] == -INFINITY ? 0.f : st.m_ref[0] * c;
    set_limit();
  }
  template <bool MASKED>
  __device__ __forceinline__ void softmax(const floatx16& s, typename T::v8 (&p)[2], uint32_t vis, bool alive, float c) {
    uint32_t pk[8];
    float blk;
    prob_block<T, MASKED, BIAS_LAST>(s, c, st.mc[0], vis, pk, blk);
    const bool trig = alive && !(blk <= sum_limit);   // (also catches a NaN sum)
    if (__any(trig)) {
      const bool row_trig = sum_xor32(trig ? 1.f : 0.f) > 0.f;   // a row refreshes on its own two lanes' evidence only
      float t0 = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) t0 = fmaxf(t0, MASKED ? keep_or_neg_inf(s[r], vis, r) : s[r]);
      rescale_rows(st, 0, row_trig, max_xor32(t0), c);
      set_limit();
      prob_block<T, MASKED, BIAS_LAST>(s, c, st.mc[0], vis, pk, blk);
    }
    st.lsum[0] += blk;
    p[0] = as_v8<T>(make_uint4(pk[0], pk[1], pk[2], pk[3]));
    p[1] = as_v8<T>(make_uint4(pk[4], pk[5], pk[6], pk[7]));
  }
  // The common step, straight-line but for the rare refresh: scores of the next block and P.V of the previous one on
  // the matrix cores, this block's probabilities on the vector ALU.  (Fetching the operands out of LDS a step ahead
  // measured no faster: 0.30 us per unit at one wavefront per SIMD, 0.245 at two, either way.)
  __device__ __forceinline__ void step(const floatx16& s_cur, floatx16& s_nxt, const typename T::v8 (&p_prev)[2],
                                       typename T::v8 (&p_cur)[2], const uint16_t* k_next, const uint16_t* v_prev,
                                       const float* b_next, bool alive, float c, int lane) {
    const int hh = lane >> 5;
    typename T::v8 ka[KS], va[2 * DB];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) ka[ks] = k_frag(k_next, ks);
#pragma unroll
    for (int i = 0; i < 2 * DB; ++i) va[i] = vt_frag(v_prev, i / DB, i % DB);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 b4 = BIAS_FIRST ? *(const float4*)&b_next[8 * g + 4 * hh] : make_float4(0.f, 0.f, 0.f, 0.f);
      s_nxt[4 * g + 0] = b4.x; s_nxt[4 * g + 1] = b4.y; s_nxt[4 * g + 2] = b4.z; s_nxt[4 * g + 3] = b4.w;
    }
    static_assert(KS == 2 * DB, "one score product alternates with one output product");
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      s_nxt = T::mfma(ka[i], q[i], s_nxt);
      st.oacc[0][i % DB] = T::mfma(va[i], p_prev[i / DB], st.oacc[0][i % DB]);
    }
    if (BIAS_LAST) add_bias(s_nxt, b_next, hh);
    softmax<false>(s_cur, p_cur, 0xFFFFu, alive, c);
  }
};

// LDS of the split kernel in 16-bit elements: the Q tile, then P ring slots of [K super tile][V super tile]; after the
// loop the same memory holds the partial results and the output patches.
template <int D, int NQ, int NK, int P>
struct SplitLds {
  static constexpr int kBlk = 32 * D;
  static constexpr int kQ = NQ * kBlk, kSlot = 2 * NK * kBlk;
  static constexpr int kRing = kQ + P * kSlot;
  static constexpr int kPart = NQ * (NK - 1) * 16 * (D / 32) * 64 * 2;   // other wavefronts' accumulator pieces
  static constexpr int kState = NQ * NK * 2 * 64 * 2;                    // reference and row sum of every wavefront
  static constexpr int kMerge = kPart + kState + NQ * epi_patch(D);
  static constexpr int kElems = kRing > kMerge ? kRing : kMerge;
};

// KNOWN_N: tc_in is the workgroup's tile (its q0 is not used) and the length is known; otherwise the body finds its tile.
template <class T, int D, int NQ, int NK, int P, bool BIAS, bool KNOWN_N = false>
__device__ __forceinline__ void split_body(const FaKernelArgs& a, TileCoord tc_in, uint16_t* lds) {
  constexpr int NW = NQ * NK, THREADS = NW * 64, BM = 32 * NQ;
  constexpr int KS = D / 16, DB = D / 32;
  typedef SplitLds<D, NQ, NK, P> L;
  constexpr bool DOUBLES = P == 4 && D != 128;   // two steps between barriers, see below (head_dim 128 has no registers for it)
  constexpr int kBlk = L::kBlk;
  constexpr int CH = D / 8, RPL = 64 / CH, LPB = 32 / RPL;   // 16-byte chunks per row, rows per load, loads per block
  // a block's loads are dealt to NL of the NQ wavefronts that share it, LW each
  constexpr int NL = NQ == 3 ? 2 : NQ, LW = LPB / NL;
  static_assert(LPB % NL == 0 && P >= 2, "whole loads per wavefront");
  float* const lds_bias = (float*)(lds + L::kElems);

  TileCoord tc = tc_in;
  if (KNOWN_N) tc.q0 = tc.qt * BM;
  else if (!locate_tile<BM, false>(a, tc)) return;
  const int N = a.max_len, q0 = tc.q0;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qb = wave % NQ, g = wave / NQ;
  const int l32 = lane & 31, hh = lane >> 5;

  const uint16_t* qp = (const uint16_t*)a.q + tc.b * a.qs[0] + tc.h * a.qs[1];
  const uint16_t* kp = (const uint16_t*)a.k + tc.b * a.ks[0] + tc.h * a.ks[1];
  const uint16_t* vp = (const uint16_t*)a.v + tc.b * a.vs[0] + tc.h * a.vs[1];
  uint16_t* op = (uint16_t*)a.o + tc.b * a.os[0] + tc.h * a.os[1];
  float* lsep = a.lse ? a.lse + ((int64_t)tc.b * a.heads + tc.h) * N : nullptr;

  const bool late_n = !KNOWN_N && a.late_n != 0;
  if (!late_n) tc.n = tc.n < 0 ? 0 : (tc.n > N ? N : tc.n);
  if (!late_n && q0 >= tc.n) {
    zero_fill<BM, D, THREADS>(a, tc, op, lsep);
    return;
  }

  // A load moves RPL rows of a 32-row block (lane: row lane / CH, chunk position lane % CH).  A block whose rows
  // all exist is addressed by a scalar base and a fixed per-lane offset; where rows would leave the tensor the
  // lane's row is clamped to the last one (such rows are masked, zeroed or never read).
  int row_at[LW];
  auto row_of = [&](int x, int lane) { return DOUBLES ? (qb * LW + x) * RPL + lane / CH : row_at[x]; };
  uint32_t koff[LW], voff[LW], kchunk[LW], vchunk[LW];
#pragma unroll
  for (int x = 0; x < LW; ++x) {
    const int r = (qb * LW + x) * RPL + lane / CH;
    row_at[x] = r;
    kchunk[x] = 2u * (uint32_t)(((lane % CH) ^ k_swz_d<D>(r)) * 8);
    vchunk[x] = 2u * (uint32_t)(((lane % CH) ^ v_swz_d<D>(r)) * 8);
    koff[x] = (uint32_t)r * 2u * (uint32_t)a.ks[2] + kchunk[x];
    voff[x] = (uint32_t)r * 2u * (uint32_t)a.vs[2] + vchunk[x];
  }
  auto load_block = [&](const uint16_t* base, int64_t rs, const uint32_t (&off)[LW], const uint32_t (&chunk)[LW], int j, uint16_t* dst) {
    if (NL < NQ && qb >= NL) return;
    if (32 * j + 32 <= N) {
      const uint16_t* gb = base + (int64_t)(32 * j) * rs;
#pragma unroll
      for (int x = 0; x < LW; ++x) load16_to_lds(gb, off[x], dst + (qb * LW + x) * RPL * D);
    } else {
      const int first = 32 * j < N ? 32 * j : N - 1;
      const uint16_t* gb = base + (int64_t)first * rs;
      const int at = DOUBLES ? lane_now() : lane;   // (no register through the loop)
#pragma unroll
      for (int x = 0; x < LW; ++x) {
        if (DOUBLES) {
          const int past = row_of(x, at) - (N - 1 - first);
          load16_to_lds(gb, off[x] - 2u * (uint32_t)(past > 0 ? past : 0) * (uint32_t)rs, dst + (qb * LW + x) * RPL * D);
        } else {
          const int r = row_at[x] < N - 1 - first ? row_at[x] : N - 1 - first;
          load16_to_lds(gb, (uint32_t)r * 2u * (uint32_t)rs + chunk[x], dst + (qb * LW + x) * RPL * D);
        }
      }
    }
  };
  uint16_t* const ring = lds + L::kQ;
  auto k_slot = [&](int i) { return ring + (i % P) * L::kSlot + g * kBlk; };
  auto v_slot = [&](int i) { return ring + (i % P) * L::kSlot + (NK + g) * kBlk; };
  auto load_k = [&](int i) { load_block(kp, a.ks[2], koff, kchunk, i * NK + g, k_slot(i)); };
  auto load_v = [&](int i) { load_block(vp, a.vs[2], voff, vchunk, i * NK + g, v_slot(i)); };
  auto load_pair = [&](int t, int steps) {   // K of step t + 2, V of step t
    if (t + 2 < steps) load_k(t + 2);
    load_v(t);
  };

  // Requests of the start, from the tensor length (late_n) or the sequence length.
  const int steps_req = ((late_n ? N : tc.n) + 32 * NK - 1) / (32 * NK);
  // Q: the block's loads are dealt to its NK wavefronts; swizzled like a K block
#pragma unroll
  for (int x = 0; x < (LPB + NK - 1) / NK; ++x) {
    const int part = x * NK + g;
    if (LPB % NK == 0 || part < LPB) {
      const int r = part * RPL + lane / CH;
      const int first = q0 + 32 * qb < N ? q0 + 32 * qb : N - 1;
      const int rr = r < N - 1 - first ? r : N - 1 - first;
      load16_to_lds(qp + (int64_t)first * a.qs[2],
                    (uint32_t)rr * 2u * (uint32_t)a.qs[2] + 2u * (uint32_t)(((lane % CH) ^ k_swz_d<D>(r)) * 8),
                    lds + qb * kBlk + part * RPL * D);
    }
  }
  load_k(0);
  if (steps_req > 1) load_k(1);
  int pairs = steps_req <= P ? steps_req : P - 2;   // pairs requested so far
  for (int t = 0; t < pairs; ++t) load_pair(t, steps_req);
  if (BIAS) {
    const uint16_t* bp = (const uint16_t*)a.key_bias + tc.b * a.kb_stride;
    for (int j = tid; j < ((N + 31) & ~31); j += THREADS) lds_bias[j] = bias_over_scale<T, D == 32>(a, bp[j < N ? j : N - 1]);
  }

  // only now the sequence length
  const int n = tc.n < 0 ? 0 : (tc.n > N ? N : tc.n);
  tc.n = n;
  if (q0 >= n) {
    wait_direct_loads();  // the loads write this workgroup's LDS: they must land before it ends
    zero_fill<BM, D, THREADS>(a, tc, op, lsep);
    return;
  }
  const int nb = (n + 31) >> 5;
  const int steps = (nb + NK - 1) / NK;                   // <= steps_req
  const int nfs = n / (32 * NK);                          // steps whose super tile is full: steps or steps - 1
  const bool wave_has_rows = q0 + 32 * qb < n;
  const int ig = q0 + 32 * qb + l32;
  const bool alive = ig < n;
  const float c = a.c;

  // Loads land in order.  Step i needs Q, K0, K1 and the pairs below i; of the pairs requested after them every
  // one holds at least V's LW loads, and K's LW too while K of its step t + 2 exists.
  auto wait_pairs_below = [&](int i) {
    const int later = pairs - i;             // requested pairs that may still be under way
    if (P > 2 && later == P - 2 && pairs + 1 < steps) wait_vmcnt<(P > 2 ? (P - 2) * 2 * LW : 0)>();
    else if (later >= 3) wait_vmcnt<3 * LW>();
    else if (later == 2) wait_vmcnt<2 * LW>();
    else if (later == 1) wait_vmcnt<LW>();
    else wait_vmcnt<0>();
  };
  auto request_up_to = [&](int t) {
    while (pairs < steps && pairs <= t) {
      load_pair(pairs, steps);
      ++pairs;
    }
  };
  // every wavefront of the workgroup is past its reads of a ring slot (a wavefront that shares its blocks with nobody
  // needs no barrier: its own reads are waited for)
  auto slots_free = [&] {
    if (NQ > 1) __syncthreads();
    else __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
  };

  SplitWave<T, D, BIAS> w;
  w.init(lane);
  floatx16 sA, sB;
  typename T::v8 pA[2], pB[2];
  pA[0] = pA[1] = pB[0] = pB[1] = as_v8<T>(make_uint4(0, 0, 0, 0));
  // V rows at or beyond n are overwritten with zeros by the lanes that fetched them, once the partial super tile has
  // landed: 0 * whatever is stored in the padding must be 0
  auto scrub = [&](int i) {
    const int lane = DOUBLES ? lane_now() : tid & 63;
#pragma unroll
    for (int x = 0; x < LW; ++x)
      if ((NL == NQ || qb < NL) && 32 * (i * NK + g) + row_of(x, lane) >= n)
        *(uint4*)&v_slot(i)[row_of(x, lane) * D + (lane % CH) * 8] = make_uint4(0, 0, 0, 0);
  };
  if (nfs == 0) {
    request_up_to(0);   // (two slots and a tensor longer than this sequence: V0 has not been requested yet)
    wait_vmcnt<0>();
    scrub(0);
  } else if (NL < NQ && qb >= NL) {
    wait_vmcnt<0>();       // a wavefront that moves no K or V: its part of Q is all it has under way
  } else {
    wait_pairs_below(0);
  }
  __syncthreads();
  auto bias_of_block = [&](int i) { return &lds_bias[BIAS ? 32 * (i * NK + g) : 0]; };
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    uint4 u = __builtin_bit_cast(uint4, w.k_frag(lds + qb * kBlk, ks));
    if (a.negate_q) {
      u.x ^= 0x80008000u; u.y ^= 0x80008000u; u.z ^= 0x80008000u; u.w ^= 0x80008000u;
    }
    w.q[ks] = as_v8<T>(u);
  }
  w.scores(sA, k_slot(0), bias_of_block(0), lane);
  w.prime(sA, nfs > 0 ? 0xFFFFu : visible_bits(32 * g, hh, 0, n - 1), c);

  // Step 0 (if its super tile is full): probabilities of block 0, scores of block 1.  (Double steps, below, make their own requests.)
  const bool doubles = DOUBLES && nfs > 5 && pairs == 2;
  if (nfs > 0) {
    if (!doubles) {
      if (steps > P) slots_free();   // K0's slot is refilled
      request_up_to(P - 2);
    }
    if (wave_has_rows) {
      const int in = steps > 1 ? 1 : 0;
      w.scores(sB, k_slot(in), bias_of_block(in), lane);
      w.template softmax<false>(sA, pA, 0xFFFFu, alive, c);
    }
  }
  // Step i (a full super tile): probabilities of block i, scores of block i + 1, P.V of block i - 1.
  int i = 1;
  {
    // The steady part, straight-line code: ring slots are compile-time constants, the row bases of the requested blocks just
    // advance, and the wait is one instruction.
    if constexpr (DOUBLES) {
      // Two steps between barriers: steps i and i + 1 request K of steps i + 3, i + 4 and V of i + 1, i + 2, into slots that
      // the two steps before left, and wait for nothing younger than those before requested.  (The requested K lie inside the full
      // super tiles.)
      if (doubles) {
        const int64_t kstep = (int64_t)(32 * NK) * a.ks[2], vstep = (int64_t)(32 * NK) * a.vs[2];
        const uint16_t* kg = kp + (int64_t)(32 * g) * a.ks[2] + 4 * kstep;
        const uint16_t* vg = vp + (int64_t)(32 * g) * a.vs[2] + 2 * vstep;
        uint16_t* const my_k = ring + g * kBlk;
        uint16_t* const my_v = ring + (NK + g) * kBlk;
        auto two = [&](auto Jc, int i) {
          constexpr int J = decltype(Jc)::value;   // i % 4: 1 or 3
          wait_vmcnt<0>();
          slots_free();
          if (NL == NQ || qb < NL) {
#pragma unroll
            for (int y = 0; y < 2; ++y) {
#pragma unroll
              for (int x = 0; x < LW; ++x) load16_to_lds(kg + y * kstep, koff[x], my_k + (J + 3 + y) % 4 * L::kSlot + (qb * LW + x) * RPL * D);
#pragma unroll
              for (int x = 0; x < LW; ++x) load16_to_lds(vg + y * vstep, voff[x], my_v + (J + 1 + y) % 4 * L::kSlot + (qb * LW + x) * RPL * D);
            }
          }
          kg += 2 * kstep;
          vg += 2 * vstep;
          if (wave_has_rows) {
            w.step(sB, sA, pA, pB, my_k + (J + 1) % 4 * L::kSlot, my_v + (J + 3) % 4 * L::kSlot, bias_of_block(i + 1), alive, c, lane);
            __builtin_amdgcn_sched_barrier(0);
            w.step(sA, sB, pB, pA, my_k + (J + 2) % 4 * L::kSlot, my_v + J * L::kSlot, bias_of_block(i + 2), alive, c, lane);
          }
        };
        for (; i + 6 < nfs; i += 4) {
          two(std::integral_constant<int, 1>{}, i);
          two(std::integral_constant<int, 3>{}, i + 2);
        }
        if (i + 4 < nfs) {
          two(std::integral_constant<int, 1>{}, i);
          i += 2;
        }
        pairs = i + 1;
      }
    }
    // P steps per turn, a barrier each.  Step i requests pair i + P - 2, whose K of step i + P lies inside the full super tiles.
    if ((P == 2 || P == 4) && !DOUBLES && i + 2 * P - 1 < nfs && pairs == P - 1) {
      const int64_t kstep = (int64_t)(32 * NK) * a.ks[2], vstep = (int64_t)(32 * NK) * a.vs[2];
      const uint16_t* kg = kp + (int64_t)(32 * g) * a.ks[2] + (P + 1) * kstep;
      const uint16_t* vg = vp + (int64_t)(32 * g) * a.vs[2] + (P - 1) * vstep;
      uint16_t* const my_k = ring + g * kBlk;
      uint16_t* const my_v = ring + (NK + g) * kBlk;
      auto steady = [&](auto Jc, floatx16& s_cur, floatx16& s_nxt, typename T::v8 (&p_prev)[2], typename T::v8 (&p_cur)[2], int i) {
        constexpr int J = decltype(Jc)::value;   // i % P
        wait_vmcnt<(P > 2 ? (P - 2) * 2 * LW : 0)>();
        slots_free();
        if (NL == NQ || qb < NL) {
#pragma unroll
          for (int x = 0; x < LW; ++x) load16_to_lds(kg, koff[x], my_k + J * L::kSlot + (qb * LW + x) * RPL * D);
#pragma unroll
          for (int x = 0; x < LW; ++x) load16_to_lds(vg, voff[x], my_v + (J + P - 2) % P * L::kSlot + (qb * LW + x) * RPL * D);
        }
        kg += kstep;
        vg += vstep;
        if (wave_has_rows)
          w.step(s_cur, s_nxt, p_prev, p_cur, my_k + (J + 1) % P * L::kSlot, my_v + (J + P - 1) % P * L::kSlot,
                 bias_of_block(i + 1), alive, c, lane);
      };
      for (; i + 2 * P - 1 < nfs; i += P) {
        steady(std::integral_constant<int, 1>{}, sB, sA, pA, pB, i);
        steady(std::integral_constant<int, 2 % P>{}, sA, sB, pB, pA, i + 1);
        if (P == 4) {
          steady(std::integral_constant<int, 3 % P>{}, sB, sA, pA, pB, i + 2);
          steady(std::integral_constant<int, 0>{}, sA, sB, pB, pA, i + 3);
        }
      }
      pairs = i + P - 2;
    }
  }
  auto step = [&](floatx16& s_cur, floatx16& s_nxt, typename T::v8 (&p_prev)[2], typename T::v8 (&p_cur)[2], int i) {
    wait_pairs_below(i);
    slots_free();
    request_up_to(i + P - 2);   // their slots were last read in step i - 1
    const int in = i + 1 < steps ? i + 1 : i;   // (the last block's successor: its scores are not used)
    if (wave_has_rows)
      w.step(s_cur, s_nxt, p_prev, p_cur, k_slot(in), v_slot(i - 1), bias_of_block(in), alive, c, lane);
  };
  for (; i + 1 < nfs; i += 2) {
    step(sB, sA, pA, pB, i);
    step(sA, sB, pB, pA, i + 1);
  }
  if (i < nfs) {
    step(sB, sA, pA, pB, i);
    pA[0] = pB[0];
    pA[1] = pB[1];
  } else if (nfs > 0) {
    sA = sB;
  }
  // (DOUBLES: the lane is formed again, no register through the loop)
  const int lane_e = DOUBLES ? lane_now() : lane, l32_e = lane_e & 31, hh_e = lane_e >> 5, ig_e = q0 + 32 * qb + l32_e;
  // Now sA holds the scores of the partial super tile (if there is one) and pA the last full block's probabilities.
  if (nfs > 0 || steps > nfs) {
    if (nfs > 0) {
      if (steps > nfs && P == 2) {   // (with more slots the last pair has been requested by now)
        slots_free();
        request_up_to(nfs);
      }
      wait_vmcnt<0>();
      if (steps > nfs) scrub(nfs);
      if (NQ > 1) __syncthreads();
      w.accumulate(pA, v_slot(nfs - 1));
    }
    // (a block that lies past the end as a whole has no part in the result; its row without a reference would only take the
    // detour for one)
    if (32 * (nfs * NK + g) < n) {
      w.template softmax<true>(sA, pA, visible_bits(32 * (nfs * NK + g), hh_e, 0, n - 1), alive, c);
      w.accumulate(pA, v_slot(nfs));
    }
  }
  wait_direct_loads();   // requests beyond the sequence's last step may still be landing in the ring
  __syncthreads();       // the ring becomes the merge memory

  // ---- merge the NK partial results of each query block: the accumulator's groups of four registers (four output
  // columns of a row; the same lane <-> (row, column) mapping in every wavefront) are dealt to the NK wavefronts,
  // group x to wavefront x % NK, which finishes it
  constexpr int G = 4 * DB;
  float4* const part = (float4*)lds + (size_t)qb * (NK - 1) * G * 64 + lane_e;       // [group][contributor][lane]
  // [wavefront][reference times c, sum][lane].  The reference goes through as the rounded product the probabilities were
  // formed against (-infinity: none); forming it again here would let the compiler fuse it into the subtraction below,
  // unrounded, and put a wavefront's share off by 2^(half a spacing of it) - 4 % at scores of 10^6
  float* const state = (float*)(lds + L::kPart) + (size_t)qb * NK * 2 * 64 + lane_e;
  uint16_t* const patch = lds + L::kPart + L::kState + qb * epi_patch(D);
  constexpr int kEpiStride = epi_stride(D);
  state[(2 * g + 0) * 64] = w.st.m_ref[0] == -INFINITY ? -INFINITY : w.st.mc[0];
  state[(2 * g + 1) * 64] = w.st.lsum[0];
#pragma unroll
  for (int x = 0; x < G; ++x) {
    if (x % NK != g) {   // (wavefront-uniform)
      const int r = 4 * (x % 4);
      part[(x * (NK - 1) + (g < x % NK ? g : g - 1)) * 64] =
          make_float4(w.st.oacc[0][x / 4][r], w.st.oacc[0][x / 4][r + 1], w.st.oacc[0][x / 4][r + 2], w.st.oacc[0][x / 4][r + 3]);
    }
  }
  __syncthreads();
  float mk[NK], mc_new = -INFINITY, fk[NK], ltot = 0.f;
#pragma unroll
  for (int x = 0; x < NK; ++x) {
    mk[x] = state[(2 * x + 0) * 64];
    mc_new = fmaxf(mc_new, mk[x]);
  }
  if (mc_new == -INFINITY) mc_new = 0.f;
#pragma unroll
  for (int x = 0; x < NK; ++x) {
    // a wavefront that saw no key has nothing accumulated (the first score sets a reference): factor 0, kept away from
    // exp2(+inf)
    fk[x] = mk[x] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mk[x] - mc_new);
    ltot = __builtin_fmaf(fk[x], state[(2 * x + 1) * 64], ltot);
  }
  ltot = sum_xor32(ltot);
  const bool live = alive && ltot > 0.f;
  const float inv = live ? 1.0f / ltot : 0.f;
#pragma unroll
  for (int x = 0; x < G; ++x) {
    if (x % NK == g) {
      const int r = 4 * (x % 4);
      const float f = fk[x % NK];
      float4 v = make_float4(w.st.oacc[0][x / 4][r] * f, w.st.oacc[0][x / 4][r + 1] * f, w.st.oacc[0][x / 4][r + 2] * f,
                             w.st.oacc[0][x / 4][r + 3] * f);
#pragma unroll
      for (int y = 0; y < NK; ++y) {
        if (y == x % NK) continue;
        const float4 u = part[(x * (NK - 1) + (y < x % NK ? y : y - 1)) * 64];
        v.x = __builtin_fmaf(fk[y], u.x, v.x);
        v.y = __builtin_fmaf(fk[y], u.y, v.y);
        v.z = __builtin_fmaf(fk[y], u.z, v.z);
        v.w = __builtin_fmaf(fk[y], u.w, v.w);
      }
      // columns 32 (x / 4) + 8 (x % 4) + 4 hh .. + 3 of the lane's row
      *(uint2*)&patch[l32_e * kEpiStride + 8 * x + 4 * hh_e] =
          live ? make_uint2(T::pack2(v.x * inv, v.y * inv), T::pack2(v.z * inv, v.w * inv)) : make_uint2(0, 0);
    }
  }
  __syncthreads();
  for (int pass = g; pass < 32 / RPL; pass += NK) {
    const int r = pass * RPL + lane_e / CH;
    const int row = q0 + 32 * qb + r;
    const uint4 v = *(const uint4*)&patch[r * kEpiStride + (lane_e % CH) * 8];
    if (row < N) *(uint4*)(op + row * a.os[2] + (lane_e % CH) * 8) = v;
  }
  if (lsep && g == 0 && hh_e == 0 && ig_e < N) lsep[ig_e] = live ? (mc_new + __builtin_amdgcn_logf(ltot)) * kLn2 : -INFINITY;
}

template <class T, int D, int NQ, int NK, int P, int WPS, bool BIAS>
__global__ __launch_bounds__(NQ * NK * 64, WPS) void fa_fwd_split_kernel(const FaKernelArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[SplitLds<D, NQ, NK, P>::kElems + (BIAS ? 2 * kSplitBiasKeys : 0)];
  split_body<T, D, NQ, NK, P, BIAS>(a, TileCoord(), lds);
}

// The same for ONE sequence in a tensor that is longer (head_dim 64): the tile's rows and the key split follow the sequence's
// length, which the host does not know.  A workgroup has twelve wavefronts and a compute unit to itself; every head has
// a.n_qtiles of them (heads * n_qtiles <= 256), and they are 64, 96 or 128 rows high, as few as hold the sequence.  (The host has
// to lay out tiles for the whole tensor, whose dead ones delay live ones: 1904 of 2048 tokens, 12 heads, bf16 20.9 -> 18.1 us.)
// Rows past what the tiles cover are padding: zeros.
template <class T>
__global__ __launch_bounds__(768, 3) void fa_fwd_split_live_kernel(const FaKernelArgs a) {
  typedef SplitLds<64, 3, 4, 4> L;
  static_assert(L::kElems >= SplitLds<64, 4, 3, 2>::kElems && L::kElems >= SplitLds<64, 2, 6, 2>::kElems, "one memory for the three shapes");
  __shared__ __attribute__((aligned(16))) uint16_t lds[L::kElems];
  // (by hand: one sequence, so that nothing comes between the arguments and its length, which every load waits for; with
  // locate_tile 0.3 - 0.5 us more: 2048 of 2048 fp16 22.3 -> 21.5 us, 1904 bf16 19.2 -> 18.7)
  const int id = blockIdx.x, t = a.map_xcd ? (id & 7) * a.xcd_per + (id >> 3) : id;
  if (t >= a.total_tiles) return;
  TileCoord tc;
  tc.b = 0;
  tc.h = t / a.n_qtiles;
  tc.qt = t - tc.h * a.n_qtiles;
  tc.n = a.seq_lens[0];
  tc.n = tc.n < 0 ? 0 : (tc.n > a.max_len ? a.max_len : tc.n);
  const int per = a.n_qtiles, rows = tc.n <= 64 * per ? 64 : (tc.n <= 96 * per ? 96 : 128);
  // rows past what the tiles cover: padding, by the workgroups of the last tiles, which often are padding themselves
  for (tc.q0 = per * rows + 32 * (per - 1 - tc.qt); tc.q0 < a.max_len; tc.q0 += 32 * per)
    zero_fill<32, 64, 768>(a, tc, (uint16_t*)a.o + tc.h * a.os[1], a.lse ? a.lse + (int64_t)tc.h * a.max_len : nullptr);
  // (each shape reads the arguments for itself: those of all three together do not fit the scalar registers)
  auto own_args = [&]() -> const FaKernelArgs& {
    typedef const __attribute__((address_space(4))) FaKernelArgs Args;
    Args* p = (Args*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p), "+s"(tc.h), "+s"(tc.qt), "+s"(tc.n));
    return *(const FaKernelArgs*)p;
  };
  tc.h = __builtin_amdgcn_readfirstlane(tc.h);
  tc.qt = __builtin_amdgcn_readfirstlane(tc.qt);
  tc.n = __builtin_amdgcn_readfirstlane(tc.n);
  if (rows == 96) split_body<T, 64, 3, 4, 4, false, true>(own_args(), tc, lds);
  else if (rows == 128) split_body<T, 64, 4, 3, 2, false, true>(own_args(), tc, lds);
  else split_body<T, 64, 2, 6, 2, false, true>(own_args(), tc, lds);
}

// ======================================================================================
// Small kernel: the smallest calls, local and global, where 32-row workgroups whose wavefronts hold all their key blocks at
// once fit the chip.  Wavefront g of NK has the blocks g, g + NK, .. of those that the workgroup's 32 rows can see, NB at
// most: their scores, an ordinary softmax over them, their P.V; the partial results meet in LDS.  (The paper's 63/64 window:
// five wavefronts, one block each.)
// Bound: latency, the chain launch - arguments - loads - blocks - merge - store.  So everything is requested at once by direct
// loads, the sequence length is looked at after that, there is no running reference, and a lane stores its eight bytes of a
// row as they are: the detour through a patch for whole rows costs a barrier and a trip through LDS.  (A copy of Q per
// wavefront instead of one behind a barrier is no faster, and its LDS halves the calls that fit a round.)  12 x 64, us on the GPU alone
// (in a graph; the host takes 5 for a call): local 487 tokens 6.6 on the resident kernel -> 4.5, global 512 6.3 on
// the split kernel -> 5.5 (one block on each of sixteen wavefronts: 6.4, twice the partial results).
// ======================================================================================
template <class T, int D, int NK, int NB, bool BIAS>
__global__ __launch_bounds__(NK * 64, 1) void fa_fwd_small_kernel(const FaKernelArgs a) {
  constexpr int THREADS = NK * 64, BM = 32;
  constexpr int KS = D / 16, DB = D / 32, kBlk = 32 * D;
  constexpr int CH = D / 8, RPL = 64 / CH, LPB = 32 / RPL;   // 16-byte chunks per row, rows per load, loads per block
  constexpr bool BIAS_LAST = BIAS && D != 64;                // as in the two-phase kernel
  // the Q block, then per wavefront its K and V blocks, which become its accumulator, [4 x column block + quad][lane] float4
  constexpr int kWave = 2 * NB * kBlk;
  static_assert(kWave * 2 >= 4 * DB * 64 * 16, "an accumulator takes the place of K and V");
  __shared__ __attribute__((aligned(16))) uint16_t lds[kBlk + NK * kWave];
  __shared__ __attribute__((aligned(16))) float lds_state[NK][2][64];   // reference times c, row sum
  __shared__ __attribute__((aligned(16))) float lds_bias[BIAS ? NK * NB : 1][32];

  fetch_args();
  TileCoord tc;
  if (!locate_tile<BM, false>(a, tc)) return;   // tc.n still as loaded: see below
  const int N = a.max_len, q0 = tc.q0;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int g = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;

  const uint16_t* qp = (const uint16_t*)a.q + tc.b * a.qs[0] + tc.h * a.qs[1];
  const uint16_t* kp = (const uint16_t*)a.k + tc.b * a.ks[0] + tc.h * a.ks[1];
  const uint16_t* vp = (const uint16_t*)a.v + tc.b * a.vs[0] + tc.h * a.vs[1];
  uint16_t* op = (uint16_t*)a.o + tc.b * a.os[0] + tc.h * a.os[1];
  float* lsep = a.lse ? a.lse + ((int64_t)tc.b * a.heads + tc.h) * N : nullptr;

  // a side without a limit reaches past the tensor
  const int wl = a.wl < 0 ? N : a.wl, wr = a.wr < 0 ? N : a.wr;
  const int key0 = 32 * ((q0 - wl > 0 ? (q0 - wl) >> 5 : 0) + g);   // the wavefront's first block; the next NK blocks on
  auto first_key = [&](int i) { return key0 + 32 * NK * i; };
  // loads of x = 0 .. LPB - 1 of the 32 rows from `first` on; rows past the tensor are its last one again (masked, zeroed or
  // never stored)
  auto load_part = [&](const uint16_t* base, int64_t rs, int first, bool is_v, int x, uint16_t* dst) {
    const int r = RPL * x + lane / CH, rc = r < N - 1 - first ? r : N - 1 - first;
    const int swz = is_v ? v_swz_d<D>(r) : k_swz_d<D>(r);
    load16_to_lds(base + (int64_t)first * rs, 2u * ((uint32_t)rc * (uint32_t)rs + (uint32_t)(((lane % CH) ^ swz) * 8)), dst + RPL * x * D);
  };
  uint16_t *const kl = lds + kBlk + g * kWave, *const vl = kl + NB * kBlk;
#pragma unroll
  for (int x = 0; x < (LPB + NK - 1) / NK; ++x)
    if (x * NK + g < LPB) load_part(qp, a.qs[2], q0, false, x * NK + g, lds);
  int there = 0;   // blocks that the tensor has
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    if (first_key(i) < N && first_key(i) <= q0 + BM - 1 + wr) {
      there = i + 1;
#pragma unroll
      for (int x = 0; x < LPB; ++x) load_part(kp, a.ks[2], first_key(i), false, x, kl + i * kBlk);
    }
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    if (i < there) {
#pragma unroll
      for (int x = 0; x < LPB; ++x) load_part(vp, a.vs[2], first_key(i), true, x, vl + i * kBlk);
    }
  }
  float bias[NB];   // of key first_key(i) + lane, lanes 0 .. 31
  if (BIAS) {
    const uint16_t* bp = (const uint16_t*)a.key_bias + tc.b * a.kb_stride;
#pragma unroll
    for (int i = 0; i < NB; ++i) bias[i] = bias_over_scale<T, BIAS_LAST>(a, bp[first_key(i) + l32 < N ? first_key(i) + l32 : N - 1]);
  }

  // only now the sequence length
  const int n = tc.n < 0 ? 0 : (tc.n > N ? N : tc.n);
  tc.n = n;
  if (q0 >= n) {
    wait_direct_loads();  // the loads write this workgroup's LDS: they must land before it ends
    zero_fill<BM, D, THREADS>(a, tc, op, lsep);
    return;
  }
  const int ig = q0 + l32, q_last = (q0 + BM < n ? q0 + BM : n) - 1;
  const bool alive = ig < n;
  const float c = a.c;
  if (BIAS) {
#pragma unroll
    for (int i = 0; i < NB; ++i) lds_bias[g * NB + i][l32] = bias[i];
  }
  // Q and K have landed
  if (NB == 2 && there == 2) wait_vmcnt<2 * LPB>();
  else if (there == 1) wait_vmcnt<LPB>();
  else wait_direct_loads();
  __syncthreads();
  int cnt = 0;   // blocks with keys that the rows see
#pragma unroll
  for (int i = 0; i < NB; ++i)
    if (first_key(i) < n && first_key(i) <= q_last + wr) cnt = i + 1;
  RowState<1, D> st;
  init_state(st);
  if (cnt > 0) {
    typename T::v8 q[KS];
    const uint32_t flip = a.negate_q ? 0x80008000u : 0u;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint4 u = __builtin_bit_cast(uint4, load_k_frag_swz_d<T, D>(lds, l32, hh, ks));
      u.x ^= flip; u.y ^= flip; u.z ^= flip; u.w ^= flip;
      q[ks] = as_v8<T>(u);
    }
    floatx16 s[NB];   // set and used for i < cnt only
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if (i >= cnt) continue;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const float4 b4 = BIAS && !BIAS_LAST ? *(const float4*)&lds_bias[g * NB + i][8 * x + 4 * hh] : make_float4(0.f, 0.f, 0.f, 0.f);
        s[i][4 * x + 0] = b4.x; s[i][4 * x + 1] = b4.y; s[i][4 * x + 2] = b4.z; s[i][4 * x + 3] = b4.w;
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) s[i] = T::mfma(load_k_frag_swz_d<T, D>(kl + i * kBlk, l32, hh, ks), q[ks], s[i]);
      if (BIAS_LAST) add_bias(s[i], lds_bias[g * NB + i], hh);
    }
    // softmax over the blocks: their maximum is the reference
    uint32_t vis[NB];
    float t0 = -INFINITY;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if (i >= cnt) continue;
      const int kb0 = first_key(i);
      if (kb0 + 32 <= n && kb0 >= q_last - wl && kb0 + 31 <= q0 + wr) {   // all rows see all keys
        vis[i] = 0xFFFFu;
#pragma unroll
        for (int r = 0; r < 16; ++r) t0 = fmaxf(t0, s[i][r]);
      } else {
        vis[i] = visible_bits(kb0, hh, ig - wl > 0 ? ig - wl : 0, ig + wr < n - 1 ? ig + wr : n - 1);
#pragma unroll
        for (int r = 0; r < 16; ++r) t0 = fmaxf(t0, keep_or_neg_inf(s[i][r], vis[i], r));
      }
    }
    const float tmax = max_xor32(t0);
    st.m_ref[0] = tmax;
    st.mc[0] = tmax == -INFINITY ? 0.f : tmax * c;   // a row without a visible key here: every p is masked to 0
    typename T::v8 p[NB][2];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if (i >= cnt) continue;
      const int kb0 = first_key(i);
      uint32_t pk[8];
      float blk;
      if (kb0 + 32 <= n && kb0 >= q_last - wl && kb0 + 31 <= q0 + wr) prob_block<T, false, BIAS_LAST>(s[i], c, st.mc[0], vis[i], pk, blk);
      else prob_block<T, true, BIAS_LAST>(s[i], c, st.mc[0], vis[i], pk, blk);
      st.lsum[0] += blk;
      p[i][0] = as_v8<T>(make_uint4(pk[0], pk[1], pk[2], pk[3]));
      p[i][1] = as_v8<T>(make_uint4(pk[4], pk[5], pk[6], pk[7]));
    }
    wait_direct_loads();   // V; its rows at or beyond n are overwritten with zeros (0 * whatever is stored there must be 0)
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if (i >= cnt) continue;
      if (first_key(i) + 32 > n) {
#pragma unroll
        for (int x = 0; x < LPB; ++x) {
          const int r = RPL * x + lane / CH;
          if (first_key(i) + r >= n) *(uint4*)&vl[i * kBlk + r * D + (lane % CH) * 8] = make_uint4(0, 0, 0, 0);
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // (other lanes' writes: order for the compiler, no instruction)
#pragma unroll
      for (int ks2 = 0; ks2 < 2; ++ks2)
#pragma unroll
        for (int db = 0; db < DB; ++db)
          st.oacc[0][db] = T::mfma(load_vt_frag_swz_d<T, D>(vl + i * kBlk, lane, ks2, db), p[i][ks2], st.oacc[0][db]);
    }
  } else {
    wait_direct_loads();   // (before their place is taken)
  }

  // ---- merge: groups of four output columns of a row, dealt round-robin to the wavefronts
  constexpr int G = 4 * DB;
  float4* const part = (float4*)kl + lane;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
  for (int x = 0; x < G; ++x) {
    const int r = 4 * (x % 4);
    part[x * 64] = make_float4(st.oacc[0][x / 4][r], st.oacc[0][x / 4][r + 1], st.oacc[0][x / 4][r + 2], st.oacc[0][x / 4][r + 3]);
  }
  // (the reference goes through as the rounded product the probabilities were formed against; -infinity: none)
  lds_state[g][0][lane] = st.m_ref[0] == -INFINITY ? -INFINITY : st.mc[0];
  lds_state[g][1][lane] = st.lsum[0];
  __syncthreads();
  float mk[NK], fk[NK], mc_new = -INFINITY, ltot = 0.f;
#pragma unroll
  for (int x = 0; x < NK; ++x) {
    mk[x] = lds_state[x][0][lane];
    mc_new = fmaxf(mc_new, mk[x]);
  }
  if (mc_new == -INFINITY) mc_new = 0.f;
#pragma unroll
  for (int x = 0; x < NK; ++x) {
    // a wavefront that saw no key has nothing accumulated: factor 0, kept away from exp2(+inf)
    fk[x] = mk[x] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mk[x] - mc_new);
    ltot = __builtin_fmaf(fk[x], lds_state[x][1][lane], ltot);
  }
  ltot = sum_xor32(ltot);
  const bool live = alive && ltot > 0.f;
  const float inv = live ? 1.0f / ltot : 0.f;
  for (int x = g; x < G; x += NK) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int y = 0; y < NK; ++y) {
      const float4 u = ((const float4*)(lds + kBlk + y * kWave))[x * 64 + lane];
      v.x = __builtin_fmaf(fk[y], u.x, v.x);
      v.y = __builtin_fmaf(fk[y], u.y, v.y);
      v.z = __builtin_fmaf(fk[y], u.z, v.z);
      v.w = __builtin_fmaf(fk[y], u.w, v.w);
    }
    if (ig < N)   // columns 8 x + 4 hh .. + 3
      *(uint2*)(op + ig * a.os[2] + 8 * x + 4 * hh) =
          live ? make_uint2(T::pack2(v.x * inv, v.y * inv), T::pack2(v.z * inv, v.w * inv)) : make_uint2(0, 0);
  }
  if (lsep && g == 0 && hh == 0 && ig < N) lsep[ig] = live ? (mc_new + __builtin_amdgcn_logf(ltot)) * kLn2 : -INFINITY;
}

// ======================================================================================
// Global kernel: a software pipeline over 64-key tiles
//
// A workgroup is NW wavefronts (4; 8 and 12 exist for head_dim 64, 8 for 128) that share one pair of rings of 32-key blocks,
// eight of K (head_dim 128: four) and four of V, filled by direct loads one tile ahead; each wavefront owns NQB blocks of 32
// query rows.
// Large calls are bound by the power limit (the clock sits at 1.8 - 2.2 of 2.4 GHz) and by issue slots together, so what
// counts is how many instructions a unit of 32 keys x 32 queries takes and what they draw:
//   * ONE test per 64-key tile decides whether the running references still hold, of row sums formed an iteration ago.
//     (A test per unit waits for the unit's sum, cuts the straight-line code and cost 3 - 9 % of the bare instruction
//     mix.)  It has to come before the tile's P.V is accumulated, so the P.V lags a whole tile behind the probabilities,
//     which wait in registers; when it trips, the tile's scores are formed again from K in LDS (head_dim 128: in global
//     memory).  Rows with peaked probabilities trip often: 8K 12 x 64 fp16, q and k of 3 N(0, 1) 232 us, of 6 N(0, 1) 258,
//     scores that rise by 100 along the keys 330 (306, 412 and 618 with K from global memory); head_dim 128 313, 391, 571;
//   * fp16 row sums, of the rounded probabilities, go to the matrix cores where the smaller shape runs (two products with a
//     constant operand instead of eight dot products and an addition), bf16 sums the unrounded fp32 ones, 16 additions;
//   * the shape of the matrix instruction per type and head size: GlobalTile;
//   * the ragged last tile is a masked iteration of the same pipeline on rows clamped into the tensor, not a second staging
//     pass through registers (a 128-row workgroup of a 512-token sequence spent 2.5 of its 12 us there).
// Measured, us, before (a test and 8 dot2 per unit, 32 x 32 x 16 products, staged tail) -> now: fp16 8K 12 x 64 192 -> 180,
// 8 x 128 236 -> 221, 32 x 512 ragged 32.3 -> 30.9; bf16 8 x 128 8K 233 -> 221, 12 x 64 8K 196 -> 193, 32K 2910 both.
// ======================================================================================
// Exchange between lanes l and l ^ 16, as swap_halves does it between l and l ^ 32.
__device__ __forceinline__ void swap_rows16(float x, float& a, float& b) {
  a = b = x;
  asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
// maximum over the wavefront
__device__ __forceinline__ float row_max64(float x) {
#pragma unroll
  for (int d = 1; d < 64; d *= 2) x = fmaxf(x, __shfl_xor(x, d));
  return x;
}
// Any associative op on integers over the wavefront, without trips through LDS: by turns of rows of 16 lanes, then between rows.
template <class Op>
__device__ __forceinline__ int reduce64(int x, Op op) {
  x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x121, 0xF, 0xF, false));   // row_ror:1, 2, 4, 8
  x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x122, 0xF, 0xF, false));
  x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x124, 0xF, 0xF, false));
  x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x128, 0xF, 0xF, false));
  float a, b;
  swap_rows16(__builtin_bit_cast(float, x), a, b);
  x = op(__builtin_bit_cast(int, a), __builtin_bit_cast(int, b));
  swap_halves(__builtin_bit_cast(float, x), a, b);
  return op(__builtin_bit_cast(int, a), __builtin_bit_cast(int, b));
}
// maximum / sum over the four lanes that hold one query
__device__ __forceinline__ float max_quad(float x) {
  float a, b;
  swap_rows16(x, a, b);
  return max_xor32(fmaxf(a, b));
}
__device__ __forceinline__ float sum_quad(float x) {
  float a, b;
  swap_rows16(x, a, b);
  return sum_xor32(a + b);
}

__device__ __forceinline__ const uint16_t* bytes_on(const uint16_t* p, uint32_t bytes) { return (const uint16_t*)((const char*)p + bytes); }

// A unit of the pipeline is 32 keys x 32 queries.  How it is laid over the lanes is a policy with two members, for the two
// shapes of the matrix instruction; per lane both hold D / 16 fragments of Q, of K and of V^T, 2 of P, 16 scores and D / 2
// output values of a query block, and one score product can alternate with one output product.
//
// Tile32: v_mfma_f32_32x32x16, laid out as in the head of this file: one query per lane, shared by lanes l and l ^ 32.
//
// Tile16: v_mfma_f32_16x16x32, D = A * B + C with A: 16 x 32, B: 32 x 16, C: 16 x 16; lane l holds A[l%16][8*(l/16)..+7],
// B[8*(l/16)..+7][l%16] and C[4*(l/16) + r][l%16], r = 0..3.  Scores are formed transposed here too: a lane's accumulators
// of a 16-query tile belong to ONE query (column l%16; two tiles, two queries per lane), four lanes share a query, and the
// 4 + 4 scores that a lane holds of a 32-key block (keys 4 (l/16) + r and 16 + 4 (l/16) + r) are, packed, its B operand of
// the second product once V^T is read in the same key order.  A product with a constant first operand sums a block's
// probabilities over all four lanes.
template <class T, int D>
struct Tile32 {
  typedef typename T::v8 v8;
  static constexpr int QT = 1, E = 16, STEPS = D / 16, COLS = 32;   // queries per lane, scores per lane and query
  typedef floatx16 Scores;
  typedef floatx16 Out[D / 32];
  static constexpr bool kMfmaSum = false, kLateStep = true;
  static __device__ __forceinline__ int k_swz(int r) { return k_swz_d<D>(r); }
  static __device__ __forceinline__ int v_swz(int r) { return v_swz_d<D>(r); }
  int col, grp;                      // the lane's query column, and which of the lanes that share it
  uint32_t kfo[D / 16], vfo[D / 32];  // operand offsets (bytes) into a 32-row block

  __device__ __forceinline__ void place(int lane) { col = lane & 31, grp = lane >> 5; }
  // to the other half of a ring of eight blocks
  __device__ __forceinline__ void flip() {
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) kfo[ks] ^= 4 * 32 * D * 2;
  }
  __device__ __forceinline__ void init(int lane) {
    place(lane);
    const int p16 = lane & 15, g = (lane >> 4) & 1, row = 4 * grp + (p16 >> 2);
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) kfo[ks] = 2 * (col * D + ((2 * ks + grp) ^ k_swz(col)) * 8);
#pragma unroll
    for (int db = 0; db < D / 32; ++db) vfo[db] = 2 * (row * D + ((4 * db + 2 * g + ((p16 & 3) >> 1)) ^ v_swz(row)) * 8 + (p16 & 1) * 4);
  }
  // fragments i = 0 .. D/16 - 1 of a block: K and Q k-step i; V^T 16-key half i / (D/32), column block i % (D/32)
  __device__ __forceinline__ v8 k_frag(const uint16_t* blk, int i) const { return as_v8<T>(*(const uint4*)bytes_on(blk, kfo[i])); }
  __device__ __forceinline__ v8 v_frag(const uint16_t* blk, int i) const {
    const uint16_t* at = bytes_on(blk, vfo[i % (D / 32)]) + (i / (D / 32)) * 16 * D;
    return tr_pair<v8>(at, at + 8 * D);
  }
  static __device__ __forceinline__ void score_step(Scores& s, const v8* k, const v8* q, int i) { s = T::mfma(k[i], q[i], s); }
  // the K fragment of step i, and whether no step before uses it
  static constexpr int frag_of(int i) { return i; }
  static constexpr bool first_use(int) { return true; }
  static __device__ __forceinline__ void out_step(Out& o, const v8* v, const v8* p, int i) {
    o[i % (D / 32)] = T::mfma(v[i], p[i / (D / 32)], o[i % (D / 32)]);
  }
  // element i of a lane's scores for its query qt: key 8 (i / 4) + 4 grp + i % 4 of the block
  static __device__ __forceinline__ float get(const Scores& s, int, int i) { return s[i]; }
  // start value of a block's scores: zero, or the block's bias (four consecutive keys per quad)
  template <bool BIAS>
  __device__ __forceinline__ void start(Scores& s, const float* bias) const {
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const floatx4 b = BIAS ? *(const floatx4*)&bias[8 * x + 4 * grp] : (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int r = 0; r < 4; ++r) s[4 * x + r] = b[r];
    }
  }
  static __device__ __forceinline__ void add(Scores& s, const Scores& bias) { s += bias; }
  __device__ __forceinline__ uint32_t visible(int blk, int n) const { return visible_bits(32 * blk, grp, 0, n - 1); }
  static __device__ __forceinline__ void pack(v8* p, int, const float (&e)[E]) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      p[h] = as_v8<T>(make_uint4(T::pack2(e[8 * h], e[8 * h + 1]), T::pack2(e[8 * h + 2], e[8 * h + 3]), T::pack2(e[8 * h + 4], e[8 * h + 5]),
                                 T::pack2(e[8 * h + 6], e[8 * h + 7])));
  }
  static __device__ __forceinline__ float row_max(float x) { return max_xor32(x); }
  static __device__ __forceinline__ float row_sum(float x) { return sum_xor32(x); }
  static __device__ __forceinline__ void scale(Out& o, int, float f) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db) o[db] *= f;
  }
  // four consecutive output columns out_col(x) .. + 3 of the lane's row, x = 0 .. D / (4 * lanes per query) - 1
  static constexpr int QUADS = D / 8;
  __device__ __forceinline__ int out_col(int x) const { return 8 * x + 4 * grp; }
  static __device__ __forceinline__ floatx4 out_quad(const Out& o, int, int x) {
    const floatx16& b = o[x / 4];
    return (floatx4){b[4 * (x % 4)], b[4 * (x % 4) + 1], b[4 * (x % 4) + 2], b[4 * (x % 4) + 3]};
  }
  // chunk (16 bytes) of a row that fragment i holds in this lane
  __device__ __forceinline__ int chunk(int i) const { return 2 * i + grp; }
};

template <class T, int D>
struct Tile16 {
  typedef typename T::v8 v8;
  static constexpr int QT = 2, E = 8, STEPS = D / 8, COLS = 16, KS = D / 32;
  struct Scores { floatx4 t[2][2]; };   // [16-key tile][16-query tile]
  typedef floatx4 Out[2][D / 16];       // [16-query tile][16 columns]
  static constexpr bool kMfmaSum = true, kLateStep = false;
  static __device__ __forceinline__ int k_swz(int r) { return k_swz16<D>(r); }
  static __device__ __forceinline__ int v_swz(int r) { return v_swz16<D>(r); }
  int col, grp;
  uint32_t kfo[KS], vfo[D / 16];

  __device__ __forceinline__ void place(int lane) { col = lane & 15, grp = lane >> 4; }
  __device__ __forceinline__ void flip() {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kfo[ks] ^= 4 * 32 * D * 2;
  }
  __device__ __forceinline__ void init(int lane) {
    place(lane);
    const int row = 4 * grp + (col >> 2);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kfo[ks] = 2 * (col * D + ((4 * ks + grp) ^ k_swz(col)) * 8);
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) vfo[dt] = 2 * (row * D + ((2 * dt + ((col & 3) >> 1)) ^ v_swz(row)) * 8 + (col & 1) * 4);
  }
  // K: 16-key tile i / KS, k-step i % KS (rows r and r + 16 have the same swizzles); Q: 16-query tile, k-step; V^T: columns
  __device__ __forceinline__ v8 k_frag(const uint16_t* blk, int i) const { return as_v8<T>(*(const uint4*)(bytes_on(blk, kfo[i % KS]) + (i / KS) * 16 * D)); }
  __device__ __forceinline__ v8 v_frag(const uint16_t* blk, int i) const {
    const uint16_t* at = bytes_on(blk, vfo[i]);
    return tr_pair<v8>(at, at + 16 * D);
  }
  static __device__ __forceinline__ void score_step(Scores& s, const v8* k, const v8* q, int i) {
    const int kt = i & 1, qt = (i >> 1) & 1, ks = i >> 2;
    s.t[kt][qt] = T::mfma16(k[kt * KS + ks], q[qt * KS + ks], s.t[kt][qt]);
  }
  static constexpr int frag_of(int i) { return (i & 1) * KS + (i >> 2); }
  static constexpr bool first_use(int i) { return !(i & 2); }
  static __device__ __forceinline__ void out_step(Out& o, const v8* v, const v8* p, int i) { o[i & 1][i >> 1] = T::mfma16(v[i >> 1], p[i & 1], o[i & 1][i >> 1]); }
  static __device__ __forceinline__ float get(const Scores& s, int qt, int i) { return s.t[i >> 2][qt][i & 3]; }
  template <bool BIAS>
  __device__ __forceinline__ void start(Scores& s, const float* bias) const {
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) s.t[kt][0] = s.t[kt][1] = BIAS ? *(const floatx4*)&bias[16 * kt + 4 * grp] : (floatx4){0.f, 0.f, 0.f, 0.f};
  }
  __device__ __forceinline__ uint32_t visible(int blk, int n) const {
    const int left = n - 32 * blk - 4 * grp;   // keys below n from the lane's first one on
    const int a0 = left < 0 ? 0 : (left > 4 ? 4 : left), a1 = left < 16 ? 0 : (left > 20 ? 4 : left - 16);
    return ((1u << a0) - 1u) | (((1u << a1) - 1u) << 4);
  }
  static __device__ __forceinline__ void pack(v8* p, int qt, const float (&e)[E]) {
    p[qt] = as_v8<T>(make_uint4(T::pack2(e[0], e[1]), T::pack2(e[2], e[3]), T::pack2(e[4], e[5]), T::pack2(e[6], e[7])));
  }
  static __device__ __forceinline__ float row_max(float x) { return max_quad(x); }
  static __device__ __forceinline__ float row_sum(float x) { return sum_quad(x); }
  static __device__ __forceinline__ void scale(Out& o, int qt, float f) {
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) o[qt][dt] *= f;
  }
  static constexpr int QUADS = D / 16;
  __device__ __forceinline__ int out_col(int x) const { return 16 * x + 4 * grp; }
  static __device__ __forceinline__ floatx4 out_quad(const Out& o, int qt, int x) { return o[qt][x]; }
  __device__ __forceinline__ int chunk(int i) const { return 4 * (i % KS) + grp; }
};

// Which of the two a call runs.  What bounds the large calls is power as much as issue slots: with random operands the
// smaller shape does 20 % (fp16) and 14 % (bf16) more work per second when nothing else is issued (1905 against 1576,
// 2006 against 1722 TFLOP/s), but it takes twice the instructions, 9 - 10 issue cycles each.  fp16 at head_dim 64, whose row
// sums go to the matrix cores as well, gains from it (8K 12 x 64 192 -> 180 us; in one short round neither: 3 x 1500 30.3, 30.4).
// bf16 keeps 16 fp32 additions per unit and loses (3 x 16K 1465 -> 1516), and so does head_dim 32 in both types, whose units
// hold twice the softmax per product and whose two queries per lane cost it a wavefront per SIMD (fp16 8K 24 x 32 254 -> 278).
// head_dim 128 gains in large calls (8K 8 x 128 fp16 236 -> 221, bf16 231 -> 217); calls of little more than one 128-row
// workgroup per unit run at full clock, and there the larger shape does: kFewTiles.
template <class T, int D>
struct GlobalTile {
  typedef typename std::conditional<D == 128 || (D == 64 && T::kSumRounded), Tile16<T, D>, Tile32<T, D>>::type type;
};
// us, Tile16 -> Tile32, fp16, bf16, 8 x 128: 288 tiles of 128 rows (3 x 1500) 44.4 -> 41.9, 43.5 -> 40.3; 320 (5 x 900) 31.4 -> 29.8,
// 30.9 -> 28.9, (1 x 5000) 121 -> 118, 119 -> 114; but 384 (8 x 700) 25.7 -> 26.7, 25.7 -> 25.4; 448 (2 x 3500) 95 -> 98, 91 -> 91.
constexpr int kFewTiles = 352;

// One row's fragments straight from global memory: the B operand of Q, and the A operand of K where a refresh forms scores
// again.  FR fragments x = 0 .. FR - 1 hold chunks chunk(x); row: inside the tensor.
template <class T, int D, class M, bool ROPE>
__device__ __forceinline__ void load_row(const FaKernelArgs& a, const M& m, const uint16_t* base, int64_t rs, int row, uint4* u) {
  constexpr int FR = M::COLS == 16 ? D / 32 : D / 16;
  const uint16_t* src = base + row * rs;
#pragma unroll
  for (int x = 0; x < FR; ++x) u[x] = *(const uint4*)(src + 8 * m.chunk(x));
  if (ROPE) {
    const float *cs = a.rope_cos + (int64_t)row * a.rope_stride, *sn = a.rope_sin + (int64_t)row * a.rope_stride;
    if (FR == 1) {
      // head_dim 32, one chunk per lane: its rotary partner f +- 16 is two lanes away, so each lane rotates both and keeps its own
      const int lo_chunk = m.chunk(0) & 1;
      uint4 lo = *(const uint4*)(src + 8 * lo_chunk), hi = *(const uint4*)(src + 16 + 8 * lo_chunk);
      rotate8<T>(lo, hi, cs + 8 * lo_chunk, sn + 8 * lo_chunk);
      u[0] = m.chunk(0) < 2 ? lo : hi;
    } else {
#pragma unroll
      for (int x = 0; x < FR / 2; ++x) {
        if (D == 128) __builtin_amdgcn_sched_barrier(0);   // (one pair's table rows at a time: 16 registers)
        rotate8<T>(u[x], u[x + FR / 2], cs + 8 * m.chunk(x), sn + 8 * m.chunk(x));
      }
    }
  }
}

template <int D, int NW>
struct GlobalLds {
  // Rings of 32-key blocks of K and of V (unpadded rows, swizzled chunks); afterwards one output patch per wavefront.  Four
  // blocks of each are what the pipeline needs; four more of K keep a tile's own until its probabilities are final, so that a
  // refresh need not fetch them again (head_dim 128: a unit's LDS holds two workgroups without them, one with).
  static constexpr int kBlk = 32 * D, kKBlocks = D == 128 ? 4 : 8;
  static constexpr int kElems = (kKBlocks + 4) * kBlk > NW * epi_patch(D) ? (kKBlocks + 4) * kBlk : NW * epi_patch(D);
};

// tc: the workgroup's tile (tc.n as loaded, not clamped).
// ROPE: q and k are rotated by position (a.rope_cos / a.rope_sin are set): a compile-time
// variant, so that the kernels without a rotation carry none of its code in their loops.
template <class T, int D, int NQB, int NW, bool BIAS, bool ROTATE = true, bool ROPE = false, class M = typename GlobalTile<T, D>::type>
__device__ __forceinline__ void global_body(const FaKernelArgs& a, const TileCoord& tc_in, uint16_t* lds, float* lds_bias) {
  static_assert(D == 32 || D == 64 || D == 128, "pipelined kernel: head_dim 32, 64 or 128");
  static_assert(NW == 4 || NW == 8 || NW == 12, "4, 8 or 12 wavefronts");
  static_assert(D != 32 || NW == 4, "head_dim 32: four wavefronts");
  constexpr int THREADS = NW * 64;
  constexpr int BM = NW * 32 * NQB;
  constexpr bool BIAS_LAST = BIAS && D == 32, BIAS_FIRST = BIAS && !BIAS_LAST;
  // a loop of its own for calls whose bias turns out to be padding alone (head_dim 32 has no registers for the choice)
  constexpr bool PLAIN_LOOP = BIAS && D != 32;
  // row sums of the rounded probabilities (fp16) on the matrix cores or by dot products, else of the unrounded ones
  constexpr bool ROUNDED = T::kSumRounded && !BIAS_LAST, MFMA_SUM = M::kMfmaSum && ROUNDED, DOT_SUM = !M::kMfmaSum && ROUNDED;
  constexpr int QT = M::QT, E = M::E, FR = D / 16;
  constexpr int kBlk = 32 * D;
  typedef typename T::v8 v8;

  TileCoord tc = tc_in;
  // (uniform by construction; said explicitly so that the addresses derived from them stay in scalar registers)
  tc.b = __builtin_amdgcn_readfirstlane(tc.b);
  tc.h = __builtin_amdgcn_readfirstlane(tc.h);
  tc.q0 = __builtin_amdgcn_readfirstlane(tc.q0);
  const int N = a.max_len, q0 = tc.q0;
  const int tid = threadIdx.x;
  int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  M m;
  m.init(lane);

  const uint16_t* qp = (const uint16_t*)a.q + tc.b * a.qs[0] + tc.h * a.qs[1];
  const uint16_t* kp = (const uint16_t*)a.k + tc.b * a.ks[0] + tc.h * a.ks[1];
  const uint16_t* vp = (const uint16_t*)a.v + tc.b * a.vs[0] + tc.h * a.vs[1];
  uint16_t* op = (uint16_t*)a.o + tc.b * a.os[0] + tc.h * a.os[1];
  float* lsep = a.lse ? a.lse + ((int64_t)tc.b * a.heads + tc.h) * N : nullptr;
  const uint16_t* bp = BIAS ? (const uint16_t*)a.key_bias + tc.b * a.kb_stride : nullptr;
  // bias of key j in raw-score units (index clamped: keys outside [0, n) are never used unmasked)
  auto bias_of = [&](int j) { return bias_over_scale<T, D == 32>(a, bp[j < N ? j : N - 1]); };

  // slot (b + 5) % KN of the K ring: with eight, blocks 2 t + 1 .. 2 t + 4 (t odd) are the lower or the upper four
  constexpr int KN = GlobalLds<D, NW>::kKBlocks;
  uint16_t* const kring = lds;
  uint16_t* const vring = lds + KN * kBlk;
  auto kblk = [&](int b) { return kring + ((b + 5) & (KN - 1)) * kBlk; };
  int khalf = 0;   // the half of the ring that the operand offsets m.kfo include
  auto kops = [&](int b) { return kblk(b) - khalf; };   // what m.k_frag takes for block b
  auto vblk = [&](int b) { return vring + (b & 3) * kBlk; };

  // A direct load moves RPL rows of a 32-row block; a block's LPB loads are dealt to the wavefronts: with four, each
  // moves LPB / 4 parts of every block (head_dim 32, two parts: wavefront w moves block w of a tile's four by itself); with
  // eight or twelve, wavefronts 0 .. 3 move the first block of K and of V, 4 .. 7 the second.
  constexpr int CH = D / 8, RPL = 64 / CH, LPB = 32 / RPL;      // D = 32: 4, 16, 2;  64: 8, 8, 4;  128: 16, 4, 8
  constexpr int LW = D == 32 ? 2 : LPB / 4;
  const int fw = wave & 3;
  auto row_of = [&](int x, int lane) { return (D == 32 ? x : fw * LW + x) * RPL + lane / CH; };
  uint32_t koff[LW], voff[LW];   // bytes (row stride included)
#pragma unroll
  for (int x = 0; x < LW; ++x) {
    const int r = row_of(x, lane);
    koff[x] = 2u * (uint32_t)(r * a.ks[2] + (((lane % CH) ^ M::k_swz(r)) * 8));
    voff[x] = 2u * (uint32_t)(r * a.vs[2] + (((lane % CH) ^ M::v_swz(r)) * 8));
    if (D == 32) koff[x] = voff[x] = wave < 2 ? koff[x] + 0u : voff[x] + 0u;   // (the wavefront's own block's)
  }
  const int part0 = D == 32 ? 0 : fw * LW;
  // K blocks kb (if k1), kb + 1 (if k2) and V blocks vb, vb + 1 (if v) into ring slots
  auto fetch = [&](int kb, bool k1, bool k2, int vb, bool v) {
    if (D == 32) {
      if (wave < 2 ? (wave == 0 ? k1 : k2) : v) {
#pragma unroll
        for (int x = 0; x < LW; ++x) {
          if (wave < 2) load16_to_lds(kp + (int64_t)(32 * (kb + wave)) * a.ks[2], koff[x], kblk(kb + wave) + x * RPL * D);
          else load16_to_lds(vp + (int64_t)(32 * (vb + wave - 2)) * a.vs[2], voff[x], vblk(vb + wave - 2) + x * RPL * D);
        }
      }
    } else if (wave < 8) {
      const int s0 = NW == 4 ? 0 : wave >> 2, s1 = NW == 4 ? 1 : s0;
#pragma unroll
      for (int s = 0; s < (NW == 4 ? 2 : 1); ++s) {
        const int b = s == 0 ? s0 : s1;
#pragma unroll
        for (int x = 0; x < LW; ++x) {
          if (b == 0 ? k1 : k2) load16_to_lds(kp + (int64_t)(32 * (kb + b)) * a.ks[2], koff[x], kblk(kb + b) + (part0 + x) * RPL * D);
          if (v) load16_to_lds(vp + (int64_t)(32 * (vb + b)) * a.vs[2], voff[x], vblk(vb + b) + (part0 + x) * RPL * D);
        }
      }
    }
  };
  // The same where rows lie past the tensor: they are clamped to its last one (masked, zeroed or never read).  Rolled up over
  // the two blocks: this is the end of a sequence, and its copies would be a third of the kernel.
  auto fetch_clamped = [&](int kb, bool k1, bool k2, int vb, bool v) {
    auto load = [&](const uint16_t* base, int64_t rs, const uint32_t (&off)[LW], int blk, uint16_t* dst) {
      const int first = 32 * blk < N ? 32 * blk : N - 1;
      const uint16_t* gb = base + (int64_t)first * rs;
      const int lane = lane_now();
#pragma unroll
      for (int x = 0; x < LW; ++x) {
        const int past = row_of(x, lane) - (N - 1 - first);
        load16_to_lds(gb, off[x] - 2u * (uint32_t)((past > 0 ? past : 0) * rs), dst + (part0 + x) * RPL * D);
      }
    };
#pragma unroll 1
    for (int s = 0; s < 2; ++s) {
      const bool k_mine = D == 32 ? wave == s : (NW == 4 || (wave >> 2) == s), v_mine = D == 32 ? wave == 2 + s : k_mine;
      if (k_mine && (s == 0 ? k1 : k2)) load(kp, a.ks[2], koff, kb + s, kblk(kb + s));
      if (v_mine && v) load(vp, a.vs[2], voff, vb + s, vblk(vb + s));
    }
  };
  // ROPE: K blocks are rotated in place once they have landed: a chain of LDS reads, arithmetic and LDS writes between two
  // barriers.  The table rows are read a tile ahead where there are registers for them.  A thread has eight pairs of one row of
  // a block, the same ones every time, so that its offset in LDS stays in a register and a block's base is scalar (formed each
  // time: 2K 12 x 64 38.9 -> 41.4 us); all threads work on both blocks at once (block by block, half of them idle: 44.4).
  static_assert(!ROPE || NW == 4, "rotation: four wavefronts");
  constexpr int HALF = D / 16, BLOCK_UNITS = 32 * HALF;   // 16-byte chunks per half row; a workgroup has 1, 2 or 4 times a block's
  auto rot_row = [&](int tid) { return (tid % BLOCK_UNITS) / HALF; };
  auto rot_ch = [&](int tid) { return tid % HALF; };
  auto rot_at = [&](int tid) { return (uint32_t)(rot_row(tid) * D + (rot_ch(tid) ^ M::k_swz(rot_row(tid))) * 8); };
  const uint32_t rot_lds = rot_at(tid);
  struct Angles {
    float c[8], s[8];
  };
  // (whole wavefronts: a block's units are a multiple of 64)
  auto rot_there = [&](int x, int units) { return (x + 1) * THREADS <= units || x * THREADS + wave * 64 < units; };
  auto rot_blk = [&](int b, int x) { return b + (x * THREADS + wave * 64) / BLOCK_UNITS; };
  // the angles of pass x over the blocks from b on
  auto load_angles = [&](int b, int x, Angles& t) {
    // (rows past the tensor are never used unmasked: its last one's angles)
    const int first = 32 * rot_blk(b, x), base = first < N ? first : N - 1, id = D == 128 ? tid : wave * 64 + lane_now();
    const int row = rot_row(id) < N - 1 - base ? rot_row(id) : N - 1 - base;
    const int64_t off = (int64_t)base * a.rope_stride + (row * a.rope_stride + 8 * rot_ch(id));
    const float *cp = a.rope_cos + off, *sp = a.rope_sin + off;
#pragma unroll
    for (int i = 0; i < 8; i += 4) {
      *(float4*)&t.c[i] = *(const float4*)(cp + i);
      *(float4*)&t.s[i] = *(const float4*)(sp + i);
    }
  };
  auto rotate_unit = [&](int b, int x, const Angles& t) {
    uint16_t* at = kblk(rot_blk(b, x));
    const uint32_t own = D == 32 && NQB == 2 ? rot_at(wave * 64 + lane_now()) : rot_lds;   // (168 registers for three wavefronts)
    uint4 *lo_at = (uint4*)&at[own], *hi_at = (uint4*)&at[own ^ (8 * HALF)];
    uint4 lo = *lo_at, hi = *hi_at;
    rotate8<T>(lo, hi, t.c, t.s);
    *lo_at = lo;
    *hi_at = hi;
  };
  constexpr int TILE_UNITS = 2 * BLOCK_UNITS;   // a tile's two blocks: a pass, half a pass or (head_dim 128) two passes
  constexpr bool AHEAD = ROPE && (D == 64 || (D == 32 && NQB == 1));
  Angles ahead;
  // The first K blocks, as far as the tensor reaches, are requested before the sequence length is looked at; in longer
  // tensors the rest of tile 1's operands (K block 3, V blocks 0 and 1) with them.  us, without -> with: 16 x 700 with a bias
  // 41.8 -> 39.6, 16 x 1024 49.7 -> 49.3, but 7 x 542 14.0 -> 14.2, 32 x 128 9.2 -> 9.9 (more to wait for before the first product).
  const bool early = N >= 640;
  auto first_fetch = [&] {
  if (early) {
    fetch(0, true, true, 0, true);
    fetch(2, true, true, 0, false);
  } else if (N >= 96) {
    fetch(0, true, true, 0, false);
    fetch(2, true, false, 0, false);
  } else {
    fetch_clamped(0, true, 32 < N, 0, false);
    fetch_clamped(2, 64 < N, false, 0, false);
  }
  };
  first_fetch();

  const int qw0 = q0 + wave * 32 * NQB;
  v8 q[NQB][FR];
  {
    constexpr int FQ = FR / QT;   // fragments of one query
    uint4 u[NQB][QT][FQ];
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        const int row = qw0 + 32 * qb + M::COLS * qt + m.col;
        load_row<T, D, M, ROPE>(a, m, qp, a.qs[2], row < N ? row : N - 1, u[qb][qt]);
      }
    // only now the sequence length
    tc.n = tc.n < 0 ? 0 : (tc.n > N ? N : tc.n);
    if (q0 >= tc.n) {
      wait_direct_loads();  // the loads write this workgroup's LDS: they must land before it ends
      zero_fill<BM, D, THREADS>(a, tc, op, lsep);
      return;
    }
    const uint32_t flip = a.negate_q ? 0x80008000u : 0u;
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        // rows past the sequence take zeros: whatever is stored there must not cost refreshes
        const bool alive = qw0 + 32 * qb + M::COLS * qt + m.col < tc.n;
#pragma unroll
        for (int x = 0; x < FQ; ++x) {
          uint4 w = u[qb][qt][x];
          w.x ^= flip; w.y ^= flip; w.z ^= flip; w.w ^= flip;
          q[qb][qt * FQ + x] = as_v8<T>(alive ? w : make_uint4(0, 0, 0, 0));
        }
      }
  }
  const int n = tc.n;
  int nk = n, T64 = (n + 63) >> 6;               // keys that count, 64-key tiles
  const bool wave_has_rows = qw0 < n;
  const float c = a.c;

  typename M::Out o[NQB];
  // Reference times c, this lane's share of the row sum.  kNoRef: no key of a finite score yet.  Such keys (-infinity) have
  // probability 0 against it, the first one that counts has an infinite one, which forces a refresh.
  float mc[NQB][QT], lsum[NQB][QT];
  constexpr float kNoRef = -3.4e38f;
  v8 p[NQB][2][2];                    // [query block][key block of the tile]: the tile's probabilities
  floatx4 z[NQB][QT];                 // [0]: the lane's share of their sum (MFMA_SUM: a quarter of the row's)
  v8 ka[FR], va[FR];
  const v8 quarter = __builtin_bit_cast(v8, make_uint4(0x34003400u, 0x34003400u, 0x34003400u, 0x34003400u));  // fp16 0.25

  typename M::Scores bcur;   // BIAS_LAST: the bias of the key block in ka (head_dim 32 has the registers, and its units are short)
  // (WITHc: with the bias; a call whose keys that count all have a bias of zero runs the loop without, see below)
  auto load_ka = [&](auto WITHc, const uint16_t* kblk, const float* bblk) {
#pragma unroll
    for (int x = 0; x < FR; ++x) ka[x] = m.k_frag(kblk, x);
    if (BIAS_LAST && decltype(WITHc)::value) m.template start<true>(bcur, bblk);
  };
  auto score_init = [&](auto WITHc, typename M::Scores& s, const float* bblk) { m.template start<BIAS_FIRST && decltype(WITHc)::value>(s, bblk); };
  auto score_end = [&](auto WITHc, typename M::Scores& s) {
    if constexpr (BIAS_LAST) {   // (Tile32 always)
      if (decltype(WITHc)::value) M::add(s, bcur);
    }
  };
  // probabilities of a block against the rows' references, packed, and their sums
  auto softmax = [&](const typename M::Scores& s, float nmc, int qb, int u, int qt, bool masked, uint32_t vis) {
    float e[E];
#pragma unroll
    for (int i = 0; i < E; ++i) {
      e[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(M::get(s, qt, i), c, nmc));
      if (masked) e[i] = keep_or_zero(e[i], vis, i);
    }
    M::pack(p[qb][u], qt, e);
    if constexpr (MFMA_SUM) {
      const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
      z[qb][qt] = T::mfma16(quarter, p[qb][u][qt], u == 0 ? zero : z[qb][qt]);
    } else {
      float l0, l1;
      if constexpr (DOT_SUM) {
        const uint4 w0 = __builtin_bit_cast(uint4, p[qb][u][0]), w1 = __builtin_bit_cast(uint4, p[qb][u][1]);
        l0 = T::sum2(w1.z, T::sum2(w1.x, T::sum2(w0.z, T::sum2_first(w0.x))));
        l1 = T::sum2(w1.w, T::sum2(w1.y, T::sum2(w0.w, T::sum2_first(w0.y))));
      } else {
        l0 = e[0], l1 = e[1];
#pragma unroll
        for (int i = 2; i < E; i += 2) {
          l0 += e[i];
          l1 += e[i + 1];
        }
      }
      z[qb][qt][0] = u == 0 ? l0 + l1 : z[qb][qt][0] + (l0 + l1);
    }
  };
  constexpr float kLimit = MFMA_SUM ? 8192.f : kPLimit;
  // Rows of tile t whose sums ran away from their reference, or that found the first key that counts: the tile's scores are
  // formed again, its maximum is the new reference if it is above the old one, and the probabilities are made anew.  Each
  // row decides on its own lanes' evidence: no dependence on the rows that share its wavefront.
  auto refresh = [&](int t, bool masked) {
    auto vis_of = [&](int u) { return masked ? m.visible(2 * t + u, nk) : 0xFFFFu; };
    auto row_any = [&](bool x) { return M::row_sum(x ? 1.f : 0.f) > 0.f; };
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      bool row_trig[QT], any = false;
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        // (a row that is NaN already stays it; & and not &&: exchanges between lanes run with all lanes on)
        row_trig[qt] = row_any(!(z[qb][qt][0] <= kLimit)) & !row_any(lsum[qb][qt] != lsum[qb][qt]);
        any = any || row_trig[qt];
      }
      if (!__any(any)) continue;
      typename M::Scores s[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int blk = 2 * t + u;
        v8 kv[FR];
        if constexpr (KN == 8) {
#pragma unroll
          for (int x = 0; x < FR; ++x) kv[x] = m.k_frag(kops(blk), x);
        } else {
          __builtin_amdgcn_sched_barrier(0);   // (one block's rows at a time)
          uint4 kk[FR];
          M mr;
          mr.place(lane_now());
#pragma unroll
          for (int kt = 0; kt < QT; ++kt) {
            const int row = 32 * blk + M::COLS * kt + mr.col;
            load_row<T, D, M, ROPE>(a, mr, kp, a.ks[2], row < N ? row : N - 1, &kk[kt * (FR / QT)]);
          }
#pragma unroll
          for (int x = 0; x < FR; ++x) kv[x] = as_v8<T>(kk[x]);
        }
        const float* b = lds_bias + (BIAS ? (blk & 7) * 32 : 0);
        m.template start<BIAS_FIRST>(s[u], b);
#pragma unroll
        for (int i = 0; i < M::STEPS; ++i) M::score_step(s[u], kv, q[qb], i);
        if constexpr (BIAS_LAST) {
          typename M::Scores bs;
          m.template start<true>(bs, b);
          M::add(s[u], bs);
        }
      }
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        if (QT > 1 && !ROPE && !__any(row_trig[qt])) continue;   // (with a rotation: registers)
        float tmax = -INFINITY;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const uint32_t vis = vis_of(u);
#pragma unroll
          for (int i = 0; i < E; ++i) tmax = fmaxf(tmax, keep_or_neg_inf(M::get(s[u], qt, i), vis, i));
        }
        // (a reference only rises: the tile of a row that was expected to be cold may still lie below it)
        const float mc_tile = M::row_max(tmax) * c, mc_old = mc[qb][qt];
        const bool take = row_trig[qt] && mc_tile > mc_old;
        const float alpha = take ? __builtin_amdgcn_exp2f(mc_old - mc_tile) : 1.f;
        if (take) mc[qb][qt] = mc_tile;
        lsum[qb][qt] *= alpha;
        M::scale(o[qb], qt, alpha);
        // (a row that keeps its reference gets the same probabilities once more)
#pragma unroll
        for (int u = 0; u < 2; ++u) softmax(s[u], -mc[qb][qt], qb, u, qt, true, vis_of(u));
      }
    }
  };
  // The probabilities of tile t are final after this: one test per tile, of sums formed an iteration ago.
  auto settle = [&](int t, bool masked) {
    bool trig = false;
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) trig = trig || !(z[qb][qt][0] <= kLimit);
    if (__any(trig)) refresh(t, masked);
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) lsum[qb][qt] += z[qb][qt][0];
  };

  // ---- prologue: the first blocks have landed; first scores, first references
  float bst = 0.f;  // BIAS: wavefront 0 carries the next tile's bias from its load to its LDS write
  // row bases of the next request: K block 2 t + 3, V block 2 t
  const int64_t k32 = 32 * a.ks[2], v32 = 32 * a.vs[2];
  const uint16_t *kreq = kp + 3 * k32, *vreq = vp;
  auto request = [&](auto WITHc, int t) {   // operands of tile t + 1
    if (t == 0 && early) {
      fetch(3, false, 2 < T64, 0, false);   // (all but K block 4 are on their way)
    } else if ((t > 0 || T64 > 1) && 64 * t + 160 <= N) {
      // Every row exists (rows past the sequence are loaded for nothing at its end): the bases just advance.  (General
      // addresses each time were 40 - 60 scalar instructions per tile: 32K bf16 2845 -> 2794 us, 3 x 16K 1438 -> 1410, 8 x 2048
      // (1500 -) fp16 96.7 -> 91.5, with a bias (1024 -) 111.8 -> 107.9.)
      if (D == 32) {
        if (wave < 2) {
#pragma unroll
          for (int x = 0; x < LW; ++x) load16_to_lds(kreq + wave * k32, koff[x], kblk(2 * t + 3 + wave) + x * RPL * D);
        } else {
#pragma unroll
          for (int x = 0; x < LW; ++x) load16_to_lds(vreq + (wave - 2) * v32, voff[x], vblk(2 * t + wave - 2) + x * RPL * D);
        }
      } else if (NW == 4) {
#pragma unroll
        for (int x = 0; x < LW; ++x) {
          load16_to_lds(kreq, koff[x], kblk(2 * t + 3) + (part0 + x) * RPL * D);
          load16_to_lds(kreq + k32, koff[x], kblk(2 * t + 4) + (part0 + x) * RPL * D);
          load16_to_lds(vreq, voff[x], vblk(2 * t) + (part0 + x) * RPL * D);
          load16_to_lds(vreq + v32, voff[x], vblk(2 * t + 1) + (part0 + x) * RPL * D);
        }
      } else if (wave < 8) {
        const int s = wave >> 2;
#pragma unroll
        for (int x = 0; x < LW; ++x) {
          load16_to_lds(kreq + s * k32, koff[x], kblk(2 * t + 3 + s) + (part0 + x) * RPL * D);
          load16_to_lds(vreq + s * v32, voff[x], vblk(2 * t + s) + (part0 + x) * RPL * D);
        }
      }
    } else if (t + 2 >= T64 && 64 * t + 64 <= N && (t + 1 >= T64 || 64 * t + 128 <= N)) {
      fetch(2 * t + 3, t + 1 < T64, false, 2 * t, true);   // (the last two requests of a sequence that fills whole blocks)
    } else {
      fetch_clamped(2 * t + 3, t + 1 < T64, t + 2 < T64, 2 * t, true);
    }
    kreq += 2 * k32;
    vreq += 2 * v32;
    if (decltype(WITHc)::value && wave == 0) bst = bias_of(64 * t + 96 + lane);
    if (AHEAD && rot_there(0, TILE_UNITS)) load_angles(2 * t + 3, 0, ahead);
  };
  if (BIAS) {
    if (tid < 96) lds_bias[tid] = bias_of(tid);
  }
  // BIAS: keys end .. n - 1 have biases of -700 or less (-1010 in the log2 domain), none above top_bias (raw units), and plain: the
  // keys before them have zeros.  While the first K blocks are on their way every wavefront looks through a quarter of the
  // keys, 512 per step from the end, two steps under way, until it has seen a key that counts and has a bias.  Bound: latency, a
  // round trip to memory per two steps and the instructions behind it; one unaligned load per lane and step, steps of zeros
  // skipped, reductions without LDS.  us, without a search -> with it (eight loads per lane, one step under way): fp16 16 x 700 (350 -) 39.9 ->
  // 37.7 (38.2), 12 x 1000 (500 -) 51.8 -> 46.1 (46.7), 1 x 8192 (4096) 150.6 -> 134.4 (137.4), but biases that are no padding, keys 100 - 130
  // excluded, 16 x 700 38.8 -> 40.5 (41.5), 12 x 1000 52.9 -> 54.2 (55.1), 1 x 8192 215.9 -> 215.8 (220.9).  (In short tensors the search
  // and the pass over the padding cost more than they give: 24 x 512 (400 -) bf16 31.9 -> 34.3.)
  int end = n;
  float top_bias = -INFINITY;
  bool plain = false;
  int* const found = (int*)(lds_bias + 260);   // [wavefront][last key that counts, first with a bias, smallest cold bias's bits, -]
  // (head_dim 32: only what the pass over the padding can cut is of use, from 1024 keys on; 12 x 700 42.6 -> 40.7)
  const bool search = BIAS && early && n >= (PLAIN_LOOP ? 8 : 1024);
  if (search) {
    constexpr uint32_t kCold = T::kWideRange ? 0xC42Fu : 0xE178u, kInf = T::kWideRange ? 0xFF80u : 0xFC00u;   // -700, -infinity
    int last = -1, first_biased = INT32_MAX;   // of the lane's keys
    uint32_t cold = 0xFFFFu;
    bool seen = false;   // a key that counts and has a bias (head_dim 32: that counts)
    for (int at = (n - 1) / 512 - ((n - 1) / 512 - wave + NW) % NW; at >= 0 && !__any(seen); at -= 2 * NW) {
      // two steps under way; a lane's eight keys, at whatever alignment, end inside the sequence
      struct __attribute__((packed, aligned(2))) Eight { uint32_t w[4]; };
      auto first = [&](int u) {
        const int f = 512 * (at - u * NW) + 8 * lane;
        return f < n - 8 ? f : n - 8;
      };
      const bool two = at >= NW;
      Eight x[2];
      x[0] = *(const Eight*)(bp + first(0));
      x[1] = *(const Eight*)(bp + first(two ? 1 : 0));
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (u == 1 && !two) break;
        if (!__any(((x[u].w[0] | x[u].w[1] | x[u].w[2] | x[u].w[3]) & 0x7FFF7FFFu) != 0)) {
          last = max(last, first(u) + 7);
          seen = seen || !PLAIN_LOOP;
          continue;
        }
        uint32_t warm = 0, biased = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const uint32_t raw = i & 1 ? x[u].w[i / 2] >> 16 : x[u].w[i / 2] & 0xFFFFu;
          const bool is_cold = raw - kCold <= kInf - kCold;   // (as integers: magnitudes rise; a NaN counts)
          cold = is_cold && raw < cold ? raw : cold;          // (that of some keys before `end` too: above the others at most)
          warm |= is_cold ? 0u : 1u << i;
          biased |= (raw & 0x7FFFu) != 0 ? 1u << i : 0u;
        }
        if (warm) last = max(last, first(u) + 31 - __clz((int)warm));
        if (biased) first_biased = min(first_biased, first(u) + __ffs((int)biased) - 1);
        seen = seen || (PLAIN_LOOP ? warm & biased : warm) != 0;
      }
    }
    last = reduce64(last, [](int x, int y) { return max(x, y); });
    first_biased = reduce64(first_biased, [](int x, int y) { return min(x, y); });
    cold = (uint32_t)reduce64((int)cold, [](int x, int y) { return min(x, y); });
    if (lane == 0) *(int4*)&found[4 * wave] = make_int4(last, first_biased, (int)cold, 0);
  }
  wait_direct_loads();
  __syncthreads();
  if (ROPE) {
#pragma unroll
    for (int x = 0; x * THREADS < 3 * BLOCK_UNITS; ++x) {   // (block 3: with tile 1)
      if (!rot_there(x, 3 * BLOCK_UNITS)) continue;
      Angles t;
      load_angles(0, x, t);
      rotate_unit(0, x, t);
    }
    __syncthreads();
  }
  if (search) {
    int last = -1, first_biased = INT32_MAX, cold = 0xFFFF;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int4 f = *(const int4*)&found[4 * w];
      last = max(last, f.x);
      first_biased = min(first_biased, f.y);
      cold = min(cold, f.z);
    }
    end = __builtin_amdgcn_readfirstlane(last) + 1;
    plain = PLAIN_LOOP && end > 0 && __builtin_amdgcn_readfirstlane(first_biased) >= end;
    if (cold < 0xFFFF) top_bias = bias_over_scale<T, D == 32>(a, (uint16_t)cold);
  }
  typename M::Scores sA, sB;
  bool rotate_prio = false;
  int wslot = 0;
  // One iteration = the 64 keys of tile t.  Units (key block 2t + u, query block qb) in the order (0,0) .. (0,NQB-1), (1,0) ..:
  // the vector ALU turns the unit's scores (s_cur) into probabilities while the matrix cores form the NEXT unit's scores
  // and add the P.V of the same unit of the PREVIOUS tile.  k1, k2: LDS blocks 2t + 1, 2t + 2 of K; v1, v2: 2t - 2, 2t - 1 of V.
  auto iter = [&](auto WITHc, auto FIRSTc, auto LASTc, int t, const uint16_t* k1, const uint16_t* k2, const uint16_t* v1, const uint16_t* v2,
                  const float* b0, const float* b1, const float* b2) {
    constexpr bool FIRST = decltype(FIRSTc)::value, LAST = decltype(LASTc)::value;
    auto unit = [&](auto Uc, auto QBc, typename M::Scores& s_cur, typename M::Scores& s_nxt) {
      constexpr int U = decltype(Uc)::value, QB = decltype(QBc)::value;
      constexpr int NQ = (QB + 1) % NQB;
      constexpr bool NEXT = !(LAST && U == 1 && NQ == 0);     // there is a next unit
      const float* bnext = NQ != 0 ? (U == 0 ? b0 : b1) : (U == 0 ? b1 : b2);   // bias of the next unit's key block
      if (NQ == 0 && NEXT) load_ka(WITHc, U == 0 ? k1 : k2, bnext);
      if (QB == 0 && !FIRST) {
#pragma unroll
        for (int x = 0; x < FR; ++x) va[x] = m.v_frag(U == 0 ? v1 : v2, x);
      }
      if (NEXT) score_init(WITHc, s_nxt, bnext);
      // Score products alternate with output products.  Those whose operands the unit has yet to read from LDS come later: Tile32
      // by a step (0.5 - 1.2 % of the bf16 calls), Tile16 with a bias and two blocks by four of its eight (1 %: the next block's
      // biases are read in front of its first product); Tile16 without lost 0.5 - 1 % by it.
      constexpr int LATE_S = NQ == 0 && NQB == 2 ? (M::kLateStep ? 1 : decltype(WITHc)::value ? M::STEPS / 2 : 0) : 0;
      constexpr int LATE_O = M::kLateStep && !LATE_S ? 1 : 0;
#pragma unroll
      for (int i = 0; i < M::STEPS + (LATE_S > LATE_O ? LATE_S : LATE_O); ++i) {
        if (NEXT && !LATE_S && i < M::STEPS) M::score_step(s_nxt, ka, q[NQ], i);
        if (!FIRST && i >= LATE_O && i - LATE_O < M::STEPS) M::out_step(o[QB], va, p[QB][U], i - LATE_O);
        if (NEXT && LATE_S && i >= LATE_S) M::score_step(s_nxt, ka, q[NQ], i - LATE_S);
      }
      if (NEXT) score_end(WITHc, s_nxt);
      const uint32_t vis = LAST ? m.visible(2 * t + U, nk) : 0xFFFFu;
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) softmax(s_cur, -mc[QB][qt], QB, U, qt, LAST, vis);
      // Units moved into each other cost registers (the variants with a bias or a rotation spill), and Tile32 1 % of its time;
      // Tile16 gains 1 - 2 % by it (8K 12 x 64 179 -> 176 us), 7 x 542 2 %.
      if (M::COLS == 32 || (BIAS && (NQB == 2 || decltype(WITHc)::value)) || ROPE) __builtin_amdgcn_sched_barrier(0);
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    if constexpr (NQB == 1) {
      unit(I0{}, I0{}, sA, sB);
      unit(I1{}, I0{}, sB, sA);
    } else {
      unit(I0{}, I0{}, sA, sB);
      unit(I0{}, I1{}, sB, sA);
      unit(I1{}, I0{}, sA, sB);
      unit(I1{}, I1{}, sB, sA);
    }
  };
  // the tile's operands have landed, in every wavefront's share
  auto landed = [&](auto WITHc, int t) {
    if (decltype(WITHc)::value && wave == 0) lds_bias[(64 * t + 32 + lane) & 255] = bst;
    wait_direct_loads();
    __syncthreads();
    if (ROPE) {
      if (AHEAD) {
        if (rot_there(0, TILE_UNITS)) rotate_unit(2 * t + 1, 0, ahead);
      } else {
#pragma unroll
        for (int x = 0; x * THREADS < TILE_UNITS; ++x) {
          if (!rot_there(x, TILE_UNITS)) continue;
          Angles now;
          load_angles(2 * t + 1, x, now);
          rotate_unit(2 * t + 1, x, now);
        }
      }
      __syncthreads();
    }
  };
  auto bblk = [&](int b) { return lds_bias + (BIAS ? (b & 7) * 32 : 0); };
  using No = std::false_type;
  using Yes = std::true_type;
  // Everything from the first scores to the last tile's probabilities, with the bias (WITHc) or without; false: the padding has a
  // part in the result after all, nothing is lost but time.  (With the first scores common to both loops the variants with a
  // bias spill; with what follows the loops in here, or a bias that is optional in `refresh`, the kernels without one are
  // scheduled worse: 32K bf16 1 %.)
  int t = 0;
  auto tiles = [&](auto WITHc) {
  constexpr bool WITH = decltype(WITHc)::value;
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) lsum[qb][qt] = 0.f;
    float* of = (float*)&o[qb];
#pragma unroll
    for (int x = 0; x < D / 2; ++x) of[x] = 0.f;
  }
  load_ka(WITHc, kops(0), lds_bias);
  if (KN == 4) __syncthreads();   // K block 0 is in registers everywhere: block 4 takes its place
  request(WITHc, 0);
  {
    // (without the bias a padded key's score is an ordinary one: the first reference is that of the keys before the padding)
    const uint32_t vis = m.visible(0, WITH ? nk : end);
#pragma unroll
    for (int qb = NQB - 1; qb >= 0; --qb) {
      score_init(WITHc, sA, lds_bias);
#pragma unroll
      for (int i = 0; i < M::STEPS; ++i) M::score_step(sA, ka, q[qb], i);
      score_end(WITHc, sA);
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        float t0 = -INFINITY;
#pragma unroll
        for (int i = 0; i < E; ++i) t0 = fmaxf(t0, keep_or_neg_inf(M::get(sA, qt, i), vis, i));
        mc[qb][qt] = fmaxf(M::row_max(t0) * c, kNoRef);
      }
    }
  }

  // Padding given as a bias (-65504 per padded key) is still a score, but its probability is exactly 0 beside any ordinary
  // key: below 2^-25 for fp16, whose sums are those of the rounded values, below the fp32 range otherwise.  The keys after
  // the last one whose bias is above -700 leave the call if that can be shown ahead of it: with the
  // largest |k| among them, every row's |q|_1, and its first reference (references only rise); and if their V is finite (0
  // times it is 0).  Showing it takes one pass over their K and V without arithmetic on them.
  // Measured, us, without -> with: 8 x 2048 (1024 -) fp16 121.7 -> 112.6, 16 x 1500 (700 -) 140 -> 134, 1 x 8192 (5000) 8 x 128 239 -> 194,
  // bf16 1 x 16804 (7024) 1075 -> 654.
  // Where the keys that are left have zeros for biases (padding is all there is) the loop runs without a bias: 8 x 2048 fp16
  // 128 rows 108 -> 99.5, 256 rows 115 -> 93.5, (2048) 256 rows 127 -> 108; 16 x 700 (300 -) 38.6 -> 35.6, 1 x 8192 (5000) 163 -> 153; bf16
  // 1 x 16384 (10000) 571 -> 502, 12 x 1000 (500 -) 8 x 128 73 -> 57.
  if constexpr (BIAS) {
    // (a pass takes 3 us and 0.5 us per tile, a tile in the pipeline 1.6: from eight tiles on, but for the loop without a bias always)
    const bool cut = end > 0 && end < n && (!WITH || (n >= 1024 && (end + 63) / 64 + 8 <= T64));
    if (cut) {
      uint32_t* const shared = (uint32_t*)(lds_bias + 256);   // [0] largest |k|, [1] largest |v| (bits), [2] a wavefront refuses
      if (tid < 3) shared[tid] = 0;
      uint32_t kbits = 0, vbits = 0;   // pairs of magnitudes as 16-bit integers (an infinity or a NaN is above all others)
      typedef unsigned short us2 __attribute__((ext_vector_type(2)));
      auto grow = [](uint32_t& m, uint4 x) {
        const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int i = 0; i < 4; ++i)
          m = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(us2, m), __builtin_bit_cast(us2, w[i] & 0x7FFF7FFFu)));
      };
      constexpr int RS = THREADS / CH;
      constexpr int AHEAD = D == 128 ? 4 : 6;   // rows of K and of V that a thread has under way
      for (int r = end + tid / CH; r < n; r += AHEAD * RS) {
        uint4 kx[AHEAD], vx[AHEAD];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
          const int rr = r + i * RS < n ? r + i * RS : r;
          kx[i] = *(const uint4*)(kp + rr * a.ks[2] + (tid % CH) * 8);
          vx[i] = *(const uint4*)(vp + rr * a.vs[2] + (tid % CH) * 8);
        }
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
          grow(kbits, kx[i]);
          grow(vbits, vx[i]);
        }
      }
      __syncthreads();
      kbits = (kbits & 0xFFFFu) > (kbits >> 16) ? kbits & 0xFFFFu : kbits >> 16;
      vbits = (vbits & 0xFFFFu) > (vbits >> 16) ? vbits & 0xFFFFu : vbits >> 16;
      // (magnitudes below 2^16 as integers are exact and ordered as floats)
      kbits = (uint32_t)row_max64((float)kbits);
      vbits = (uint32_t)row_max64((float)vbits);
      if (lane == 0) {
        atomicMax(&shared[0], kbits);
        atomicMax(&shared[1], vbits);
      }
      __syncthreads();
      const uint32_t inf = T::kWideRange ? 0x7F80u : 0x7C00u;
      const float kmax = T::to_float((uint16_t)shared[0]);
      bool nothing = shared[0] < inf && shared[1] < inf;
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
          float q1 = 0.f;
#pragma unroll
          for (int x = 0; x < FR / QT; ++x) {
            const uint4 w = __builtin_bit_cast(uint4, q[qb][qt * (FR / QT) + x]);
            const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int i = 0; i < 4; ++i)
              q1 += __builtin_fabsf(T::to_float((uint16_t)ww[i])) + __builtin_fabsf(T::to_float((uint16_t)(ww[i] >> 16)));
          }
          // (1.01: the roundings of the bound and of the score itself)
          const float most = __builtin_fmaf(M::row_sum(q1) * 1.01f, kmax, top_bias * 0.99f);
          nothing = nothing && __builtin_fmaf(most, c, -mc[qb][qt]) < (MFMA_SUM ? -26.f : -160.f);
        }
      if (!__all(nothing)) shared[2] = 1;
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(shared[2]) == 0) {
        nk = end;
        T64 = (end + 63) >> 6;
      } else if (!WITH) {
        return false;
      }
    }
  }

  rotate_prio = ROTATE && NQB == 1 && T64 >= 64;
  if (rotate_prio) {
    unsigned hw_id;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(hw_id));
    wslot = (int)(hw_id & 15u);  // wave slot within the SIMD
  }

    // (a refresh reads the ring of biases: zeros, what the keys that count have)
    if (BIAS && !WITH && tid < 256) lds_bias[tid] = 0.f;
    if (T64 > 1) {
      if (wave_has_rows) iter(WITHc, Yes{}, No{}, 0, kops(1), kops(2), nullptr, nullptr, bblk(0), bblk(1), bblk(2));
      auto steady = [&](auto ODDc, int t) {
        constexpr int ODD = decltype(ODDc)::value;   // t & 1: ring slots are compile-time constants
        if (rotate_prio) {
          const int ph = (t + wslot) % 3;
          if (ph == 0) __builtin_amdgcn_s_setprio(2);
          else if (ph == 1) __builtin_amdgcn_s_setprio(1);
          else __builtin_amdgcn_s_setprio(0);
        }
        landed(WITHc, t);
        request(WITHc, t);
        if (wave_has_rows) {
          settle(t - 1, false);
          const uint16_t* k1 = kring + 2 * (1 - ODD) * kBlk;   // kops(2 t + 1)
          iter(WITHc, No{}, No{}, t, k1, k1 + kBlk, vblk(2 * ODD - 2), vblk(2 * ODD - 1), bblk(2 * t), bblk(2 * t + 1), bblk(2 * t + 2));
        }
      };
      t = 1;
      while (t + 1 < T64) {
        steady(std::integral_constant<int, 1>{}, t);
        if (++t + 1 >= T64) break;
        steady(std::integral_constant<int, 0>{}, t);
        ++t;
        if (KN == 8) {
          m.flip();
          khalf ^= 4 * kBlk;
        }
      }
      if (rotate_prio) __builtin_amdgcn_s_setprio(0);
      if (!decltype(WITHc)::value) m.place(lane_now());
      // t = T64 - 1: the last tile, masked
      landed(WITHc, t);
      request(WITHc, t);
      if (wave_has_rows) {
        settle(t - 1, false);
        iter(WITHc, No{}, Yes{}, t, kops(2 * t + 1), nullptr, vblk(2 * t - 2), vblk(2 * t - 1), bblk(2 * t), bblk(2 * t + 1), nullptr);
      }
    } else {
      if (wave_has_rows) iter(WITHc, Yes{}, Yes{}, 0, kops(1), nullptr, nullptr, nullptr, bblk(0), bblk(1), nullptr);
    }
  return true;
  };
  if constexpr (PLAIN_LOOP) {
    bool done = false;
    if (plain) {
      done = tiles(No{});
      if (!done) {
        // the padding counts after all: from the start
        wait_direct_loads();
        __syncthreads();
        kreq = kp + 3 * k32;
        vreq = vp;
        end = n;
        first_fetch();
        wait_direct_loads();
        __syncthreads();
      }
    }
    if (!done) tiles(Yes{});
  } else {
    tiles(std::integral_constant<bool, BIAS>{});
  }
  // ---- drain: V of the last tile; rows at or beyond nk are overwritten with zeros by the lanes that fetched them
  // (0 * whatever is stored in the padding must be 0)
  wait_direct_loads();
  lane = lane_now();
  m.place(lane);
  {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const bool mine = D == 32 ? wave == 2 + s : (NW == 4 || (wave >> 2) == s);
      if (mine) {
#pragma unroll
        for (int x = 0; x < LW; ++x)
          if (32 * (2 * t + s) + row_of(x, lane) >= nk) *(uint4*)&vblk(2 * t + s)[row_of(x, lane) * D + (lane % CH) * 8] = make_uint4(0, 0, 0, 0);
      }
    }
  }
  __syncthreads();
  if (wave_has_rows) {
    settle(t, true);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
      for (int x = 0; x < FR; ++x) va[x] = m.v_frag(vblk(2 * t + u), x);
#pragma unroll
      for (int i = 0; i < M::STEPS; ++i)
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) M::out_step(o[qb], va, p[qb][u], i);
    }
  }
  __syncthreads();  // all operands consumed: the rings become the output patches

  // ---- epilogue: o = O / l, cast, transposed through a private LDS patch so that whole rows are stored; lse
  {
    constexpr int kEpiStride = epi_stride(D);
    uint16_t* const patch = lds + wave * epi_patch(D);
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        const int r = M::COLS * qt + m.col, ig = qw0 + 32 * qb + r;
        const float ltot = M::row_sum(lsum[qb][qt]);
        const bool live = ig < n && ltot > 0.f;
        const float inv = live ? 1.0f / ltot : 0.f;
#pragma unroll
        for (int x = 0; x < M::QUADS; ++x) {
          const floatx4 v = M::out_quad(o[qb], qt, x);
          // padded rows and rows with no visible key: zeros
          *(uint2*)&patch[r * kEpiStride + m.out_col(x)] =
              live ? make_uint2(T::pack2(v[0] * inv, v[1] * inv), T::pack2(v[2] * inv, v[3] * inv)) : make_uint2(0, 0);
        }
        if (lsep && m.grp == 0 && ig < N) lsep[ig] = live ? (mc[qb][qt] + __builtin_amdgcn_logf(ltot)) * kLn2 : -INFINITY;
      }
      // same wavefront writes and reads the patch: program order is enough
#pragma unroll
      for (int pass = 0; pass < 32 / RPL; ++pass) {
        const int r = pass * RPL + lane / CH;
        const uint4 v = *(const uint4*)&patch[r * kEpiStride + (lane % CH) * 8];
        const int row = qw0 + 32 * qb + r;
        if (row < N) *(uint4*)(op + row * a.os[2] + (lane % CH) * 8) = v;
      }
    }
  }
}

template <class T, int D, int NQB, int NW, bool BIAS = false, bool ROPE = false, class M = typename GlobalTile<T, D>::type>
// (one block of rows per wavefront at head_dim 64: 168 registers for three wavefronts per SIMD, asked for where the compiler
// would take a few more: 16 x 700 with a bias 38.5 -> 49.8 us at two.  At head_dim 32 one block has room for four, two for
// three: 8K bf16 272 -> 247, 16 x 700 46.6 -> 43.3, with a bias 59.8 -> 51.2.)
__global__ __launch_bounds__(NW * 64, NW == 4 ? (D == 64 && NQB == 1 ? 3 : D == 32 ? (NQB == 1 ? 4 : (BIAS ? 2 : 3)) : 2) : 1) void fa_fwd_global_kernel(const FaKernelArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[GlobalLds<D, NW>::kElems];
  __shared__ __attribute__((aligned(16))) float lds_bias[BIAS ? 276 : 4];  // ring of eight key blocks, bias / |scale|; words of the pass over padding and of the search for it
  TileCoord tc;
  if (!locate_tile<NW * 32 * NQB, false, false, true>(a, tc)) return;
  global_body<T, D, NQB, NW, BIAS, true, ROPE, M>(a, tc, lds, lds_bias);
}

// ======================================================================================
// Mixed-shape global kernel (head_dim 64, ONE sequence): 256-row and 128-row workgroups in one
// launch.  A launch of 256-row workgroups alone ends, unless their number is a multiple of 512,
// with a round in which units hold one workgroup (a single wavefront per SIMD overlaps its own
// matrix and vector work badly and runs at less than half the rate) or none; the 128-row shape
// alone moves twice the K/V tile traffic per flop.  Here full rounds of 256-row pairs are
// followed by 128-row workgroups, or by pairs of one of each, on the rows that remain (one
// 8K-token sequence of 12 heads: 248 pairs on 256 units; one 16K-token sequence: 512 + 512).
// The split is made ON THE DEVICE from the sequence length, which the host does not know; the
// id -> tile arithmetic and its rules are in fa_mix_map.h.  The host launches mix_ids_a +
// kMixIdsB ids, enough for every length up to max_len.  Ids without a tile zero-fill the tiles
// that lie entirely in the padding (rows at or beyond 128 T), or exit.
// ======================================================================================
template <class T>
__global__ __launch_bounds__(kThreads, 2) void fa_fwd_global_mixed_kernel(const FaKernelArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[GlobalLds<kD, 4>::kElems];
  const int N = a.max_len, H = a.heads;
  int n = N;
  if (a.seq_lens) {
    n = a.seq_lens[0];
    n = n < 0 ? 0 : (n > N ? N : n);
  }
  const int tiles = (n + 127) >> 7;
  const FaMixTile m = fa_mix_locate((int)blockIdx.x, a.map_xcd != 0, a.mix_ids_a, kMixIdsB, H, tiles);
  TileCoord tc;
  tc.b = 0;
  tc.n = n;
  // (wavefront-uniform by construction; said explicitly so that the addresses derived from
  // them stay in scalar registers)
  tc.h = __builtin_amdgcn_readfirstlane(m.head);
  tc.q0 = __builtin_amdgcn_readfirstlane(m.q0);
  if (m.kind == 1) {
    tc.qt = m.q0 >> 8;
    global_body<T, kD, 2, 4, false, false>(a, tc, lds, nullptr);
  } else if (m.kind == 2) {
    tc.qt = m.q0 >> 7;
    global_body<T, kD, 1, 4, false, false>(a, tc, lds, nullptr);
  } else if (m.kind == 3) {
    // tiles T .. ceil(max_len / 128) - 1 of every head are padding only: o = 0, lse = -inf.
    // The spare ids share them out in a strided loop (there are normally more ids than tiles).
    const int pad = ((N + 127) >> 7) - tiles;
    for (int z = m.spare; z < pad * H; z += m.spares) {
      tc.h = z / pad;
      tc.qt = tiles + z % pad;
      tc.q0 = 128 * tc.qt;
      zero_fill<128, kD, kThreads>(a, tc, (uint16_t*)a.o + tc.h * a.os[1], a.lse ? a.lse + (int64_t)tc.h * N : nullptr);
    }
  }
}

// ======================================================================================
// Rotation of q and k ahead of a global layer.  A global layer that rotates K inside the call
// rotates every K tile once per query tile; when the caller lends scratch memory, q and k are
// rotated once here instead (the same rotate8, the same rounding: the attention kernel then
// sees bit for bit what the in-call rotation would have produced) and the plain kernels run on
// the copies.  One thread rotates eight pairs of one row; blockIdx.z < batch: q, else k.
// ======================================================================================
template <class T>
__global__ __launch_bounds__(256) void fa_rope_rotate_kernel(const FaRopeArgs r) {
  const int half = r.head_dim / 16;                      // 16-byte chunks per half row: 2, 4 or 8
  const int rows_per_block = 256 / half;
  const int row = blockIdx.x * rows_per_block + (int)threadIdx.x / half, c = (int)threadIdx.x % half;
  if (row >= r.max_len) return;
  const int h = blockIdx.y;
  const bool is_k = (int)blockIdx.z >= r.batch;
  const int b = is_k ? (int)blockIdx.z - r.batch : (int)blockIdx.z;
  const int64_t* st = is_k ? r.ks : r.qs;
  const uint16_t* src = (const uint16_t*)(is_k ? r.k : r.q) + b * st[0] + h * st[1] + row * st[2];
  uint16_t* dst = (uint16_t*)(is_k ? r.k_out : r.q_out) + (((int64_t)b * r.heads + h) * r.max_len + row) * r.head_dim;
  uint4 lo = *(const uint4*)(src + 8 * c), hi = *(const uint4*)(src + r.head_dim / 2 + 8 * c);
  const int64_t t = (int64_t)row * r.rope_stride + 8 * c;
  rotate8<T>(lo, hi, r.rope_cos + t, r.rope_sin + t);
  *(uint4*)(dst + 8 * c) = lo;
  *(uint4*)(dst + r.head_dim / 2 + 8 * c) = hi;
}

// Scratch for callers that cannot allocate (fa_fwd_ex_static_scratch): one array per GPU, held
// until the process ends.  The name below is a host-side stand-in for the symbol; the device
// address is looked up once per device and only that address is ever handed to a kernel.
static __device__ __align__(256) unsigned char fa_static_scratch_array[FA_STATIC_SCRATCH_BYTES];

typedef void (*Kernel)(const FaKernelArgs);
template <class T, int OPT>
Kernel twophase_kernel(int head_dim) {
  return head_dim == 32 ? fa_fwd_window_twophase_kernel<T, 32, OPT>
                        : (head_dim == 64 ? fa_fwd_window_twophase_kernel<T, 64, OPT> : fa_fwd_window_twophase_kernel<T, 128, OPT>);
}

// The split kernel's shapes: NQ query blocks x NK key splits, ring slots, wavefronts per SIMD asked for.  Slots fill
// the LDS of a compute unit that such a workgroup has to itself, or its share of one (head_dim 64: 1 x 4 half of it, 2 x 2
// a third; head_dim 32 without a bias a half and a third).
template <class T, bool BIAS>
Kernel split_kernel(int head_dim, int split) {
  switch (head_dim * 256 + split) {
    case 64 * 256 + 0x14: return BIAS ? nullptr : (Kernel)fa_fwd_split_kernel<T, 64, 1, 4, 2, 2, false>;
    case 64 * 256 + 0x18: return fa_fwd_split_kernel<T, 64, 1, 8, 2, 2, BIAS>;
    case 64 * 256 + 0x24: return fa_fwd_split_kernel<T, 64, 2, 4, 4, 2, BIAS>;
    case 64 * 256 + 0x34: return fa_fwd_split_kernel<T, 64, 3, 4, BIAS ? 3 : 4, 3, BIAS>;
    case 64 * 256 + 0x42: return BIAS ? (Kernel)fa_fwd_split_kernel<T, 64, 4, 2, 4, 2, true> : nullptr;
    // (without a key bias only: with one its LDS would allow two workgroups per unit instead of three)
    case 64 * 256 + 0x22: return BIAS ? nullptr : (Kernel)fa_fwd_split_kernel<T, 64, 2, 2, 2, 3, false>;
    case 128 * 256 + 0x14: return fa_fwd_split_kernel<T, 128, 1, 4, 2, 1, BIAS>;
    case 128 * 256 + 0x24: return fa_fwd_split_kernel<T, 128, 2, 4, 2, 2, BIAS>;
    case 128 * 256 + 0x42: return fa_fwd_split_kernel<T, 128, 4, 2, BIAS ? 2 : 4, 2, BIAS>;
    case 32 * 256 + 0x14: return fa_fwd_split_kernel<T, 32, 1, 4, 4, BIAS ? 1 : 2, BIAS>;
    case 32 * 256 + 0x22: return fa_fwd_split_kernel<T, 32, 2, 2, 4, 3, BIAS>;
    default: return nullptr;
  }
}

// The small kernel's shapes: wavefronts (the key splits) x key blocks of each.
template <class T, bool BIAS>
Kernel small_kernel(int head_dim, int shape) {
  switch (head_dim * 256 + shape) {
    case 32 * 256 + 0x51: return fa_fwd_small_kernel<T, 32, 5, 1, BIAS>;
    case 32 * 256 + 0x41: return fa_fwd_small_kernel<T, 32, 4, 1, BIAS>;
    case 32 * 256 + 0x42: return fa_fwd_small_kernel<T, 32, 4, 2, BIAS>;
    case 32 * 256 + 0x82: return fa_fwd_small_kernel<T, 32, 8, 2, BIAS>;
    case 64 * 256 + 0x51: return fa_fwd_small_kernel<T, 64, 5, 1, BIAS>;
    case 64 * 256 + 0x41: return fa_fwd_small_kernel<T, 64, 4, 1, BIAS>;
    case 64 * 256 + 0x42: return fa_fwd_small_kernel<T, 64, 4, 2, BIAS>;
    case 64 * 256 + 0x82: return fa_fwd_small_kernel<T, 64, 8, 2, BIAS>;
    case 128 * 256 + 0x51: return fa_fwd_small_kernel<T, 128, 5, 1, BIAS>;
    case 128 * 256 + 0x41: return fa_fwd_small_kernel<T, 128, 4, 1, BIAS>;
    case 128 * 256 + 0x42: return fa_fwd_small_kernel<T, 128, 4, 2, BIAS>;
    default: return nullptr;
  }
}

template <class T>
int launch(const FaKernelArgs& a, int bm, int v_path, int win_kernel, void* stream) {
  // (a grid of its own, whatever rows the host has laid out)
  if (a.live_tiles) {
    // one workgroup per unit, whatever the length turns out to be
    FaKernelArgs args = a;
    args.n_qtiles = a.live_tiles;
    args.total_tiles = a.live_tiles * a.heads;
    args.xcd_per = (args.total_tiles + 7) / 8;
    args.late_n = 0;
    void* argv[] = {&args};
    return (int)hipLaunchKernel((const void*)fa_fwd_split_live_kernel<T>, dim3(a.map_xcd ? 8u * (unsigned)args.xcd_per : (unsigned)args.total_tiles),
                                dim3(768), argv, 0, (hipStream_t)stream);
  }
  unsigned grid = (unsigned)a.total_tiles;
  if (a.map_xcd) grid = 8u * (unsigned)a.xcd_per * (unsigned)a.batch;
  if (bm == 0) grid = a.mix_ids_a + kMixIdsB;
  const bool global = a.wl < 0 && a.wr < 0;
  // per-lane 32-bit byte offsets into a (batch, head) slice
  const bool slice_fits_32bit = (double)a.max_len * (double)(a.ks[2] > a.vs[2] ? a.ks[2] : a.vs[2]) * 2.0 < 4.0e9;
  // 32-key blocks a 128-row query tile of a two-sided window can touch (tiles start at multiples of 128)
  const int win_blocks = (a.wl >= 0 && a.wr >= 0) ? (127 + a.wr) / 32 + (a.wl + 31) / 32 + 1 : 1 << 30;
  // 32-key blocks the 32 queries of one wavefront can see (they start at a multiple of 32)
  const int wave_blocks = (a.wl >= 0 && a.wr >= 0) ? (31 + a.wr) / 32 + (a.wl + 31) / 32 + 1 : 1 << 30;
  const bool few = ((int64_t)a.max_len + 127) / 128 * a.batch * a.heads <= kFewTiles;
  Kernel kern = nullptr;
  unsigned threads = kThreads;
  int rows = 128;   // query rows per workgroup of the kernel chosen below: what the grid has to be made for
  // rotary embedding is applied by the two-phase window kernel, the pipelined global kernel
  // (four-wavefront shapes) and the masked kernel
  const bool rope = a.rope_cos != nullptr;
  // Calls of at most 1.5 tiles per compute unit are bound by one workgroup's latency, not by
  // bandwidth: there the pipelined kernel with K and V resident (ONE memory round trip per
  // workgroup instead of two) is as fast or a little faster (measured, 12 heads: 2K tokens 7.4
  // against 7.8 us, 4K equal, 8K 17.3 against 14.9 us, 32K 43 against 37 us); it exists for
  // head_dim 64 only.
  const bool latency_bound = a.head_dim == kD && a.total_tiles <= 384;
  if (a.small) {
    // (the host has checked that the blocks fit the shape, and that it exists for the head size)
    kern = a.key_bias ? small_kernel<T, true>(a.head_dim, a.small) : small_kernel<T, false>(a.head_dim, a.small);
    threads = 64u * (unsigned)(a.small >> 4);
    rows = 32;
    if (!kern) return (int)hipErrorInvalidValue;
  } else if (a.split) {
    // (the host has checked that this shape exists for the head size)
    kern = a.key_bias ? split_kernel<T, true>(a.head_dim, a.split) : split_kernel<T, false>(a.head_dim, a.split);
    threads = 64u * (unsigned)((a.split >> 4) * (a.split & 15));
    rows = 32 * (a.split >> 4);
    if (!kern) return (int)hipErrorInvalidValue;
  } else
  if (!(a.key_bias && (rope || !(a.inv_abs_scale > 0.f))) && !global && v_path == 0 && bm == 128 && slice_fits_32bit &&
      win_blocks <= kResBlocks && wave_blocks <= kTwoPhaseBlocks && win_kernel != 1 &&
      !(latency_bound && !rope && win_kernel != 2)) {
    // local layer with a narrow two-sided window (the paper's 63/64), any head_dim
    kern = rope ? twophase_kernel<T, kTwoPhaseRope>(a.head_dim)
                : (a.key_bias ? twophase_kernel<T, kTwoPhaseBias>(a.head_dim) : twophase_kernel<T, kTwoPhasePlain>(a.head_dim));
  } else if (a.key_bias && !rope && !global && v_path == 0 && a.inv_abs_scale > 0.f && a.head_dim == kD && bm == 128 && slice_fits_32bit &&
      win_blocks <= kResBlocks) {
    // additive key bias on a local layer whose key range stays resident in LDS
    kern = fa_fwd_window_resident_kernel<T, true>;
  } else if (a.key_bias && !rope && global && v_path == 0 && a.inv_abs_scale > 0.f) {
    // additive key bias on a global layer: the pipelined kernel with the bias as MFMA C operand
    if (bm == 256 && a.head_dim != 128) rows = 256;
    if (a.head_dim == 32) kern = rows == 256 ? fa_fwd_global_kernel<T, 32, 2, 4, true> : fa_fwd_global_kernel<T, 32, 1, 4, true>;
    else if (a.head_dim == 128) kern = few ? fa_fwd_global_kernel<T, 128, 1, 4, true, false, Tile32<T, 128>> : fa_fwd_global_kernel<T, 128, 1, 4, true>;
    else if (rows == 256) kern = fa_fwd_global_kernel<T, 64, 2, 4, true>;
    else kern = fa_fwd_global_kernel<T, 64, 1, 4, true>;
  } else if (a.key_bias) {
    // additive key bias otherwise: the masked kernel, 128-row tiles, any head_dim and window
    if (a.head_dim == 32) kern = fa_fwd_masked_kernel<T, 32, 1, true, true>;
    else if (a.head_dim == 64) kern = fa_fwd_masked_kernel<T, 64, 1, true, true>;
    else kern = fa_fwd_masked_kernel<T, 128, 1, true, true>;
  } else if (rope && global && v_path == 0) {
    // rotation on a global layer: the pipelined kernel's four-wavefront shapes
    if (bm == 256 && a.head_dim != 128) rows = 256;
    // (the same arithmetic as a call whose q and k were rotated ahead of it, few tiles or many: the same bits)
    if (a.head_dim == 128) kern = few ? fa_fwd_global_kernel<T, 128, 1, 4, false, true, Tile32<T, 128>> : fa_fwd_global_kernel<T, 128, 1, 4, false, true>;
    else if (a.head_dim == 32) kern = rows == 256 ? fa_fwd_global_kernel<T, 32, 2, 4, false, true> : fa_fwd_global_kernel<T, 32, 1, 4, false, true>;
    else kern = rows == 256 ? fa_fwd_global_kernel<T, 64, 2, 4, false, true> : fa_fwd_global_kernel<T, 64, 1, 4, false, true>;
  } else if (a.head_dim == 128 && global && v_path == 0) {
    if (bm == 256) {
      kern = few ? fa_fwd_global_kernel<T, 128, 1, 8, false, false, Tile32<T, 128>> : fa_fwd_global_kernel<T, 128, 1, 8>;   // eight wavefronts on one pair of rings
      threads = 512;
      rows = 256;
    } else {
      kern = few ? fa_fwd_global_kernel<T, 128, 1, 4, false, false, Tile32<T, 128>> : fa_fwd_global_kernel<T, 128, 1, 4>;
    }
  } else if (a.head_dim == 32 && global && v_path == 0) {
    if (bm == 256) rows = 256;
    kern = rows == 256 ? fa_fwd_global_kernel<T, 32, 2, 4> : fa_fwd_global_kernel<T, 32, 1, 4>;
  } else if (a.head_dim != kD) {
    // wide or one-sided windows of head_dim 32 / 128 (and the 16-bit V-read path): the masked
    // kernel covers every mask; bm is 128 here
    if (a.head_dim == 32) kern = v_path == 0 ? fa_fwd_masked_kernel<T, 32, 1, true> : fa_fwd_masked_kernel<T, 32, 1, false>;
    else kern = v_path == 0 ? fa_fwd_masked_kernel<T, 128, 1, true> : fa_fwd_masked_kernel<T, 128, 1, false>;
  } else if (global && v_path == 0) {
    rows = bm;
    if (bm == 0) {
      kern = fa_fwd_global_mixed_kernel<T>;
    } else if (bm == 512) {
      kern = fa_fwd_global_kernel<T, 64, 2, 8>;
      threads = 512;
    } else if (bm == 384) {
      kern = fa_fwd_global_kernel<T, 64, 1, 12>;
      threads = 768;
    } else if (bm == 256) {
      kern = fa_fwd_global_kernel<T, 64, 2, 4>;
    } else {
      kern = fa_fwd_global_kernel<T, 64, 1, 4>;
      rows = 128;
    }
  } else if (!global && !rope && v_path == 0 && bm == 128 && slice_fits_32bit) {
    kern = win_blocks <= kResBlocks ? fa_fwd_window_resident_kernel<T> : fa_fwd_window_kernel<T>;
  } else if (bm == 256) {
    rows = 256;
    kern = v_path == 0 ? fa_fwd_masked_kernel<T, 64, 2, true> : fa_fwd_masked_kernel<T, 64, 2, false>;
  } else {
    kern = v_path == 0 ? fa_fwd_masked_kernel<T, 64, 1, true> : fa_fwd_masked_kernel<T, 64, 1, false>;
  }
  if (rows != bm) return (int)hipErrorInvalidValue;   // the grid is made of tiles of another size
  // hipLaunchKernel returns THIS launch's status; an error left by the caller's earlier HIP
  // work stays where it is (neither reported as ours nor cleared)
  FaKernelArgs args = a;
  void* argv[] = {&args};
  return (int)hipLaunchKernel((const void*)kern, dim3(grid), dim3(threads), argv, 0, (hipStream_t)stream);
}

}  // namespace

int fa_launch_rope_rotate(const FaRopeArgs& r, int is_bf16, void* stream) {
  const int rows_per_block = 256 / (r.head_dim / 16);
  const dim3 grid((unsigned)((r.max_len + rows_per_block - 1) / rows_per_block), (unsigned)r.heads, 2u * (unsigned)r.batch);
  FaRopeArgs args = r;
  void* argv[] = {&args};
  const void* kern = is_bf16 ? (const void*)fa_rope_rotate_kernel<BF16> : (const void*)fa_rope_rotate_kernel<F16>;
  return (int)hipLaunchKernel(kern, grid, dim3(256), argv, 0, (hipStream_t)stream);
}

int fa_static_scratch(void** ptr) {
  constexpr int kMaxDevices = 64;
  static void* per_device[kMaxDevices] = {};   // each GPU holds its own copy of the array at its own address
  static std::mutex lock;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  if (dev < 0 || dev >= kMaxDevices) return (int)hipErrorInvalidDevice;
  std::lock_guard<std::mutex> guard(lock);
  if (!per_device[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(fa_static_scratch_array));
    if (e != hipSuccess) return (int)e;
    per_device[dev] = p;
  }
  *ptr = per_device[dev];
  return 0;
}

int fa_launch_f16(const FaKernelArgs& a, int bm, int v_path, int win_kernel, void* stream) {
  return launch<F16>(a, bm, v_path, win_kernel, stream);
}
int fa_launch_bf16(const FaKernelArgs& a, int bm, int v_path, int win_kernel, void* stream) {
  return launch<BF16>(a, bm, v_path, win_kernel, stream);
}
