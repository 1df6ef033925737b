// Expert FFNs of the selected experts only (SwiGLU, nn.Linear [out, in] weights, bf16):
//   gate/up:  H[p, :] = silu(x_i W1_e^T) * (x_i W3_e^T)      for every permuted row p = (i, r)
//   down:     Y[i*k + r, :] = H[p, :] W2_e^T
// H is kept as hi = bf16(H) and lo = bf16(H - hi) (about 16 significant bits): with H in
// bf16 alone its rounding moved large outputs across a bf16 rounding boundary of y.  The two
// are interleaved in 8-element chunks, so a token's hi and lo for one k-range share a cache
// line.  The down GEMM feeds both to one MFMA: 8 tokens per 16-row tile, hi rows 0-7 and lo
// rows 8-15, summed after the reduction.
//   combine:  y_i = sum_r w_ir Y[i*k + r, :]  (rank order, fp32) -> bf16
// Always-on shared experts (Section 2.1) are extra slots after the routed ones, with all T
// tokens; their output rows are added after the routed terms with weight 1.  The router
// GEMM h = W_g x uses the same wave pass with the router rows as weights.
//
// Decode batches give an expert 1..T tokens, so each weight element is used a few times:
// the GEMMs are bound by streaming the selected experts' weights from HBM.  Each wave owns
// 16 weight rows and the whole reduction dimension; weights go from HBM straight into the
// B operand of v_mfma_f32_16x16x32_bf16 (lane (n, g) loads 16 contiguous bytes of row n per
// MFMA, so a wave reads 16 rows x 32*U contiguous elements per step), tokens form the M
// dimension (16 per tile, up to two tiles per pass), accumulation is fp32.  The block's
// four waves share the expert and its token rows, which the block stages in LDS one step
// at a time (block_pass); the next step's loads are issued before the current step's
// MFMAs (register double buffering).  A reduction that is no multiple of the step ends in a
// partial step of whole 32-element MFMAs (kRest), for any d and f the library takes: with a
// step that divides them instead (32 elements and per-wave token loads for odd multiples of
// 32) T=37 N=60 k=6 d=2720 f=1376 M=30 took 190 us a layer, now 162.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "internal.h"
#include "xshare.h"

namespace xs {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kBlock = 256;       // 4 waves
constexpr int kWaves = kBlock / 64;
constexpr int kCols = 16;         // weight rows (output columns) per wave
constexpr int kTiles = 2;         // 16-token tiles per pass over the weights

// Block timeline of the expert GEMMs, in a profiling build only (XS_BLOCK_TIMES 1, the
// library libxshare_timeline.so): thread 0 of every block of a gate/up and a down launch
// stamps its start and end, and every block of a persistent down launch its start and the
// end of each unit, from the 100 MHz global clock (s_memrealtime), by block id; each launch
// overwrites the entries of its blocks.  xshare_block_times copies them out.
#ifndef XS_BLOCK_TIMES
#define XS_BLOCK_TIMES 0
#endif
constexpr int kTimeSeqStride = XSHARE_TIME_SEQ_STRIDE;  // a block's start, then 32 unit ends
#if XS_BLOCK_TIMES
constexpr int kTimeBlocks = XSHARE_TIME_BLOCKS;         // stamped blocks of a grid launch
constexpr int kTimeSeqBlocks = XSHARE_TIME_SEQ_BLOCKS;  // stamped persistent down blocks
__device__ unsigned long long xs_times_gu[2 * kTimeBlocks];
__device__ unsigned long long xs_times_dn[2 * kTimeBlocks];
__device__ unsigned long long xs_times_seq[kTimeSeqBlocks * kTimeSeqStride];
__device__ __forceinline__ unsigned block_id3() {
  return (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
}
#define XS_TIME(arr, idx, lim)                                                          \
  do {                                                                                  \
    if (threadIdx.x == 0 && (idx) < (lim)) arr[idx] = __builtin_amdgcn_s_memrealtime(); \
  } while (0)
#else
#define XS_TIME(arr, idx, lim) \
  do {                         \
  } while (0)
#endif

__device__ __forceinline__ bf16x8 load8(const uint16_t* p) {
  return *reinterpret_cast<const bf16x8*>(p);
}

__device__ __forceinline__ floatx4 mfma(const bf16x8& a, const bf16x8& b, const floatx4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ uint16_t to_bf16(float v) {
  uint32_t b = __float_as_uint(v);
  b += 0x7FFFu + ((b >> 16) & 1u);  // round to nearest even
  return (uint16_t)(b >> 16);
}

__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// 8 FP8 E4M3FN codes (two words, element order = byte order) -> 8 bf16.  The hardware
// conversion gives fp32; an E4M3 value has at most 4 significant bits, so its upper 16 bits
// are the exact bf16 (v_perm_b32 gathers the upper halves of two floats).
__device__ __forceinline__ bf16x8 fp8x8_to_bf16(uint2 v) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const f32x2 a = __builtin_amdgcn_cvt_pk_f32_fp8((int)v.x, false);
  const f32x2 b = __builtin_amdgcn_cvt_pk_f32_fp8((int)v.x, true);
  const f32x2 c = __builtin_amdgcn_cvt_pk_f32_fp8((int)v.y, false);
  const f32x2 d = __builtin_amdgcn_cvt_pk_f32_fp8((int)v.y, true);
  u32x4 r;
  r.x = __builtin_amdgcn_perm(__float_as_uint(a.y), __float_as_uint(a.x), 0x07060302u);
  r.y = __builtin_amdgcn_perm(__float_as_uint(b.y), __float_as_uint(b.x), 0x07060302u);
  r.z = __builtin_amdgcn_perm(__float_as_uint(c.y), __float_as_uint(c.x), 0x07060302u);
  r.w = __builtin_amdgcn_perm(__float_as_uint(d.y), __float_as_uint(d.x), 0x07060302u);
  return __builtin_bit_cast(bf16x8, r);
}

__device__ __forceinline__ uint2 load_q8(const uint8_t* p) {
  return *reinterpret_cast<const uint2*>(p);
}

// Weight formats of the expert GEMMs.
constexpr int kBf16 = 0;   // bf16
constexpr int kFp8 = 1;    // OCP FP8 E4M3FN codes, one fp32 scale per output row
constexpr int kMx4 = 2;    // MXFP4: E2M1 codes, two per byte, one E8M0 scale per 32 elements

// 8U packed E2M1 codes of one lane and step (U words, 8 elements each, low nibble first).
template <int U>
struct Q4 {
  uint32_t w[U];
};
template <int U>
__device__ __forceinline__ Q4<U> load_q4(const uint8_t* p) {
  Q4<U> r;
  if constexpr (U == 16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint4 v = *reinterpret_cast<const uint4*>(p + 16 * i);
      r.w[4 * i] = v.x;
      r.w[4 * i + 1] = v.y;
      r.w[4 * i + 2] = v.z;
      r.w[4 * i + 3] = v.w;
    }
  } else if constexpr (U == 8) {
    const uint4 v = *reinterpret_cast<const uint4*>(p);
    const uint4 w = *reinterpret_cast<const uint4*>(p + 16);
    r.w[0] = v.x;
    r.w[1] = v.y;
    r.w[2] = v.z;
    r.w[3] = v.w;
    r.w[4] = w.x;
    r.w[5] = w.y;
    r.w[6] = w.z;
    r.w[7] = w.w;
  } else {
    static_assert(U == 4, "4, 8 or 16 words");
    const uint4 v = *reinterpret_cast<const uint4*>(p);
    r.w[0] = v.x;
    r.w[1] = v.y;
    r.w[2] = v.z;
    r.w[3] = v.w;
  }
  return r;
}

// E8M0 scale byte -> 2^(e - 127) as fp32 (e = 0 is the subnormal 2^-127).
__device__ __forceinline__ float e8m0_scale(uint32_t e) {
  return e ? __uint_as_float(e << 23) : __uint_as_float(0x00400000u);
}

// 8 E2M1 codes (one word) times their block scale -> 8 bf16.  The conversion (one byte, two
// elements, per instruction; low nibble first) multiplies by a power of two, so the result
// is exact for scales that keep the weights in bf16's normal range.
__device__ __forceinline__ bf16x8 fp4x8_to_bf16(uint32_t w, float scale) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 p0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, scale, 0);
  const bf16x2 p1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, scale, 1);
  const bf16x2 p2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, scale, 2);
  const bf16x2 p3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, scale, 3);
  bf16x8 r;
  r[0] = p0[0];
  r[1] = p0[1];
  r[2] = p1[0];
  r[3] = p1[1];
  r[4] = p2[0];
  r[5] = p2[1];
  r[6] = p3[0];
  r[7] = p3[1];
  return r;
}

// Stores v = H[p, c] as hi = bf16(v) and lo = bf16(v - hi) in the interleaved rows of 2f
// elements: hi at 16 (c / 8) + c % 8, lo 8 elements further.
__device__ __forceinline__ void store_hilo(uint16_t* h2, size_t p, int c, int f, float v) {
  const uint16_t h = to_bf16(v);
  uint16_t* const at = h2 + p * 2 * (size_t)f + 2 * (c & ~7) + (c & 7);
  at[0] = h;
  at[8] = to_bf16(v - from_bf16(h));
}

// Reduction offsets of the bf16 passes: MFMA u of a step and lane group g.  The four lane
// groups of one MFMA read 32 contiguous elements, so one load instruction touches half as many
// cache lines as with 8U contiguous elements a lane; measured 0.3-1.2 % faster.
__device__ __forceinline__ constexpr int kstep(int u) { return 32 * u; }
__device__ __forceinline__ constexpr int klane(int g) { return 8 * g; }

// One pass of a wave of the router GEMM over the reduction dimension K for up to kTiles token
// tiles: acc[rt] += A_rt (16 x K) * B^T (K x 16).  `arow[rt]` points at the token row this lane
// feeds (a duplicate of a valid row for padding lanes, whose output rows are discarded;
// duplicate addresses coalesce, which measured faster than masking those lanes), `brow` at the
// weight row of this lane's column; both already offset by klane.  Loads run one step ahead.
template <int U>
__device__ __forceinline__ void wave_pass(const uint16_t* const (&arow)[kTiles], int nt,
                                          const uint16_t* brow, int K, floatx4 (&acc)[kTiles]) {
  constexpr int KB = 32 * U;
  bf16x8 b[U], x[kTiles][U];
#pragma unroll
  for (int u = 0; u < U; ++u) b[u] = load8(brow + kstep(u));
#pragma unroll
  for (int rt = 0; rt < kTiles; ++rt)
    if (rt < nt)
#pragma unroll
      for (int u = 0; u < U; ++u) x[rt][u] = load8(arow[rt] + kstep(u));
  for (int kb = 0; kb < K; kb += KB) {
    bf16x8 nb[U], nx[kTiles][U];
    const bool more = kb + KB < K;
    if (more) {
#pragma unroll
      for (int u = 0; u < U; ++u) nb[u] = load8(brow + kb + KB + kstep(u));
#pragma unroll
      for (int rt = 0; rt < kTiles; ++rt)
        if (rt < nt)
#pragma unroll
          for (int u = 0; u < U; ++u) nx[rt][u] = load8(arow[rt] + kb + KB + kstep(u));
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int rt = 0; rt < kTiles; ++rt)
        if (rt < nt) acc[rt] = mfma(x[rt][u], b[u], acc[rt]);
    if (more) {
#pragma unroll
      for (int u = 0; u < U; ++u) b[u] = nb[u];
#pragma unroll
      for (int rt = 0; rt < kTiles; ++rt)
#pragma unroll
        for (int u = 0; u < U; ++u) x[rt][u] = nx[rt][u];
    }
  }
}

// MXFP4 block scales in the tiled layout (xshare_mx_scales_tile): per matrix of R rows and K
// inputs, [R / 16][G][16 rows][8 bytes] with G = ceil(K / 256) granules of 8 blocks of 32
// inputs, so the scale bytes of one 16-row weight tile over 256 inputs are one 128-byte
// piece, read once and whole: the byte of row r and block c sits at ((r / 16) G + c / 8) 128
// + (r % 16) 8 + c % 8.  mx_row: where row r's bytes of its tile start (granule 0).
__device__ __forceinline__ int mx_granules(int K) { return (K + 255) >> 8; }
__device__ __forceinline__ const uint8_t* mx_row(const uint8_t* mat, int r, int G) {
  return mat + (size_t)(r >> 4) * G * 128 + (r & 15) * 8;
}
// The scale bytes of a lane whose step starts at input k (8U inputs: one block for U <= 4,
// two for U = 8, four for U = 16; a lane's blocks share one granule since k is a multiple of
// 8U), from its row `row` (mx_row).
template <int U>
__device__ __forceinline__ uint32_t load_mx_scales(const uint8_t* row, int k) {
  const int c = k >> 5;
  const uint8_t* const p = row + ((c >> 3) << 7) + (c & 7);
  if constexpr (U >= 16)
    return *reinterpret_cast<const uint32_t*>(p);
  else if constexpr (U == 8)
    return *reinterpret_cast<const uint16_t*>(p);
  else
    return *p;
}

// Token rows staged in LDS.  With tokens loaded per wave (wave_pass*), every wave of a block
// gathers the same token rows again, as half-line loads; with MXFP4 weights (a quarter of
// bf16's bytes) these were as many load instructions as the weights', or more.  In both
// expert GEMMs the four waves of a block share the expert, the token rows and the reduction
// range: this pass has the block load each step's token rows once, coalesced (16 bytes per
// thread, P threads per row), into a double-buffered LDS tile, and the waves read their A
// operands from it.  The loads of step s + 1 (tokens, then weights) are issued before the
// MFMAs of step s, with no branch around them, so the wait before the LDS write covers the
// token loads only and the weight loads stay in flight across the barrier.  One barrier per
// step: the writes into the other buffer come after this step's reads of it were fenced by
// the previous barrier.
//   gate/up (kDown false): staged rows are x rows, 16 per MFMA tile (lane row n).
//   down (kDown true): staged rows are H rows (hi and lo chunks interleaved, two elements
//   per k), 8 per tile: lanes n < 8 read token n's hi chunk, lanes n >= 8 its lo chunk.
constexpr int kStageRows = 32;            // token rows per pass
template <int U, bool kDown>
struct Stage {
  static constexpr int KB = 32 * U;                  // reduction elements per step
  static constexpr int AS = kDown ? 2 : 1;           // staged elements per reduction element
  static constexpr int P = AS * KB / 8;              // 16-byte pieces per row and step
  static_assert(P * kStageRows >= kBlock, "256 threads cover at most the 32 rows of a step");
  static constexpr int TR = kDown ? 8 : 16;          // token rows per MFMA tile
  // LDS row stride (elements): the rows of one A read start 16 B (x) or 32 B (H, whose lo
  // lanes read 16 B past their hi lanes) apart modulo 256 B, so they fall in distinct banks
  static constexpr int LS = AS * KB + (kDown ? 16 : 8);
  static constexpr int kElems = 2 * kStageRows * LS; // both buffers
};

// One lane's weights of one step for one 16-row tile, by format: where they are (w: this
// lane's first element; sc: MXFP4 scale bytes), the registers that hold them, their loads
// for step s and the B operand of MFMA u.  `koff(g, u)`: the reduction offset, within a
// step, of lane group g's elements in MFMA u (the A operand reads the same).
// The `rest` members serve the last, partial step of a reduction that is no multiple of the
// step: elements 32u + 8g of each lane group in MFMA u, so that every lane of an MFMA has
// elements.  load_rest takes the MFMAs u0 <= u < n, each from a constant offset (clamped addresses
// took registers for every one of them).
template <int kW, int U>
struct WTile;
template <int U>
struct WTile<kBf16, U> {
  struct Ptr { const uint16_t* w; };
  struct Regs { bf16x8 w[U]; };
  using Rest = Regs;
  __device__ static constexpr int koff(int g, int u) { return kstep(u) + klane(g); }
  __device__ static Regs load(const Ptr& p, int s) {
    Regs r;
#pragma unroll
    for (int u = 0; u < U; ++u) r.w[u] = load8(p.w + s + kstep(u));
    return r;
  }
  __device__ static bf16x8 operand(const Regs& r, int u) { return r.w[u]; }
  __device__ static Rest load_rest(const Ptr& p, int s, int, int u0, int n) {
    Rest r;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (u >= u0 && u < n) r.w[u] = load8(p.w + s + 32 * u);
    return r;
  }
  __device__ static bf16x8 operand_rest(const Rest& r, int u) { return r.w[u]; }
};
template <int U>
struct WTile<kFp8, U> {
  struct Ptr { const uint8_t* w; };
  struct Regs { uint2 w[U]; };
  using Rest = Regs;
  __device__ static constexpr int koff(int g, int u) { return 8 * U * g + 8 * u; }
  __device__ static Regs load(const Ptr& p, int s) {
    Regs r;
#pragma unroll
    for (int u = 0; u < U; ++u) r.w[u] = load_q8(p.w + s + 8 * u);
    return r;
  }
  __device__ static bf16x8 operand(const Regs& r, int u) { return fp8x8_to_bf16(r.w[u]); }
  __device__ static Rest load_rest(const Ptr& p, int s, int g, int u0, int n) {
    const uint8_t* const w = p.w - (8 * U - 8) * g + s;
    Rest r;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (u >= u0 && u < n) r.w[u] = load_q8(w + 32 * u);
    return r;
  }
  __device__ static bf16x8 operand_rest(const Rest& r, int u) { return operand(r, u); }
};
template <int U>
struct WTile<kMx4, U> {
  // w: this lane's codes; sc: its row's tiled scales (mx_row); k: its first input (absolute)
  struct Ptr { const uint8_t* w; const uint8_t* sc; int k; };
  // scale bytes (block u / 4 in byte u / 4) in a type no wider than their load: a widening
  // at the end of a step would wait for the load
  using E8 = typename std::conditional<(U == 8), uint16_t, uint8_t>::type;
  using E = typename std::conditional<(U > 8), uint32_t, E8>::type;
  struct Regs { Q4<U> q; E e; };
  struct Rest { uint32_t w[U]; uint8_t e[U]; };
  __device__ static constexpr int koff(int g, int u) { return 8 * U * g + 8 * u; }
  __device__ static Regs load(const Ptr& p, int s) {
    Regs r;
    r.q = load_q4<U>(p.w + s / 2);
    r.e = (E)load_mx_scales<U>(p.sc, p.k + s);
    return r;
  }
  __device__ static bf16x8 operand(const Regs& r, int u) {
    const uint32_t e = r.e;
    return fp4x8_to_bf16(r.q.w[u], e8m0_scale((e >> (8 * (u >> 2))) & 0xFFu));
  }
  __device__ static Rest load_rest(const Ptr& p, int s, int g, int u0, int n) {
    const uint8_t* const w = p.w - (4 * U - 4) * g + s / 2;
    const int k = p.k - 8 * U * g + s;
    Rest r;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u < u0 || u >= n) continue;
      r.w[u] = *reinterpret_cast<const uint32_t*>(w + 16 * u);
      r.e[u] = (uint8_t)load_mx_scales<1>(p.sc, k + 32 * u);
    }
    return r;
  }
  __device__ static bf16x8 operand_rest(const Rest& r, int u) {
    return fp4x8_to_bf16(r.w[u], e8m0_scale(r.e[u]));
  }
};

// NT: token tiles of the pass (R <= TR * NT rows); NL: loads per thread and step, at least
// ceil(R * P / 256) (pieces beyond R * P repeat the last one).  Staged row r (r < R) is
// x[tok[r] * ld ...], x already offset to this block's reduction range.  acc[m][rt]: the sums of
// weight tile m and token tile rt.  kRest: K is no multiple of the step (k_first is 0).
template <int kW, int U, bool kDown, int NM, int NT, int NL, bool kRest, int TA>
__device__ __forceinline__ void block_pass(const uint16_t* x, size_t ld, const int* tok, int R,
                                           const typename WTile<kW, U>::Ptr (&wp)[NM], int K,
                                           int k_first, floatx4 (&acc)[NM][TA], uint16_t* lds) {
  using S = Stage<U, kDown>;
  using WT = WTile<kW, U>;
  constexpr int KB = S::KB;
  static_assert(NT <= TA && S::TR * NT <= kStageRows, "tiles of the pass");
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const int t = threadIdx.x, lane = t & 63;
  const int n = lane & 15, g = lane >> 4;
  const uint16_t* src[NL];   // this thread's pieces: global source and LDS offset
  int wofs[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int q = min(t + i * kBlock, R * S::P - 1);
    const int row = q / S::P, piece = q % S::P;
    src[i] = x + (size_t)tok[row] * ld + piece * 8;
    wofs[i] = row * S::LS + piece * 8;
  }
  int rofs[NT];              // this lane's A rows (padding lanes repeat the last token row)
#pragma unroll
  for (int rt = 0; rt < NT; ++rt)
    rofs[rt] = kDown ? min(8 * rt + (n & 7), R - 1) * S::LS + (n & 8)
                     : min(16 * rt + n, R - 1) * S::LS;

  u32x4 v[NL];
  typename WT::Regs b[NM];
  // kRest: the reduction ends in a partial step of `ut` MFMAs of 32 elements, the last ut of the
  // full step that ends with it (its loads then run under the step before it, as every step's
  // do), or the first ut of one that starts with it where it is shorter than a step.  The 64-row
  // down instances leave the short case to the 32-row ones: with it they spilled.
  constexpr bool kShort = !(kDown && NM > 2);
  const int ut = K % KB >> 5, Kf = K - 32 * ut;
  typename WT::Rest rb[kRest ? NM : 1];
  auto step_rest = [&](const uint16_t* cur, int u0, int u1) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u < u0 || u >= u1) continue;
      const int ka = S::AS * (32 * u + 8 * g);
      bf16x8 xa[NT];
#pragma unroll
      for (int rt = 0; rt < NT; ++rt)
        xa[rt] = *reinterpret_cast<const bf16x8*>(cur + rofs[rt] + ka);
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        const bf16x8 bv = WT::operand_rest(rb[kRest ? m : 0], u);
#pragma unroll
        for (int rt = 0; rt < NT; ++rt) acc[m][rt] = mfma(xa[rt], bv, acc[m][rt]);
      }
    }
  };
  if (kRest && kShort && Kf == 0) {
    // a piece past the row reads the row's start; no MFMA takes it
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int piece = min(t + i * kBlock, R * S::P - 1) % S::P;
      v[i] = *reinterpret_cast<const u32x4*>(src[i] - (piece < 4 * S::AS * ut ? 0 : piece * 8));
    }
#pragma unroll
    for (int m = 0; m < NM; ++m) rb[kRest ? m : 0] = WT::load_rest(wp[m], 0, g, 0, ut);
#pragma unroll
    for (int i = 0; i < NL; ++i) *reinterpret_cast<u32x4*>(lds + wofs[i]) = v[i];
    __syncthreads();
    step_rest(lds, 0, ut);
    __syncthreads();
    return;
  }
#pragma unroll
  for (int i = 0; i < NL; ++i) v[i] = *reinterpret_cast<const u32x4*>(src[i] + S::AS * k_first);
#pragma unroll
  for (int m = 0; m < NM; ++m) b[m] = WT::load(wp[m], k_first);
#pragma unroll
  for (int i = 0; i < NL; ++i) *reinterpret_cast<u32x4*>(lds + wofs[i]) = v[i];
  __syncthreads();

  // MFMAs of one step from LDS buffer `cur`
  auto step = [&](const uint16_t* cur) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int ka = S::AS * WT::koff(g, u);
      bf16x8 xa[NT];
#pragma unroll
      for (int rt = 0; rt < NT; ++rt)
        xa[rt] = *reinterpret_cast<const bf16x8*>(cur + rofs[rt] + ka);
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        const bf16x8 bv = WT::operand(b[m], u);
#pragma unroll
        for (int rt = 0; rt < NT; ++rt) acc[m][rt] = mfma(xa[rt], bv, acc[m][rt]);
      }
    }
  };
  int buf = 0;
  // loads of step kn, MFMAs of the step before it, then kn's tokens into the other buffer
  auto advance = [&](int kn) {
#pragma unroll
    for (int i = 0; i < NL; ++i) v[i] = *reinterpret_cast<const u32x4*>(src[i] + S::AS * kn);
    typename WT::Regs nb[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) nb[m] = WT::load(wp[m], kn);
    step(lds + buf * kStageRows * S::LS);
    uint16_t* const nxt = lds + (buf ^ 1) * kStageRows * S::LS;
#pragma unroll
    for (int i = 0; i < NL; ++i) *reinterpret_cast<u32x4*>(nxt + wofs[i]) = v[i];
#pragma unroll
    for (int m = 0; m < NM; ++m) b[m] = nb[m];
    __syncthreads();
    buf ^= 1;
  };
  // the pass starts at step k_first and wraps around (two plain loops: a wrap test inside
  // one loop measured slower)
  for (int kn = k_first + KB; kn < (kRest ? Kf : K); kn += KB) advance(kn);
  for (int kn = 0; kn < k_first; kn += KB) advance(kn);
  if constexpr (kRest) {
    const int kr = K - KB;
#pragma unroll
    for (int i = 0; i < NL; ++i) v[i] = *reinterpret_cast<const u32x4*>(src[i] + S::AS * kr);
    // bf16: the first half of that step is loaded only where the partial step reaches into it (a
    // gate/up of d an odd multiple of 128 1 % faster; FP8 and MXFP4 measured no gain)
    if (kW != kBf16 || ut > U / 2) {
#pragma unroll
      for (int m = 0; m < NM; ++m) rb[m] = WT::load_rest(wp[m], kr, g, 0, U);
    } else {
#pragma unroll
      for (int m = 0; m < NM; ++m) rb[m] = WT::load_rest(wp[m], kr, g, U / 2, U);
    }
    step(lds + buf * kStageRows * S::LS);
    uint16_t* const nxt = lds + (buf ^ 1) * kStageRows * S::LS;
#pragma unroll
    for (int i = 0; i < NL; ++i) *reinterpret_cast<u32x4*>(nxt + wofs[i]) = v[i];
    __syncthreads();
    step_rest(nxt, U - ut, U);
  } else {
    step(lds + buf * kStageRows * S::LS);
  }
  __syncthreads();                         // the block's next pass rewrites both buffers
}

// The staged pass over R token rows, by block-uniform instance: the fewest tiles that hold
// R rows and the loads per thread that the largest R of that tile count needs.
template <int kW, int U, bool kDown, int NM, bool kRest, int TA>
__device__ __forceinline__ void staged_pass(const uint16_t* x, size_t ld, const int* tok,
                                               int R, const typename WTile<kW, U>::Ptr (&wp)[NM],
                                               int K, int k_first, floatx4 (&acc)[NM][TA],
                                               uint16_t* lds) {
  using S = Stage<U, kDown>;
  constexpr int TR = S::TR;
  constexpr int L1 = (TR * S::P + kBlock - 1) / kBlock, L2 = (2 * TR * S::P + kBlock - 1) / kBlock;
  if constexpr (TA == 2) {          // gate/up: up to two 16-row tiles
    constexpr int L1h = (TR / 2 * S::P + kBlock - 1) / kBlock;
    constexpr int L2h = (3 * TR / 2 * S::P + kBlock - 1) / kBlock;
    if (R <= TR / 2)
      block_pass<kW, U, kDown, NM, 1, L1h, kRest, TA>(x, ld, tok, R, wp, K, k_first, acc, lds);
    else if (R <= TR)
      block_pass<kW, U, kDown, NM, 1, L1, kRest, TA>(x, ld, tok, R, wp, K, k_first, acc, lds);
    else if (R <= 3 * TR / 2)
      block_pass<kW, U, kDown, NM, 2, L2h, kRest, TA>(x, ld, tok, R, wp, K, k_first, acc, lds);
    else
      block_pass<kW, U, kDown, NM, 2, L2, kRest, TA>(x, ld, tok, R, wp, K, k_first, acc, lds);
  } else {                          // down: up to four 8-token tiles
    static_assert(TA == 2 || TA == 4, "two or four 8-token tiles");
    if (R <= TR) {
      block_pass<kW, U, kDown, NM, 1, L1, kRest, TA>(x, ld, tok, R, wp, K, k_first, acc, lds);
    } else if (TA == 2 || R <= 2 * TR) {
      block_pass<kW, U, kDown, NM, 2, L2, kRest, TA>(x, ld, tok, R, wp, K, k_first, acc, lds);
    } else if constexpr (TA == 4) {
      constexpr int L3 = (3 * TR * S::P + kBlock - 1) / kBlock;
      constexpr int L4 = (4 * TR * S::P + kBlock - 1) / kBlock;
      if (R <= 3 * TR)
        block_pass<kW, U, kDown, NM, 3, L3, kRest, TA>(x, ld, tok, R, wp, K, k_first, acc, lds);
      else
        block_pass<kW, U, kDown, NM, 4, L4, kRest, TA>(x, ld, tok, R, wp, K, k_first, acc, lds);
    }
  }
}

// Unroll (32-element k-groups per step) and token-operand buffering of the two GEMMs.
#ifndef XS_GATE_UP_U
#define XS_GATE_UP_U 4
#endif
#ifndef XS_DOWN_U
#define XS_DOWN_U 2
#endif
#ifndef XS_Q8_GATE_UP_U
#define XS_Q8_GATE_UP_U 4
#endif
#ifndef XS_Q8_DOWN_U
#define XS_Q8_DOWN_U 4
#endif
// gate/up launches whose grid keeps at least this many blocks with two column tiles per
// wave use two (measured: DeepSeek T=32 gate/up -1 % bf16, -5 % FP8, -10 % MXFP4; a grid
// half that size, as at T=8, ran 10-14 % slower).
// bf16 and FP8 down launches use twice the base tiles per wave when the routed rows are at
// least XS_DN_WIDE_TOKENS per expected expert and the grid keeps XS_DN_WIDE_MIN_BLOCKS blocks
// (measured on DeepSeek T=32 and the speculative batch: bf16 down -1.6 % and -3 %, FP8 -10 %
// and -13 %; with 1-3 tokens per expert, as at T=8, wide waves ran 4-20 % slower).
#ifndef XS_DN_WIDE_TOKENS
#define XS_DN_WIDE_TOKENS 4
#endif
#ifndef XS_DN_WIDE_MIN_BLOCKS
#define XS_DN_WIDE_MIN_BLOCKS 768
#endif
#ifndef XS_GU_CT2_MIN_BLOCKS
#define XS_GU_CT2_MIN_BLOCKS 768
#endif
#ifndef XS_Q4_GU_CT2_MIN_BLOCKS
#define XS_Q4_GU_CT2_MIN_BLOCKS XS_GU_CT2_MIN_BLOCKS
#endif
#ifndef XS_Q4_GATE_UP_U
#define XS_Q4_GATE_UP_U 8
#endif
// Unroll of one-tile gate/up launches (small grids), twice the two-tile one for bf16:
// twice the weight bytes in flight per wave where there are fewer waves.  Same-box A/B:
// bf16 DeepSeek T=32 M=24 gate/up 246 -> 237 us, Mixtral 232 -> 215, T=8 239 -> 234.  FP8
// at 8 words gained on Mixtral and lost on Qwen and T=8.  MXFP4 gained from 16 words while
// every step read its scales; with scales read once per four steps, 8 words are ahead
// (DeepSeek T=8 M=24 gate/up 76.2 -> 74.5 us, Mixtral 69.1 -> 67.1 us).
#ifndef XS_GATE_UP_U1
#define XS_GATE_UP_U1 8
#endif
#ifndef XS_Q8_GATE_UP_U1
#define XS_Q8_GATE_UP_U1 XS_Q8_GATE_UP_U
#endif
// FP8 gate/up instances of up to 4 words a step held to 3 waves per SIMD (168 registers, no
// spills; left alone the compiler kept 2).  Same-box A/B, gate/up us (2 -> 3 waves):
// DeepSeek T=32 M=48 252.0 -> 246.6, speculative 335.5 -> 331.8, T=8 M=24 127.0 -> 124.5,
// Qwen 32.9 -> 32.4, Mixtral 137.8 -> 135.0.  Not kept at 3 waves: the two-tile MXFP4
// gate/up (72 bytes spilled; DeepSeek T=32 138 -> 152 us) and the 32-row FP8 down (no
// change).
#ifndef XS_Q8_GU_W3
#define XS_Q8_GU_W3 1
#endif
#ifndef XS_Q4_GATE_UP_U1
#define XS_Q4_GATE_UP_U1 8
#endif
#ifndef XS_Q4_DOWN_U
#define XS_Q4_DOWN_U 8
#endif
#ifndef XS_Q4_DN_WIDE
#define XS_Q4_DN_WIDE 1
#endif
#ifndef XS_Q4_DOWN_ROT
#define XS_Q4_DOWN_ROT 0
#endif
// K steps between the starts of consecutive down waves (blocks, when the pass is staged):
// one with bf16 weights (per wave: DeepSeek T=32 down 270 -> 263 us; per block, staged:
// 266 -> 258 us, speculative 358 -> 351 us); none with FP8, where it measured no gain.
#ifndef XS_DOWN_ROT
#define XS_DOWN_ROT 1
#endif
#ifndef XS_Q8_DOWN_ROT
#define XS_Q8_DOWN_ROT 0
#endif
// Expert slots from which the down grid keeps each slot's column blocks on one XCD (with
// fewer, whole XCDs would idle: five experts left three of eight without work).
#ifndef XS_DOWN_XCD_SLOTS
#define XS_DOWN_XCD_SLOTS 16
#endif
static_assert(XS_DOWN_XCD_SLOTS >= 8, "at least one slot per XCD");
#ifndef XS_DOWN_TL
#define XS_DOWN_TL 4                 // 8-token (hi + lo) tiles per pass of the down GEMM
#endif
// Seven 16-row W2 tiles per wave (448 output rows per block, one block per CU) for the bf16
// down GEMM when that grid is a whole number of rounds: at d = 7168 the DeepSeek layer's 48
// slots give 768 blocks, three rounds, where 64-row waves leave 2.6 rounds of 512.  With
// U = 4 a wave keeps 28 KB of weights in flight.  Same-box A/B, down us (64-row waves ->
// seven tiles): DeepSeek T=32 M=48 256 -> 245, iid logits 257 -> 245, speculative 347 ->
// 333; M=96 (six rounds against 5.25) 464 -> 464; at U = 2 M=48 ran 260, and on grids
// that leave a partial round the seven tiles lose (M=24 138 -> 148, the layer with its
// shared expert 262 -> 295).  FP8 gained nothing (DeepSeek 137 -> 136, speculative 188 ->
// 191) and MXFP4 lost (81 -> 85 us), so they keep their waves.
#ifndef XS_DOWN_NM7
#define XS_DOWN_NM7 1
#endif
#ifndef XS_DOWN_NM7_U
#define XS_DOWN_NM7_U 4
#endif
// The seven-tile bf16 down launch as a persistent grid (down_seq_kernel).  Same-box A/B,
// down us (grid of rounds -> persistent): DeepSeek T=32 M=48 246.0 / 245.8 -> 243.5 / 242.5,
// speculative 333.2 / 334.9 -> 331.9 / 333.1.  With 2 waves per SIMD (FP8 and bf16 64- and
// 32-row waves) it lost: FP8 DeepSeek T=32 137.4 -> 147.0, bf16 T=8 M=24 130 -> 133.5 (a
// CU's second block already overlaps the first one's start there), so only this launch
// takes it.
#ifndef XS_DOWN_SEQ
#define XS_DOWN_SEQ 1
#endif


#ifndef XS_DOWN_WAVES_PER_EU
#define XS_DOWN_WAVES_PER_EU 2       // waves per SIMD of the staged down instances (3: spills)
#endif

// Every format stages the token rows in LDS.  Same-box A/B against per-wave token loads,
// gate/up and down (us):
//   bf16  DeepSeek T=32 M=48  469 / 262 -> 460 / 258   M=24  250 / 165 -> 245 / 138
//         Qwen M=32            64 /  40 ->  53 /  32   DeepSeek T=8  236 / 132 -> 237 / 132
//   FP8   DeepSeek T=32 M=48  249 / 147 -> 249 / 138   speculative  371 / 209 -> 329 / 189
//   MXFP4 DeepSeek T=32 M=48  193 / 142 -> 170 /  99   Qwen M=32     44 /  32 ->  25 /  19
// A down pass rotates its start by block, not by wave (the waves of a block share one token
// step).

// Work of grid row `slot` of the expert GEMMs: the always-on shared experts first (all T
// tokens, rows T*k + s*T + t, kSlotRows of them a slot at most; their blocks are the longest,
// so they start first and do not trail the launch), then the routed active experts (their
// tokens' rows in permuted order).  False for rows beyond both.  `e` is the shared or the
// routed expert.  kW: weight format (shared experts have bf16 weights, so the others' kernels
// carry no trace of them: the two-tile FP8 gate/up spilled two registers of its 168 with it).
struct SlotWork {
  int e, p0, te;
  bool shared;
};

template <int kW>
__device__ __forceinline__ bool slot_work(const FfnArgs& a, int slot, SlotWork& w) {
  if (kW == kBf16 && slot < a.shared_slots) {
    int t0 = 0, t1 = a.T;
    w.e = slot;
    if (a.shared_parts > 1) {
      w.e = slot / a.shared_parts;
      t0 = a.T * (slot - w.e * a.shared_parts) / a.shared_parts;
      t1 = a.T * (slot - w.e * a.shared_parts + 1) / a.shared_parts;
    }
    w.p0 = a.T * a.k + w.e * a.T + t0;
    w.te = t1 - t0;
    w.shared = true;
    return true;
  }
  const int r = slot - (kW == kBf16 ? a.shared_slots : 0);
  // both loads are issued together; the record is used only below the count
  const int n_active = a.counters[kCntActive];
  const int4 rec = a.active[r < a.max_active ? r : 0];
  if (r >= n_active) return false;
  w.e = rec.x;
  w.p0 = rec.y;
  w.te = rec.z;
  w.shared = false;
  return true;
}

// The slot's bf16 weight matrix (routed or shared), or its FP8 codes (routed only).
__device__ __forceinline__ const uint16_t* slot_w(const FfnArgs& a, const SlotWork& w,
                                                  const uint16_t* routed,
                                                  const uint16_t* shared) {
  return (w.shared ? shared : routed) + (size_t)w.e * a.f * a.d;
}
__device__ __forceinline__ const uint8_t* slot_q(const FfnArgs& a, const SlotWork& w,
                                                 const uint8_t* codes) {
  return codes + (size_t)w.e * a.f * a.d;
}

// kSplit: the block covers one part of the reduction (blockIdx.z) and writes fp32 gate and
// up partials; otherwise it covers all of d and writes H directly.
// CT: column tiles (16 weight rows of W1 and of W3 each) per wave; with two, one token load
// feeds four weight tiles instead of two, at the cost of registers and of half as many
// blocks (the launch takes two only for grids that stay large).
// The MXFP4 one-tile instance is held to 168 registers (3 waves per SIMD): left alone the
// compiler took 175 and 2 waves, and DeepSeek T=8 gate/up ran 14 % slower.  So are the FP8
// instances of up to 4 words a step (XS_Q8_GU_W3) but the split two-tile one, which would spill
// (it runs the few blocks of a launch's tail).  The two-tile bf16 and FP8 instances with a
// partial step are compiled for at most 1 and 2 waves (the compiler then reserves the registers
// that keep them there): with one wave more they ran slower (rows that start inside a cache line share it
// with the next row; gate/up us at d=4128 f=2976 T=16 M=40: bf16 384 -> 408, FP8 236 -> 247).
template <int kW, int U, int CT, bool kRest>
constexpr int gu_max_waves() {
  if (kRest && CT == 2 && kW != kMx4) return kW == kBf16 ? 1 : 2;
  return 8;
}
template <int kW, int U, int CT, bool kSplit, bool kRest>
constexpr int gu_waves() {
  if (kW == kMx4 && CT == 1) return 3;
  if (kW == kFp8 && U <= 4 && XS_Q8_GU_W3 && !((kSplit || kRest) && CT == 2)) return 3;
  return kRest && !(kW == kBf16 && CT == 2) ? 2 : 1;
}
template <int U, bool kSplit, int kW, int CT, bool kRest>
__global__ __attribute__((amdgpu_waves_per_eu(gu_waves<kW, U, CT, kSplit, kRest>(),
                                              gu_max_waves<kW, U, CT, kRest>())))
__launch_bounds__(kBlock) void gate_up_kernel(FfnArgs a) {
  constexpr int NM = 2 * CT;                   // weight tiles: W1 and W3 of each column tile
  SlotWork sw;
  if (!slot_work<kW>(a, a.slot_base + blockIdx.y, sw)) return;
  XS_TIME(xs_times_gu, 2 * block_id3(), 2u * kTimeBlocks);
  const int p0 = sw.p0, te = sw.te;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int j0 = (blockIdx.x * kWaves + wave) * kCols * CT;
  // the staged pass needs the whole block: a wave past f stays for the staging and the
  // barriers (its columns are clamped into range and its stores skipped)
  const int n = lane & 15, g = lane >> 4;
  const int d = a.d, f = a.f;
  const int Kg = kSplit ? d / a.gu_splits : d;   // this block's part of the reduction
  const size_t kbase = kSplit ? (size_t)blockIdx.z * Kg : 0;
  const size_t k0 = kbase + (size_t)(kW == kBf16 ? klane(g) : g * 8 * U);
  const size_t plane = (size_t)a.part_rows * f;   // one fp32 partial plane [part_rows, f]
  int col[CT];                                 // this lane's column of each tile (< f)
  float sc[NM];                                // FP8 per-row scales (else 1)
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    col[ct] = min(j0 + 16 * ct, f - 16) + n;
    sc[2 * ct] = kW == kFp8 ? a.s1[(size_t)sw.e * f + col[ct]] : 1.0f;
    sc[2 * ct + 1] = kW == kFp8 ? a.s3[(size_t)sw.e * f + col[ct]] : 1.0f;
  }

  for (int c0 = 0; c0 < te; c0 += 16 * kTiles) {
    const int nt = min(kTiles, (te - c0 + 15) / 16);
    floatx4 acc[NM][kTiles];
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int rt = 0; rt < kTiles; ++rt) acc[m][rt] = floatx4{0.f, 0.f, 0.f, 0.f};
    typename WTile<kW, U>::Ptr wp[NM];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const size_t wrow = (size_t)col[ct] * d + k0;
      if constexpr (kW == kBf16) {
        wp[2 * ct].w = slot_w(a, sw, a.w1, a.sw1) + wrow;
        wp[2 * ct + 1].w = slot_w(a, sw, a.w3, a.sw3) + wrow;
      } else if constexpr (kW == kFp8) {
        wp[2 * ct].w = slot_q(a, sw, a.q1) + wrow;
        wp[2 * ct + 1].w = slot_q(a, sw, a.q3) + wrow;
      } else {        // row col of the expert: d / 2 code bytes; its tiled scale row
        const size_t r = (size_t)sw.e * f + col[ct];
        const int G = mx_granules(d);
        const size_t emat = (size_t)sw.e * f * G * 8;     // the expert's scale matrix
        wp[2 * ct] = {a.q1 + r * (d / 2) + k0 / 2, mx_row(a.e1 + emat, col[ct], G), (int)k0};
        wp[2 * ct + 1] = {a.q3 + r * (d / 2) + k0 / 2, mx_row(a.e3 + emat, col[ct], G), (int)k0};
      }
    }
    __shared__ __align__(16) uint16_t stage[Stage<U, false>::kElems];
    __shared__ int s_tok[kStageRows];
    const int R = min(kStageRows, te - c0);
    if (threadIdx.x < R)
      s_tok[threadIdx.x] =
          sw.shared ? p0 - a.T * (a.k + sw.e) + c0 + threadIdx.x   // shared rows: token order
                    : a.perm[p0 + c0 + threadIdx.x] / a.k;
    __syncthreads();
    staged_pass<kW, U, false, NM, kRest, kTiles>(a.x + kbase, d, s_tok, R, wp, Kg, 0, acc, stage);
#pragma unroll
    for (int rt = 0; rt < kTiles; ++rt) {
      if (rt >= nt) break;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = c0 + rt * 16 + 4 * g + i;
        if (t < te) {
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            if (j0 + 16 * ct >= f) break;
            const float h1 = acc[2 * ct][rt][i] * sc[2 * ct];
            const float h3 = acc[2 * ct + 1][rt][i] * sc[2 * ct + 1];
            if (!kSplit) {
              store_hilo(a.h, p0 + t, col[ct], f, h1 / (1.0f + __expf(-h1)) * h3);
            } else {
              // the tail's planes hold its slots' rows only
              const size_t prow = a.part_compact ? (size_t)blockIdx.y * a.T + t : (size_t)(p0 + t);
              const size_t at = prow * f + col[ct];
              float* const part = a.gpart + 2 * blockIdx.z * plane;
              part[at] = h1;
              part[plane + at] = h3;
            }
          }
        }
      }
    }
  }
  XS_TIME(xs_times_gu, 2 * block_id3() + 1, 2u * kTimeBlocks);
}

// Gate/up of a few small experts that hold a few rows each, where the launch would otherwise
// split d over blocks: here the four waves of a block split it over the same 16 columns and add
// their sums through LDS, so there are no partial planes and no finish pass (4.7 us, most of it
// its launch).  Each wave reads its own part of the token rows.  Measured, layer us (split grid
// and finish pass -> this; steps of 2 / 4 / 8 groups): Qwen T=1 bf16 41.6 -> 37.0 / 38.0 / 41.0,
// FP8 35.3 -> 32.9 / 32.0 / 32.8, MXFP4 36.8 -> 34.3 / 34.0 / 34.3; T=2 bf16 49.1 -> 45.0, FP8
// 38.7 -> 36.5, MXFP4 35.7 -> 34.2.
template <int U, int kW>
__global__ __launch_bounds__(kBlock) void gate_up_narrow_kernel(FfnArgs a) {
  using WT = WTile<kW, U>;
  constexpr int KB = 32 * U;
  SlotWork sw;
  if (!slot_work<kW>(a, blockIdx.y, sw)) return;
  XS_TIME(xs_times_gu, 2 * block_id3(), 2u * kTimeBlocks);
  const int p0 = sw.p0, te = sw.te;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int n = lane & 15, g = lane >> 4;
  const int d = a.d, f = a.f;
  const int K = d / kWaves;                      // this wave's part (a multiple of 32)
  const int kbase = wave * K;
  const int col = blockIdx.x * kCols + n;
  const size_t k0 = (size_t)kbase + (kW == kBf16 ? klane(g) : g * 8 * U);
  typename WT::Ptr wp[2];
  const size_t wrow = (size_t)col * d + k0;
  if constexpr (kW == kBf16) {
    wp[0].w = slot_w(a, sw, a.w1, a.sw1) + wrow;
    wp[1].w = slot_w(a, sw, a.w3, a.sw3) + wrow;
  } else if constexpr (kW == kFp8) {
    wp[0].w = slot_q(a, sw, a.q1) + wrow;
    wp[1].w = slot_q(a, sw, a.q3) + wrow;
  } else {
    const size_t r = (size_t)sw.e * f + col;
    const int G = mx_granules(d);
    const size_t emat = (size_t)sw.e * f * G * 8;
    wp[0] = {a.q1 + r * (d / 2) + k0 / 2, mx_row(a.e1 + emat, col, G), (int)k0};
    wp[1] = {a.q3 + r * (d / 2) + k0 / 2, mx_row(a.e3 + emat, col, G), (int)k0};
  }
  const float s1 = kW == kFp8 ? a.s1[(size_t)sw.e * f + col] : 1.0f;
  const float s3 = kW == kFp8 ? a.s3[(size_t)sw.e * f + col] : 1.0f;
  __shared__ floatx4 sums[kWaves][2][64];        // per 16-row tile: gate and up of every wave

  for (int c0 = 0; c0 < te; c0 += 16) {
    const int t = min(c0 + n, te - 1);
    const int tok = sw.shared ? p0 - a.T * (a.k + sw.e) + t : a.perm[p0 + t] / a.k;
    const uint16_t* const xr = a.x + (size_t)tok * d + kbase;
    floatx4 acc[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
    const int Kf = K / KB * KB, ut = (K - Kf) >> 5;
    typename WT::Regs b[2];
    bf16x8 x[U];
    auto load = [&](typename WT::Regs (&rb)[2], bf16x8 (&rx)[U], int k) {
#pragma unroll
      for (int m = 0; m < 2; ++m) rb[m] = WT::load(wp[m], k);
#pragma unroll
      for (int u = 0; u < U; ++u) rx[u] = load8(xr + k + WT::koff(g, u));
    };
    if (Kf > 0) load(b, x, 0);
    for (int k = 0; k < Kf; k += KB) {
      typename WT::Regs nb[2];
      bf16x8 nx[U];
      load(nb, nx, min(k + KB, Kf - KB));        // past the last step: that step again
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int m = 0; m < 2; ++m) acc[m] = mfma(x[u], WT::operand(b[m], u), acc[m]);
#pragma unroll
      for (int m = 0; m < 2; ++m) b[m] = nb[m];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = nx[u];
    }
    // the partial step (bf16 has none, its d is a multiple of 256 here; but compiled without this
    // branch the Qwen T=1 layer ran 37.8 -> 38.6 us)
    if (ut) {
      typename WT::Rest rb[2];
#pragma unroll
      for (int m = 0; m < 2; ++m) rb[m] = WT::load_rest(wp[m], Kf, g, 0, ut);
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = load8(xr + Kf + 32 * min(u, ut - 1) + 8 * g);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (u >= ut) break;
#pragma unroll
        for (int m = 0; m < 2; ++m) acc[m] = mfma(x[u], WT::operand_rest(rb[m], u), acc[m]);
      }
    }
    sums[wave][0][lane] = acc[0];
    sums[wave][1][lane] = acc[1];
    __syncthreads();
    // wave i finishes row 4g + i of each lane group: the waves' sums in order
    float h1 = 0.f, h3 = 0.f;
#pragma unroll
    for (int v = 0; v < kWaves; ++v) {
      h1 += sums[v][0][lane][wave];
      h3 += sums[v][1][lane][wave];
    }
    h1 *= s1;
    h3 *= s3;
    if (c0 + 4 * g + wave < te)
      store_hilo(a.h, p0 + c0 + 4 * g + wave, col, f, h1 / (1.0f + __expf(-h1)) * h3);
    __syncthreads();                             // the next rows rewrite the sums
  }
  XS_TIME(xs_times_gu, 2 * block_id3() + 1, 2u * kTimeBlocks);
}

// NM: 16-row W2 tiles per wave (the launch picks it per weight format and batch shape).
// Staged down instances are held to 2 waves per SIMD: left alone the compiler took 1 for the
// 64-row bf16 and FP8 instances (FP8 DeepSeek T=32 down 166 -> 138 us with the hint).
// TL: token tiles per pass, 8 tokens each (hi and lo rows).
template <int U, int kW, int NM, bool kRest, int TL = XS_DOWN_TL>
__global__ __attribute__((amdgpu_waves_per_eu(NM <= 4 ? XS_DOWN_WAVES_PER_EU
                                                                          : 1)))
__launch_bounds__(kBlock) void down_kernel(FfnArgs a) {
  // (bx, slot): this block's column block and expert slot.  In grids of at least
  // XS_DOWN_XCD_SLOTS slots, with `live` slots holding work (shared, then active), all
  // column blocks of slot y < 8 * (live / 8) run on XCD y mod 8 (the dispatcher deals
  // consecutive workgroups to the 8 XCDs in turn), so one L2 serves the slot's H rows to
  // all of them; the blocks of the other slots keep the plain order, which spreads the
  // last live % 8 slots over all XCDs.
  int bx = blockIdx.x, slot = blockIdx.y;
  if (gridDim.y >= XS_DOWN_XCD_SLOTS) {
    const int L = blockIdx.x + gridDim.x * blockIdx.y;
    const int live = a.shared_slots + a.counters[kCntActive];   // <= gridDim.y
    if (L < (int)gridDim.x * (live & ~7)) {
      const int s = L >> 3;
      slot = (L & 7) + 8 * (s / gridDim.x);
      bx = s % gridDim.x;
    }
  }
  SlotWork sw;
  if (!slot_work<kW>(a, slot, sw)) return;
  XS_TIME(xs_times_dn, 2 * block_id3(), 2u * kTimeBlocks);
  const int p0 = sw.p0, te = sw.te;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int n0 = (bx * kWaves + wave) * kCols * NM;
  // the staged pass needs the whole block (see gate_up_kernel)
  const int n = lane & 15, g = lane >> 4;
  const int d = a.d, f = a.f;
  const int Ks = f / a.splits;                 // this block's part of the reduction
  const size_t k0 = (size_t)blockIdx.z * Ks + (size_t)(kW == kBf16 ? klane(g) : g * 8 * U);
  float* const ypart = a.yslot + (size_t)blockIdx.z * a.rows * d;
  size_t wrow[NM];
  int rowm[NM];
  float sc[NM];                                        // FP8 per-row scales (else 1)
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    rowm[m] = min(n0 + 16 * m, d - 16) + n;
    wrow[m] = (size_t)rowm[m] * f + k0;
    sc[m] = kW == kFp8 ? a.s2[(size_t)sw.e * d + rowm[m]] : 1.0f;
  }

  for (int c0 = 0; c0 < te; c0 += 8 * TL) {
    const int nt = min(TL, (te - c0 + 7) / 8);
    floatx4 acc[NM][TL];
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int rt = 0; rt < TL; ++rt) acc[m][rt] = floatx4{0.f, 0.f, 0.f, 0.f};
    // Consecutive blocks start their pass over K one step apart (and wrap around): W2 rows
    // are f elements apart, often a power of two, so blocks that stepped through K in the
    // same order would read the same offsets of every row at the same time.
    const int rot = kW == kBf16 ? XS_DOWN_ROT : (kW == kFp8 ? XS_Q8_DOWN_ROT : XS_Q4_DOWN_ROT);
    const int k_first = kRest ? 0 : (int)((bx * rot) % (Ks / (32 * U))) * 32 * U;
    static_assert(TL == 2 || TL == 4, "two or four 8-token tiles");
    typename WTile<kW, U>::Ptr wp[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      if constexpr (kW == kBf16) {
        wp[m].w = slot_w(a, sw, a.w2, a.sw2) + wrow[m];
      } else if constexpr (kW == kFp8) {
        wp[m].w = slot_q(a, sw, a.q2) + wrow[m];
      } else {         // f / 2 code bytes of row rowm; its tiled scale row
        const size_t r = (size_t)sw.e * d + rowm[m];
        const int G = mx_granules(f);
        wp[m] = {a.q2 + r * (f / 2) + k0 / 2,
                 mx_row(a.e2 + (size_t)sw.e * d * G * 8, rowm[m], G), (int)k0};
      }
    }
    __shared__ __align__(16) uint16_t stage[Stage<U, true>::kElems];
    __shared__ int s_tok[kStageRows];
    const int R = min(8 * TL, te - c0);
    if (threadIdx.x < R) s_tok[threadIdx.x] = p0 + c0 + threadIdx.x;   // H rows
    __syncthreads();
    staged_pass<kW, U, true, NM, kRest, TL>(a.h + 2 * (size_t)blockIdx.z * Ks, 2 * (size_t)f,
                                            s_tok, R, wp, Ks, k_first, acc, stage);
#pragma unroll
    for (int rt = 0; rt < TL; ++rt) {
      if (rt >= nt) break;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        // lanes g = 0, 1 hold the hi rows of tokens 4g + i, lanes 32 above them the lo rows
        float v[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m)
          v[m] = (acc[m][rt][i] + __shfl_xor(acc[m][rt][i], 32, 64)) * sc[m];
        const int t = c0 + rt * 8 + 4 * g + i;
        if (g < 2 && t < te) {
          // routed rows go to their (token, slot) row, shared rows keep their own
          float* yrow = ypart + (size_t)(sw.shared ? p0 + t : a.perm[p0 + t]) * d;
#pragma unroll
          for (int m = 0; m < NM; ++m)
            if (n0 + 16 * m < d) yrow[n0 + 16 * m + n] = v[m];
        }
      }
    }
  }
  XS_TIME(xs_times_dn, 2 * block_id3() + 1, 2u * kTimeBlocks);
}

// ---- Persistent down GEMM, for launches of whole rounds with one block per CU (the
// seven-tile bf16 waves).  Such a launch runs its rounds in lock step: the blocks of a round
// stream the same bytes, so they end together, and every CU then spends the next block's
// start (dispatch, its slot record, then the first weight loads) with no reads in flight, at
// the same moment.  Here the grid holds one block per CU and each block walks a fixed list
// of work units: units b, b + G, b + 2G, ... (G blocks), a unit being one column block of
// one expert slot, taken in passes of up to 8 * TL token rows.  The block reads its units'
// slot records once, into LDS; the first step's loads of its next pass are issued in the
// last step of the current one, so a CU's weight stream does not drain between units.  The
// MFMAs always cover TL token tiles (one code path for every pass; rows past the pass repeat
// its last row and are not stored).  Units map to (slot, column block) as in down_kernel's
// grid, so with G a multiple of 8 every unit of a slot below 8 * (live / 8) runs on the XCD
// of that slot.  Blocks share nothing: no counters, no flags, no block waits for another.
constexpr int kSeqUnits = 32;     // units per block of a persistent launch, at most
static_assert(kTimeSeqStride == 1 + kSeqUnits, "a stamp per unit of a persistent block");

__device__ __forceinline__ void down_unit(int L, int CB, int live, bool xcd, int& slot, int& bx) {
  if (xcd && L < CB * (live & ~7)) {
    const int s = L >> 3;
    slot = (L & 7) + 8 * (s / CB);
    bx = s % CB;
  } else {
    slot = L / CB;
    bx = L % CB;
  }
}

// Lane state of one pass that its loads need: weight pointers, token pieces and the pass's
// first reduction step.
template <int kW, int U, int NM, int NLM>
struct DnLoads {
  typename WTile<kW, U>::Ptr wp[NM];
  const uint16_t* src[NLM];
  int wofs[NLM];
  int kb;
};

// A pass: unit record {expert | shared << 30, first permuted row, rows, column block} and
// the pass's first row.
struct DnPass {
  int4 rec;
  int c0;
  __device__ int e() const { return rec.x & 0x3FFFFFFF; }
  __device__ bool shared() const { return (rec.x >> 30) & 1; }
};

template <int kW, int U, int NM, int NLM, int TL>
__device__ __forceinline__ void dn_loads(const FfnArgs& a, const DnPass& ps, int wave, int n,
                                         size_t kl, int nsteps, int rot,
                                         DnLoads<kW, U, NM, NLM>& L) {
  using S = Stage<U, true>;
  const int d = a.d, f = a.f;
  const int bx = ps.rec.w, p0 = ps.rec.y, te = ps.rec.z;
  const int n0 = (bx * kWaves + wave) * kCols * NM;
  const size_t ebase = (size_t)ps.e() * d * f;
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    const size_t wrow = (size_t)(min(n0 + 16 * m, d - 16) + n) * f + kl;
    if constexpr (kW == kBf16) L.wp[m].w = (ps.shared() ? a.sw2 : a.w2) + ebase + wrow;
    else L.wp[m].w = a.q2 + ebase + wrow;
  }
  const int R = max(1, min(8 * TL, te - ps.c0));
#pragma unroll
  for (int i = 0; i < NLM; ++i) {
    const int q = min((int)threadIdx.x + i * kBlock, R * S::P - 1);
    const int row = q / S::P, piece = q % S::P;
    L.src[i] = a.h + (size_t)(p0 + ps.c0 + row) * 2 * f + piece * 8;
    L.wofs[i] = row * S::LS + piece * 8;
  }
  L.kb = ((bx * rot) % nsteps) * S::KB;
}

template <int U, int kW, int NM, int TL>
__global__ __attribute__((amdgpu_waves_per_eu(NM <= 4 ? XS_DOWN_WAVES_PER_EU : 1)))
__launch_bounds__(kBlock) void down_seq_kernel(FfnArgs a) {
  using S = Stage<U, true>;
  using WT = WTile<kW, U>;
  static_assert(kW != kMx4, "bf16 and FP8 weights");
  constexpr int KB = S::KB;
  constexpr int NLM = (TL * S::TR * S::P + kBlock - 1) / kBlock;
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int n = lane & 15, g = lane >> 4;
  const int d = a.d, f = a.f;
  const int CB = (d + kWaves * kCols * NM - 1) / (kWaves * kCols * NM);
  const int live = a.shared_slots + a.counters[kCntActive];
  const int units = live * CB;
  const int G = (int)gridDim.x;
  const int nu = (int)blockIdx.x < units ? min((units - (int)blockIdx.x + G - 1) / G, kSeqUnits) : 0;
  if (nu == 0) return;   // uniform: the whole block leaves before any barrier
  XS_TIME(xs_times_seq, blockIdx.x * kTimeSeqStride, (unsigned)(kTimeSeqBlocks * kTimeSeqStride));
  const bool xcd = a.max_active + a.shared_slots >= XS_DOWN_XCD_SLOTS;
  const int nsteps = f / KB;                    // unsplit: the launch takes one K part
  const int rot = kW == kBf16 ? XS_DOWN_ROT : XS_Q8_DOWN_ROT;
  const size_t kl = (size_t)(kW == kBf16 ? klane(g) : g * 8 * U);

  // the block's unit records, one thread each
  __shared__ int4 s_rec[kSeqUnits];
  if (tid < nu) {
    int slot, bx;
    down_unit((int)blockIdx.x + tid * G, CB, live, xcd, slot, bx);
    SlotWork sw;
    const bool ok = slot_work<kW>(a, slot, sw);   // slot < live: always work
    s_rec[tid] = ok ? make_int4(sw.e | (sw.shared ? 1 << 30 : 0), sw.p0, sw.te, bx)
                    : make_int4(0, 0, 0, bx);
  }
  __syncthreads();

  int j = 0;                                    // current unit
  DnPass cur{s_rec[0], 0};
  __shared__ __align__(16) uint16_t lds[S::kElems];
  DnLoads<kW, U, NM, NLM> L;
  dn_loads<kW, U, NM, NLM, TL>(a, cur, wave, n, kl, nsteps, rot, L);

  u32x4 v[NLM];
  typename WT::Regs b[NM];
#pragma unroll
  for (int i = 0; i < NLM; ++i) v[i] = *reinterpret_cast<const u32x4*>(L.src[i] + S::AS * L.kb);
#pragma unroll
  for (int m = 0; m < NM; ++m) b[m] = WT::load(L.wp[m], L.kb);
#pragma unroll
  for (int i = 0; i < NLM; ++i) *reinterpret_cast<u32x4*>(lds + L.wofs[i]) = v[i];
  __syncthreads();

  floatx4 acc[NM][TL];
#pragma unroll
  for (int m = 0; m < NM; ++m)
#pragma unroll
    for (int rt = 0; rt < TL; ++rt) acc[m][rt] = floatx4{0.f, 0.f, 0.f, 0.f};

  int buf = 0;
  // MFMAs of one step from LDS buffer `buf`: all TL tiles (rows past the pass repeat its last
  // row; their sums are not stored), so every pass runs the same code
  auto mfma_step = [&](const int (&rofs)[TL]) {
    const uint16_t* const cl = lds + buf * kStageRows * S::LS;
#pragma unroll
    for (int uu = 0; uu < U; ++uu) {
      const int ka = S::AS * WT::koff(g, uu);
      bf16x8 xa[TL];
#pragma unroll
      for (int rt = 0; rt < TL; ++rt) xa[rt] = *reinterpret_cast<const bf16x8*>(cl + rofs[rt] + ka);
#pragma unroll
      for (int rt = 0; rt < TL; ++rt)
#pragma unroll
        for (int m = 0; m < NM; ++m) acc[m][rt] = mfma(xa[rt], WT::operand(b[m], uu), acc[m][rt]);
    }
  };
  while (true) {
    const int te = cur.rec.z, p0 = cur.rec.y;
    const int R = max(1, min(8 * TL, te - cur.c0));
    const int nt = (R + 7) >> 3;
    const int n0 = (cur.rec.w * kWaves + wave) * kCols * NM;
    int rofs[TL];
#pragma unroll
    for (int rt = 0; rt < TL; ++rt) rofs[rt] = min(8 * rt + (n & 7), R - 1) * S::LS + (n & 8);
    // every step but the last: loads of the next step, MFMAs of this one
    for (int ks = 0; ks < nsteps - 1; ++ks) {
      int kn = L.kb + KB;
      if (kn >= f) kn -= f;
#pragma unroll
      for (int i = 0; i < NLM; ++i) v[i] = *reinterpret_cast<const u32x4*>(L.src[i] + S::AS * kn);
      typename WT::Regs nb[NM];
#pragma unroll
      for (int m = 0; m < NM; ++m) nb[m] = WT::load(L.wp[m], kn);
      mfma_step(rofs);
      uint16_t* const nl = lds + (buf ^ 1) * kStageRows * S::LS;
#pragma unroll
      for (int i = 0; i < NLM; ++i) *reinterpret_cast<u32x4*>(nl + L.wofs[i]) = v[i];
#pragma unroll
      for (int m = 0; m < NM; ++m) b[m] = nb[m];
      __syncthreads();
      buf ^= 1;
      L.kb = kn;
    }
    // the last step: the loads of the block's next pass (the unit's next rows, else its next
    // unit; after the block's last pass the same loads again), then this step's MFMAs and the
    // pass's epilogue
    DnPass nxt = cur;
    int jn = j;
    bool has_nxt = true;
    if (cur.c0 + 8 * TL < te) {
      nxt.c0 += 8 * TL;
    } else {
      jn = j + 1;
      has_nxt = jn < nu;
      if (has_nxt) nxt = DnPass{s_rec[jn], 0};
    }
    DnLoads<kW, U, NM, NLM> Ln = L;
    if (has_nxt) dn_loads<kW, U, NM, NLM, TL>(a, nxt, wave, n, kl, nsteps, rot, Ln);
    int yrow[TL][4];
#pragma unroll
    for (int rt = 0; rt < TL; ++rt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = max(0, min(cur.c0 + rt * 8 + 4 * (g & 1) + i, te - 1));
        yrow[rt][i] = cur.shared() ? p0 + t : a.perm[p0 + t];
      }
    float sc[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m)
      sc[m] = kW == kFp8 ? a.s2[(size_t)cur.e() * d + min(n0 + 16 * m, d - 16) + n] : 1.0f;
#pragma unroll
    for (int i = 0; i < NLM; ++i) v[i] = *reinterpret_cast<const u32x4*>(Ln.src[i] + S::AS * Ln.kb);
    typename WT::Regs nb[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) nb[m] = WT::load(Ln.wp[m], Ln.kb);
    mfma_step(rofs);
    // lanes g = 0, 1 hold the hi rows of tokens 4g + i, lanes 32 above them the lo rows;
    // routed rows go to their (token, slot) row, shared rows keep their own
#pragma unroll
    for (int rt = 0; rt < TL; ++rt) {
      if (rt >= nt) break;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float o[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m)
          o[m] = (acc[m][rt][i] + __shfl_xor(acc[m][rt][i], 32, 64)) * sc[m];
        const int t = cur.c0 + rt * 8 + 4 * g + i;
        if (g < 2 && t < te) {
          float* const yr = a.yslot + (size_t)yrow[rt][i] * d;
#pragma unroll
          for (int m = 0; m < NM; ++m)
            if (n0 + 16 * m < d) yr[n0 + 16 * m + n] = o[m];
        }
      }
    }
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int rt = 0; rt < TL; ++rt) acc[m][rt] = floatx4{0.f, 0.f, 0.f, 0.f};
    uint16_t* const nl = lds + (buf ^ 1) * kStageRows * S::LS;
#pragma unroll
    for (int i = 0; i < NLM; ++i) *reinterpret_cast<u32x4*>(nl + Ln.wofs[i]) = v[i];
#pragma unroll
    for (int m = 0; m < NM; ++m) b[m] = nb[m];
    __syncthreads();
    buf ^= 1;
    if (jn != j)
      XS_TIME(xs_times_seq, blockIdx.x * kTimeSeqStride + 1 + j,
              (unsigned)(kTimeSeqBlocks * kTimeSeqStride));
    if (!has_nxt) break;
    cur = nxt;
    j = jn;
    L = Ln;
  }
}

#include "ffn_wide.h"

// Sums the gate and up partials of hidden element c..c+3 of partial row `prow` in split
// order, then H[hrow] = silu(gate) * up as bf16 hi and lo.
__device__ __forceinline__ void finish_row(const FfnArgs& a, size_t prow, size_t hrow, int c) {
  const size_t plane = (size_t)a.part_rows * a.f;
  const size_t at = prow * a.f + c;
  float4 gs = *reinterpret_cast<const float4*>(a.gpart + at);
  float4 us = *reinterpret_cast<const float4*>(a.gpart + plane + at);
  for (int z = 1; z < a.gu_splits; ++z) {
    const float4 gz = *reinterpret_cast<const float4*>(a.gpart + 2 * z * plane + at);
    const float4 uz = *reinterpret_cast<const float4*>(a.gpart + (2 * z + 1) * plane + at);
    gs.x += gz.x; gs.y += gz.y; gs.z += gz.z; gs.w += gz.w;
    us.x += uz.x; us.y += uz.y; us.z += uz.z; us.w += uz.w;
  }
  store_hilo(a.h, hrow, c + 0, a.f, gs.x / (1.0f + __expf(-gs.x)) * us.x);
  store_hilo(a.h, hrow, c + 1, a.f, gs.y / (1.0f + __expf(-gs.y)) * us.y);
  store_hilo(a.h, hrow, c + 2, a.f, gs.z / (1.0f + __expf(-gs.z)) * us.z);
  store_hilo(a.h, hrow, c + 3, a.f, gs.w / (1.0f + __expf(-gs.w)) * us.w);
}

// Split gate/up reduction: H for every hidden row from its partials.  Block row y takes
// hidden rows y, y + gridDim.y, ... (the grid keeps at most 65535 rows); routed rows beyond
// the routed count, and rows whose expert the GEMMs did not cover (another GPU group's),
// are skipped.
__global__ __launch_bounds__(kBlock) void gate_up_finish_kernel(FfnArgs a) {
  const int c = (blockIdx.x * kBlock + threadIdx.x) * 4;
  if (c >= a.f) return;
  for (long p = blockIdx.y; p < a.rows; p += gridDim.y) {
    const bool shared_row = p >= (long)a.T * a.k;
    if (!shared_row && p >= a.offsets[a.N]) continue;
    if (!shared_row && a.local_group >= 0) {
      const int e = a.ids[a.perm[p]];
      if ((a.group ? a.group[e] : e / (a.N / a.G)) != a.local_group) continue;
    }
    finish_row(a, (size_t)p, (size_t)p, c);
  }
}

// The finish pass of the gate/up tail: block row y is partial row y of the tail's compact
// planes, token y % T of slot slot_base + y / T (at most T rows a slot: a token takes an
// expert once; a shared expert takes every token).
__global__ __launch_bounds__(kBlock) void gate_up_tail_finish_kernel(FfnArgs a) {
  SlotWork sw;
  if (!slot_work<kBf16>(a, a.slot_base + blockIdx.y / a.T, sw)) return;
  const int t = blockIdx.y % a.T;
  if (t >= sw.te) return;
  const int c = (blockIdx.x * kBlock + threadIdx.x) * 4;
  if (c >= a.f) return;
  finish_row(a, blockIdx.y, (size_t)(sw.p0 + t), c);
}

__global__ __launch_bounds__(kBlock) void combine_kernel(FfnArgs a) {
  const int i = blockIdx.y;
  const int c = (blockIdx.x * kBlock + threadIdx.x) * 4;
  if (c >= a.d) return;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  // kR ranks at a time: their ids, weights and rows are loaded together (the rows of the
  // ranks that turn out unused, empty slots and other GPU groups' experts, hold stale
  // values and are left out of the sums), so a group costs one round trip; the sums keep
  // rank order and, per rank, split order
  constexpr int kR = 8;
  for (int r0 = 0; r0 < a.k; r0 += kR) {
    int e[kR];
    float wr[kR];
    float4 v[kR];
#pragma unroll
    for (int j = 0; j < kR; ++j) {
      const bool in = r0 + j < a.k;
      e[j] = in ? a.ids[i * a.k + r0 + j] : -1;
      wr[j] = in ? a.w[i * a.k + r0 + j] : 0.0f;
      v[j] = *reinterpret_cast<const float4*>(a.yslot +
                                              (size_t)(i * a.k + min(r0 + j, a.k - 1)) * a.d + c);
    }
    bool use[kR];
#pragma unroll
    for (int j = 0; j < kR; ++j)
      use[j] = e[j] >= 0 &&   // another GPU group's terms of y_i are left out
               (a.local_group < 0 ||
                (a.group ? a.group[e[j]] : e[j] / (a.N / a.G)) == a.local_group);
    for (int s = 1; s < a.splits; ++s) {   // partial sums of a split reduction, in order
#pragma unroll
      for (int j = 0; j < kR; ++j) {
        if (!use[j]) continue;
        const float4 u = *reinterpret_cast<const float4*>(
            a.yslot + ((size_t)s * a.rows + i * a.k + r0 + j) * a.d + c);
        v[j].x += u.x;
        v[j].y += u.y;
        v[j].z += u.z;
        v[j].w += u.w;
      }
    }
#pragma unroll
    for (int j = 0; j < kR; ++j) {
      if (!use[j]) continue;
      acc[0] += wr[j] * v[j].x;
      acc[1] += wr[j] * v[j].y;
      acc[2] += wr[j] * v[j].z;
      acc[3] += wr[j] * v[j].w;
    }
  }
  for (int sh = 0; sh < a.n_shared; ++sh) {  // shared experts, weight 1, after the routed terms
    const size_t row = (size_t)a.T * a.k + (size_t)sh * a.T + i;
    float4 v = *reinterpret_cast<const float4*>(a.yslot + row * a.d + c);
    for (int s = 1; s < a.splits; ++s) {
      const float4 u = *reinterpret_cast<const float4*>(
          a.yslot + ((size_t)s * a.rows + row) * a.d + c);
      v.x += u.x;
      v.y += u.y;
      v.z += u.z;
      v.w += u.w;
    }
    acc[0] += v.x;
    acc[1] += v.y;
    acc[2] += v.z;
    acc[3] += v.w;
  }
  const uint32_t lo = (uint32_t)to_bf16(acc[0]) | ((uint32_t)to_bf16(acc[1]) << 16);
  const uint32_t hi = (uint32_t)to_bf16(acc[2]) | ((uint32_t)to_bf16(acc[3]) << 16);
  *reinterpret_cast<uint2*>(a.y + (size_t)i * a.d + c) = make_uint2(lo, hi);
}

// Router GEMM h = W_g x: each wave owns 16 router rows (experts) and part blockIdx.z of d,
// for the token tiles of blockIdx.y; fp32 results go to that part's plane.
template <int U>
__global__ __launch_bounds__(kBlock) void router_kernel(RouterArgs r) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int j0 = (blockIdx.x * kWaves + wave) * kCols;
  if (j0 >= r.N) return;
  const int n = lane & 15, g = lane >> 4;
  const int Kp = r.d / r.parts;
  const size_t k0 = (size_t)blockIdx.z * Kp + (size_t)klane(g);
  const uint16_t* const brow = r.wg + (size_t)min(j0 + n, r.N - 1) * r.d + k0;
  float* const out = r.planes + (size_t)blockIdx.z * r.T * r.N;
  for (int c0 = blockIdx.y * 16 * kTiles; c0 < r.T; c0 += gridDim.y * 16 * kTiles) {
    const int nt = min(kTiles, (r.T - c0 + 15) / 16);
    const uint16_t* arow[kTiles];
#pragma unroll
    for (int rt = 0; rt < kTiles; ++rt)
      arow[rt] = r.x + (size_t)min(c0 + rt * 16 + n, r.T - 1) * r.d + k0;
    floatx4 acc[kTiles];
#pragma unroll
    for (int rt = 0; rt < kTiles; ++rt) acc[rt] = floatx4{0.f, 0.f, 0.f, 0.f};
    wave_pass<U>(arow, nt, brow, Kp, acc);
#pragma unroll
    for (int rt = 0; rt < kTiles; ++rt) {
      if (rt >= nt) break;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = c0 + rt * 16 + 4 * g + i;
        if (t < r.T && j0 + n < r.N) out[(size_t)t * r.N + j0 + n] = acc[rt][i];
      }
    }
  }
}

// logits = sum of the router's part planes, in part order.
__global__ __launch_bounds__(kBlock) void router_sum_kernel(RouterArgs r) {
  const size_t idx = (size_t)blockIdx.x * kBlock + threadIdx.x;
  const size_t plane = (size_t)r.T * r.N;
  if (idx >= plane) return;
  float v = r.planes[idx];
  int z = 1;
  for (; z + 8 <= r.parts; z += 8) {   // eight loads in flight, then the adds in order
    float t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = r.planes[(z + u) * plane + idx];
#pragma unroll
    for (int u = 0; u < 8; ++u) v = v + t[u];
  }
  for (; z < r.parts; ++z) v = v + r.planes[z * plane + idx];
  r.logits[idx] = v;
}

// Column tiles per wave: two if the expected active blocks stay enough with them.
bool gu_two_tiles(const FfnArgs& a, int kW, unsigned splits) {
  const long min_blocks = kW == kMx4 ? XS_Q4_GU_CT2_MIN_BLOCKS : XS_GU_CT2_MIN_BLOCKS;
  return (long)((a.f + 2 * kWaves * kCols - 1) / (2 * kWaves * kCols)) *
             (a.est_active + a.shared_slots) * splits >= min_blocks;
}

// Blocks of the kernel that the GPU runs at once (0: unknown).  The callers keep the figure in
// `cached`, one per instance (one device type; callers on several threads may fill it at once).
template <typename K>
int resident_blocks(K kernel, std::atomic<int>& cached, int threads = kBlock) {
  int r = cached.load(std::memory_order_relaxed);
  if (r == 0) {
    int per_cu = 0, dev = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        per_cu <= 0)
      return 0;
    r = per_cu * cus;
    cached.store(r, std::memory_order_relaxed);
  }
  return r;
}

// An unsplit gate/up launch of grid (B, S): when its last round of blocks holds slots
// S_main .. S - 1 and under a quarter of the resident blocks, those slots run after the
// main launch, split `ts` ways along d (partials, then their finish pass).  Returns ts (1:
// no tail launch) and S_main.
template <int U>
int gu_tail_split(const FfnArgs& a, dim3 grid, int resident, int& s_main) {
  s_main = (int)grid.y;
  if (a.gu_tail_splits < 2 || a.slot_base != 0 || resident <= 0 || a.T <= 0) return 1;
  const long B = grid.x, S = grid.y;
  const long rounds = S * B / resident;
  if (rounds < 1) return 1;
  const long main_slots = rounds * resident / B;
  const long tail = S - main_slots;
  if (tail <= 0 || 4 * tail * B > resident || tail > XS_GU_TAIL_MAX_SLOTS) return 1;
  if (tail * a.T > 65535) return 1;                 // the finish pass's grid rows
  int ts = 1;
  while (2 * ts <= a.gu_tail_splits && a.d % (2 * ts * 32 * U) == 0 &&
         tail * B * 2 * ts <= resident)
    ts *= 2;
  if (ts < 2) return 1;
  s_main = (int)main_slots;
  return ts;
}

template <int U, int kW, int CT>
void launch_gu_tail(const FfnArgs& a, dim3 grid, int s_main, int ts, hipStream_t stream) {
  FfnArgs t = a;
  t.slot_base = s_main;
  t.gu_splits = ts;
  t.part_rows = (long)gu_tail_rows(a.T);     // compact planes: (slot - s_main) * T + t
  t.part_compact = 1;
  const int tail = (int)grid.y - s_main;
  const dim3 g(grid.x, tail, ts), block(kBlock);
  hipLaunchKernelGGL((gate_up_kernel<U, true, kW, CT, false>), g, block, 0, stream, t);
  const dim3 fg((a.f + kBlock * 4 - 1) / (kBlock * 4), tail * a.T);
  hipLaunchKernelGGL(gate_up_tail_finish_kernel, fg, block, 0, stream, t);
}

// The gate/up launch of one instance; an unsplit one with its last round's slots split off when
// that pays (see gu_tail_split; its parts are whole steps).
template <int U, int kW, int CT, bool kRest>
void launch_gu(const FfnArgs& a, dim3 grid, hipStream_t stream) {
  const dim3 block(kBlock);
  grid.x = (a.f + CT * kWaves * kCols - 1) / (CT * kWaves * kCols);
  if constexpr (kRest) {
    hipLaunchKernelGGL((gate_up_kernel<U, false, kW, CT, true>), grid, block, 0, stream, a);
  } else if (grid.z > 1) {
    hipLaunchKernelGGL((gate_up_kernel<U, true, kW, CT, false>), grid, block, 0, stream, a);
  } else {
    static std::atomic<int> resident{0};
    int s_main = (int)grid.y;
    const int ts = gu_tail_split<U>(
        a, grid, resident_blocks(gate_up_kernel<U, false, kW, CT, false>, resident), s_main);
    if (s_main > 0)
      hipLaunchKernelGGL((gate_up_kernel<U, false, kW, CT, false>), dim3(grid.x, s_main, 1), block,
                         0, stream, a);
    if (ts > 1) launch_gu_tail<U, kW, CT>(a, grid, s_main, ts, stream);
  }
}

// Steps for reductions that are no multiple of the full step, U groups of 32: half of it where it
// is whole (always in the parts of a split reduction, multiples of 128) and the partial-step
// instance would be slower.  MXFP4 at odd multiples of 128, layer us, partial-step instance ->
// whole half steps: d=4224 f=2944 T=4 139 -> 125, T=32 287 -> 256, d=5120 f=1664 195 -> 177.
constexpr int half_step(int U) { return U == 8 ? 4 : U; }
// Step of the partial-step instances: half for MXFP4 (its 8-word one spilled 80 registers).
template <int kW, int U>
constexpr int rest_step() { return kW == kMx4 ? half_step(U) : U; }

// bf16 one-tile launches at odd multiples of 128: whole half steps between one and two blocks a
// CU (there the CUs with two blocks set the time, and the half steps' three blocks would fit) of
// experts with two rows or more.  Gate/up us at d=4992, partial step -> whole half steps: f=768
// T=16 M=24 (288 blocks) 96 -> 89, f=1664 T=4 M=12 (312) 94 -> 89, M=16 (416) 100 -> 99; outside,
// f=768 M=12 (144) 43 -> 57, f=1664 T=4 M=20 (520) 145 -> 157, T=32 M=40 (1040) 247 -> 260.
template <int U>
bool gu_half_steps(const FfnArgs& a, int K) {
  if (K % (32 * half_step(U)) != 0 || a.est_active <= 0 || (long)a.T * a.k < 2L * a.est_active)
    return false;
  static std::atomic<int> cached{0};
  const long r = resident_blocks(gate_up_kernel<U, false, kBf16, 1, true>, cached);
  const long blocks =
      (long)((a.f + kWaves * kCols - 1) / (kWaves * kCols)) * (a.est_active + a.shared_slots);
  return 2 * blocks > r && blocks <= r;
}

template <int kW, int U, int CT>
void launch_gu_step(const FfnArgs& a, int K, dim3 grid, hipStream_t stream) {
  constexpr int H = half_step(U);
  if constexpr (kW == kBf16 && CT == 1) {
    if (K % (32 * U) != 0 && grid.z == 1 && gu_half_steps<U>(a, K)) {
      launch_gu<H, kW, CT, false>(a, grid, stream);
      return;
    }
  }
  if (K % (32 * U) == 0)
    launch_gu<U, kW, CT, false>(a, grid, stream);
  else if (grid.z > 1 || (kW == kMx4 && K % (32 * H) == 0))
    launch_gu<H, kW, CT, false>(a, grid, stream);
  else
    launch_gu<rest_step<kW, U>(), kW, CT, true>(a, grid, stream);
}

// U2 / U1: steps of two-tile and of one-tile launches for weight format kW, over reductions of K.
template <int kW, int U2, int U1>
void launch_gu_fmt(const FfnArgs& a, int K, dim3 grid, hipStream_t stream) {
  static_assert(half_step(U2) <= 4 && half_step(U1) <= 4, "whole in the parts of a split");
  if (gu_two_tiles(a, kW, grid.z)) launch_gu_step<kW, U2, 2>(a, K, grid, stream);
  else launch_gu_step<kW, U1, 1>(a, K, grid, stream);
}

// Blocks of a down instance that the GPU runs at once.
template <int U, int kW, int NM, bool kRest, int TL = XS_DOWN_TL>
int down_resident() {
  static std::atomic<int> cached{0};
  return resident_blocks(down_kernel<U, kW, NM, kRest, TL>, cached);
}

// The same of the instance for reductions of K.
template <int U, int kW, int NM>
int down_wide_resident(int K) {
  return K % (32 * U) == 0 ? down_resident<U, kW, NM, false>() : down_resident<U, kW, NM, true>();
}

template <int U, int kW, int NM, bool kRest, int TL>
void launch_down_step(const FfnArgs& a, hipStream_t stream) {
  const int cols = kWaves * kCols * NM;
  hipLaunchKernelGGL((down_kernel<U, kW, NM, kRest, TL>),
                     dim3((a.d + cols - 1) / cols, a.max_active + a.shared_slots, a.splits),
                     dim3(kBlock), 0, stream, a);
}
// FP8 with 32-row waves at odd multiples of 64: whole half steps (three blocks a CU) where they
// make one round of blocks and the partial-step instance (two) makes two.  Down us at d=2752,
// partial step -> whole half steps: f=832 T=16 M=24 (528 blocks) 20 -> 16, f=1472 T=8 M=32 (704)
// 37 -> 31; outside, f=1472 T=4 M=20 (440) 21 -> 23, T=16 M=40 (880) 41 -> 53.
template <int U, int NM>
bool down_half_steps(const FfnArgs& a, int K) {
  if (K % (16 * U) != 0 || a.est_active <= 0) return false;
  const int cols = kWaves * kCols * NM;
  const long blocks = (long)((a.d + cols - 1) / cols) * a.est_active * a.splits;
  return blocks > down_resident<U, kFp8, NM, true>() &&
         blocks <= down_resident<U / 2, kFp8, NM, false>();
}
// NM: rows per wave / 16; a reduction shorter than a partial-step instance's step takes kNarrow.
template <int U, int kW, int NM, int kNarrow, int TL = XS_DOWN_TL>
void launch_down_fmt(const FfnArgs& a, hipStream_t stream) {
  constexpr int H = half_step(U), kStep = rest_step<kW, U>();
  static_assert(kNarrow <= 2, "has the short case");
  const int K = a.f / a.splits;
  if constexpr (kW == kFp8 && NM == kNarrow) {
    if (K % (32 * U) != 0 && down_half_steps<U, NM>(a, K)) {
      launch_down_step<U / 2, kW, NM, false, TL>(a, stream);
      return;
    }
  }
  if (K % (32 * U) == 0) launch_down_step<U, kW, NM, false, TL>(a, stream);
  else if (K % (32 * H) == 0) launch_down_step<H, kW, NM, false, TL>(a, stream);
  else if (K > 32 * kStep) launch_down_step<kStep, kW, NM, true, TL>(a, stream);
  else launch_down_step<kStep, kW, kNarrow, true, XS_DOWN_TL>(a, stream);
}

// The persistent down launch (down_seq_kernel): one block per resident slot, rounded up to a
// multiple of 8 (one XCD per slot's units) and to at least the unit bound / kSeqUnits.
// False if the instance's residency is unknown.
template <int U, int kW, int NM, int TL = XS_DOWN_TL>
bool launch_down_seq(const FfnArgs& a, hipStream_t stream) {
  static std::atomic<int> cached{0};
  const int r = resident_blocks(down_seq_kernel<U, kW, NM, TL>, cached);
  if (r == 0) return false;
  const int CB = (a.d + kWaves * kCols * NM - 1) / (kWaves * kCols * NM);
  const long max_units = (long)(a.max_active + a.shared_slots) * CB;
  long G = std::max<long>(r, (max_units + kSeqUnits - 1) / kSeqUnits);
  G = (G + 7) & ~7L;
  hipLaunchKernelGGL((down_seq_kernel<U, kW, NM, TL>), dim3((unsigned)G), dim3(kBlock), 0, stream,
                     a);
  return true;
}

// Gate/up with 256 weight rows a block where that leaves at least 1024 blocks (bf16) or 512 (FP8
// and MXFP4, whose steps are twice as long then), else 128 (two blocks a CU).  Gate/up us with 256
// / 128 rows: bf16 Mixtral T=64 (560 blocks of 256) 251 / 221, DeepSeek T=64 M=24 (384) 275 / 253,
// T=256 M=64 (1264) 667 / 682, T=512 M=96 (2048) 1043 / 1057, Mixtral T=1024 (2577) 660 / 687; FP8
// DeepSeek T=64 M=32 (512) 171 / 187, M=24 (384) 147 / 172, T=256 M=64 356 / 397, Qwen T=256 (384)
// 63 / 59; MXFP4 Qwen T=256 (384) 53 / 48, Mixtral T=64 (560) 95 / 125, DeepSeek T=256 M=64 275 /
// 353.  One GPU group's share is taken for the slots of the whole batch's rows: DeepSeek T=512 FP8
// 115 / 93 and MXFP4 101 / 81 would run faster with 128 rows, but with its own slots at the same
// limits others lose (d=4096 f=4096 T=512 MXFP4 249 a layer with 256, 273 with 128).
struct WideGrid {
  int rows;              // weight rows of a gate/up block
  long gu, dn;           // blocks of the two launches with the slots expected
};
WideGrid wide_grid(const FfnArgs& a) {
  // slots, not experts: Mixtral T=1024 has 8 experts in about 20 slots
  const int act = a.est_active > 0 ? slot_bound(a.est_active, a.T, a.k) : a.max_active;
  const long est = std::min(act, a.max_active) + a.shared_slots;
  const long b256 = (long)((a.f + 127) / 128) * est * a.gu_splits;
  const long b128 = (long)((a.f + 63) / 64) * est * a.gu_splits;
  const bool big = b256 >= (a.wfmt == kBf16 ? 1024 : 512);
  return {big ? 256 : 128, big ? b256 : b128, (long)((a.d + 255) / 256) * est * a.splits};
}

// A grid of more than one and fewer than `rounds` rounds of blocks whose last round is at most
// three quarters full.
bool short_last_round(long blocks, long resident, int rounds) {
  if (resident <= 0 || blocks <= resident || blocks >= rounds * resident) return false;
  const long last = blocks % resident;
  return last != 0 && 4 * last <= 3 * resident;
}
template <int kW>
bool gu_wide_short_round(const WideGrid& w, int rounds) {
  static std::atomic<int> c256{0}, c128{0};
  return short_last_round(w.gu, w.rows == 256
                                    ? resident_blocks(gate_up_wide_kernel<kW, 256>, c256, 512)
                                    : resident_blocks(gate_up_wide_kernel<kW, 128>, c128, 256),
                          rounds);
}
template <int kW>
bool dn_wide_short_round(const WideGrid& w, int rounds) {
  static std::atomic<int> cached{0};
  return short_last_round(w.dn, resident_blocks(down_wide_kernel<kW, 256>, cached, 512), rounds);
}

// Launches for large batches (ffn_wide.h) where an expert holds 16 rows or more on average (24
// with MXFP4; 20 with bf16 up to 64 tokens) and the batch can give one more than 32, the rows of
// a pass of the staged launches.  Layer us, staged -> this: bf16 DeepSeek T=96 12 rows an expert
// 1016 -> 1048, T=128 16 rows 1176 -> 1069, Mixtral T=80 20 rows 762 -> 572; FP8 DeepSeek T=128 16
// rows 643 -> 579, d=2048 f=1408 T=64 M=30 12.8 rows 74 -> 81 (but d=5120 f=1536 T=64 10.7 rows
// 285 -> 267); MXFP4 DeepSeek T=128 16 rows 404 -> 463, d=5120 f=1536 T=256 26 rows 428 -> 372.
// With few passes to save, an uneven last round of this launch's larger blocks costs more than
// they do, and it takes more rows: FP8 19 up to 64 tokens with one to two rounds of gate/up blocks
// (d=3072 f=1536 k=8 T=64 M=32, 1.5 rounds, 123 -> 141, T=52 M=26 110 -> 131, d=1024 f=2048 T=36
// 16 rows 56 -> 63; at 19.6 rows 67 -> 64), MXFP4 28 below 128 tokens (Mixtral T=96 24 rows, 3.5
// rounds, 234 -> 263, T=112 28 rows 263 -> 266; d=5120 f=1536 T=96 24 rows, 1.5 rounds, 185 ->
// 213; d=4096 f=8192 T=64 26 rows 124 -> 136; in whole rounds T=96 24 rows 175 -> 158).
bool wide_batch(const FfnArgs& a) {
  if (a.T <= kStageRows) return false;
  // a group's share is expected to hold its part of the routed rows
  const long rows = (long)a.T * a.k / (a.local_group >= 0 ? a.G : 1) + (long)a.n_shared * a.T;
  const long experts = (a.est_active > 0 ? a.est_active : a.max_active) + a.n_shared;
  long least = a.wfmt == kBf16 && a.T <= 64 ? 20 : 16;
  if (a.wfmt == kFp8 && a.T <= 64 && gu_wide_short_round<kFp8>(wide_grid(a), 2)) least = 19;
  if (a.wfmt == kMx4) {
    const WideGrid w = wide_grid(a);
    const bool uneven = gu_wide_short_round<kMx4>(w, 4) ||
                        (a.splits == 1 && dn_wide_short_round<kMx4>(w, 2));
    least = a.T < 128 && uneven ? 28 : 24;
  }
  return rows >= least * experts;
}

template <int kW>
void launch_gu_wide(const FfnArgs& a, hipStream_t stream) {
  const unsigned slots = a.max_active + a.shared_slots;
  const int rows = wide_grid(a).rows, cols = rows / 2;
  const dim3 grid((a.f + cols - 1) / cols, slots, a.gu_splits);
  if (rows == 256)
    hipLaunchKernelGGL((gate_up_wide_kernel<kW, 256>), grid, dim3(512), 0, stream, a);
  else
    hipLaunchKernelGGL((gate_up_wide_kernel<kW, 128>), grid, dim3(256), 0, stream, a);
}
// Down always with 256 rows.  Down us with 128 / 256: DeepSeek T=256 M=64 FP8 295 / 237, T=512 FP8
// 527 / 396, Mixtral T=1024 bf16 741 / 563, Qwen T=1024 FP8 138 / 100; the other way Qwen T=256
// MXFP4 37 / 40, Mixtral T=64 bf16 130 / 136.
template <int kW>
void launch_dn_wide(const FfnArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL((down_wide_kernel<kW, 256>),
                     dim3((a.d + 255) / 256, a.max_active + a.shared_slots, a.splits), dim3(512), 0,
                     stream, a);
}

// Gate/up with the waves of a block splitting d (gate_up_narrow_kernel): where the grid would
// split d (few or small experts; its parts are multiples of 128, so d is one of 256) and no
// expert can hold more than one tile of 16 rows, 4 on average (each block reads its rows of x for
// 16 columns only).  FP8 takes it up to 1024 waves of 16 columns, where the grid no longer splits
// but has one block a CU: DeepSeek T=1 (8 experts) 101 -> 88 us a layer; past that it gains and
// loses with the shape (Mixtral T=1, 1792 waves, 84 -> 91, T=4, 4480 waves, 204 -> 179), bf16
// loses there (DeepSeek T=1 141 -> 145), and MXFP4 does by 15-60 %.
bool narrow_batch(const FfnArgs& a) {
  const bool few = a.gu_splits > 1 || (a.wfmt == kFp8 && (long)a.est_active * (a.f / 16) <= 1024);
  return few && a.T <= 16 && a.est_active > 0 && a.d % (32 * kWaves) == 0 &&
         (long)a.T * a.k <= 4L * a.est_active && a.n_shared == 0;
}
template <int U, int kW>
void launch_gu_narrow(const FfnArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL((gate_up_narrow_kernel<U, kW>),
                     dim3(a.f / kCols, a.max_active + a.shared_slots), dim3(kBlock), 0, stream, a);
}

}  // namespace

hipError_t launch_gate_up(const FfnArgs& a, hipStream_t stream) {
  if (narrow_batch(a)) {
    if (a.wfmt == kFp8) launch_gu_narrow<4, kFp8>(a, stream);
    else if (a.wfmt == kMx4) launch_gu_narrow<4, kMx4>(a, stream);
    else launch_gu_narrow<2, kBf16>(a, stream);
    return hipGetLastError();
  }
  const int cols = kWaves * kCols;            // one column tile per wave; launch_gu may take two
  const dim3 grid((a.f + cols - 1) / cols, a.max_active + a.shared_slots, a.gu_splits),
      block(kBlock);
  const int K = a.d / a.gu_splits;
  if (wide_batch(a)) {
    if (a.wfmt == kFp8) launch_gu_wide<kFp8>(a, stream);
    else if (a.wfmt == kMx4) launch_gu_wide<kMx4>(a, stream);
    else launch_gu_wide<kBf16>(a, stream);
  } else if (a.wfmt == kFp8)
    launch_gu_fmt<kFp8, XS_Q8_GATE_UP_U, XS_Q8_GATE_UP_U1>(a, K, grid, stream);
  else if (a.wfmt == kMx4)
    launch_gu_fmt<kMx4, XS_Q4_GATE_UP_U, XS_Q4_GATE_UP_U1>(a, K, grid, stream);
  else
    launch_gu_fmt<kBf16, XS_GATE_UP_U, XS_GATE_UP_U1>(a, K, grid, stream);
  if (a.gu_splits > 1) {
    const dim3 fgrid((a.f + kBlock * 4 - 1) / (kBlock * 4), (unsigned)std::min(a.rows, 65535L));
    hipLaunchKernelGGL(gate_up_finish_kernel, fgrid, block, 0, stream, a);
  }
  return hipGetLastError();
}

hipError_t launch_down(const FfnArgs& a, hipStream_t stream) {
  const int K = a.f / a.splits;
  const long est = a.est_active + a.shared_slots;
  if (wide_batch(a)) {
    if (a.wfmt == kFp8) launch_dn_wide<kFp8>(a, stream);
    else if (a.wfmt == kMx4) launch_dn_wide<kMx4>(a, stream);
    else launch_dn_wide<kBf16>(a, stream);
    return hipGetLastError();
  }
  if (a.wfmt == kMx4) {
    // twice the rows per wave (twice the weight bytes in flight) over 16-token passes, when
    // experts hold 8 rows or fewer on average (an expert past 16 rows reads its weights
    // once per pass) and the grid stays large.  Same-box A/B: DeepSeek T=32 M=48 down
    // 98.5 -> 93.6 us, speculative 135.6 -> 127.2 us; at T=8 (672 blocks) 50.6 -> 53.2 us.
    const int wcols = kWaves * kCols * 2 * XS_Q4_DOWN_NM;
    const bool wide = XS_Q4_DN_WIDE && est > 0 && (long)a.T * a.k <= 8 * est &&
                      (long)((a.d + wcols - 1) / wcols) * est * a.splits >= XS_DN_WIDE_MIN_BLOCKS;
    if (wide)
      launch_down_fmt<XS_Q4_DOWN_U, kMx4, 2 * XS_Q4_DOWN_NM, XS_Q4_DOWN_NM, 2>(a, stream);
    else
      launch_down_fmt<XS_Q4_DOWN_U, kMx4, XS_Q4_DOWN_NM, XS_Q4_DOWN_NM>(a, stream);
    return hipGetLastError();
  }
  // bf16 and FP8: twice the rows per wave (one token load feeding twice the weight tiles)
  // pays when experts hold several tokens each and the grid stays large, or fills whole
  // rounds of the blocks the GPU runs at once: the Qwen-MoE shape at M=64 (512 wide blocks,
  // one round) ran down 53.6 -> 45.8 us wide, while 672 wide blocks (DeepSeek T=32 M=24,
  // 1.3 rounds) ran 137 -> 158 us.
  const int nm = a.wfmt == kFp8 ? XS_Q8_DOWN_NM : XS_DOWN_NM;
  const long wide_blocks =
      (long)((a.d + kWaves * kCols * 2 * nm - 1) / (kWaves * kCols * 2 * nm)) * est * a.splits;
  bool wide = est > 0 && (long)a.T * a.k >= XS_DN_WIDE_TOKENS * est &&
              wide_blocks >= XS_DN_WIDE_MIN_BLOCKS;
  if (!wide && est > 0 && (long)a.T * a.k >= XS_DN_WIDE_TOKENS * est) {
    const int r = a.wfmt == kFp8 ? down_wide_resident<XS_Q8_DOWN_U, kFp8, 2 * XS_Q8_DOWN_NM>(K)
                                 : down_wide_resident<XS_DOWN_U, kBf16, 2 * XS_DOWN_NM>(K);
    wide = r > 0 && wide_blocks >= r && wide_blocks % r == 0;
  }
#if XS_DOWN_NM7
  // bf16: seven tiles per wave where that grid fills whole rounds (see XS_DOWN_NM7); not
  // for one GPU group's share, whose expected count (the group's experts under plain top-k)
  // overstates its live slots: the plain top-k share of DeepSeek T=32 (about 12 live of 32
  // slots) ran down 296 us with 64-row waves and 324 us with seven tiles
  if (a.wfmt == kBf16 && est > 0 && a.local_group < 0 && K % (32 * XS_DOWN_NM7_U) == 0 &&
      (long)a.T * a.k >= XS_DN_WIDE_TOKENS * est) {
    const long b7 = (long)((a.d + kWaves * kCols * 7 - 1) / (kWaves * kCols * 7)) * est * a.splits;
    const int r7 = down_resident<XS_DOWN_NM7_U, kBf16, 7, false>();
    if (r7 > 0 && b7 >= r7 && b7 % r7 == 0) {
#if XS_DOWN_SEQ
      if (a.splits == 1 && launch_down_seq<XS_DOWN_NM7_U, kBf16, 7>(a, stream))
        return hipGetLastError();
#endif
      launch_down_step<XS_DOWN_NM7_U, kBf16, 7, false, XS_DOWN_TL>(a, stream);
      return hipGetLastError();
    }
  }
#endif
  if (a.wfmt == kFp8) {
    if (wide)
      launch_down_fmt<XS_Q8_DOWN_U, kFp8, 2 * XS_Q8_DOWN_NM, XS_Q8_DOWN_NM>(a, stream);
    else
      launch_down_fmt<XS_Q8_DOWN_U, kFp8, XS_Q8_DOWN_NM, XS_Q8_DOWN_NM>(a, stream);
  } else {
    if (wide)
      launch_down_fmt<XS_DOWN_U, kBf16, 2 * XS_DOWN_NM, XS_DOWN_NM>(a, stream);
    else
      launch_down_fmt<XS_DOWN_U, kBf16, XS_DOWN_NM, XS_DOWN_NM>(a, stream);
  }
  return hipGetLastError();
}

hipError_t launch_router(const RouterArgs& r, hipStream_t stream) {
  const dim3 grid((r.N + kWaves * kCols - 1) / (kWaves * kCols), router_token_groups(r.T),
                  r.parts),
      block(kBlock);
  const int K = r.d / r.parts;
  if (K % 128 == 0) hipLaunchKernelGGL(router_kernel<4>, grid, block, 0, stream, r);
  else if (K % 64 == 0) hipLaunchKernelGGL(router_kernel<2>, grid, block, 0, stream, r);
  else hipLaunchKernelGGL(router_kernel<1>, grid, block, 0, stream, r);
  const size_t n = (size_t)r.T * r.N;
  hipLaunchKernelGGL(router_sum_kernel, dim3((unsigned)((n + kBlock - 1) / kBlock)), block, 0,
                     stream, r);
  return hipGetLastError();
}

// MXFP4 scales [n_mat, rows, K / 32] -> the tiled layout [n_mat, rows / 16, G, 16, 8] (G =
// ceil(K / 256)); bytes past the last block of a row are 127 (scale 1), never read.
__global__ __launch_bounds__(kBlock) void mx_scales_tile_kernel(const uint8_t* src, uint8_t* dst,
                                                                long total, int rows, int K) {
  const long i = (long)blockIdx.x * kBlock + threadIdx.x;
  if (i >= total) return;
  const int G = (K + 255) >> 8, nb = K >> 5;
  const long per_mat = (long)rows * G * 8;
  const long mat = i / per_mat;
  const int r = (int)(i % per_mat);
  const int tile = r / (G * 128), in_tile = r % (G * 128);
  const int gran = in_tile >> 7, row = tile * 16 + ((in_tile >> 3) & 15);
  const int c = gran * 8 + (in_tile & 7);
  dst[i] = c < nb ? src[(mat * rows + row) * nb + c] : (uint8_t)127;
}

hipError_t launch_mx_scales_tile(const uint8_t* src, uint8_t* dst, int n_mat, int rows, int K,
                                 hipStream_t stream) {
  const long total = (long)n_mat * rows * ((K + 255) / 256) * 8;
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(mx_scales_tile_kernel, dim3((unsigned)((total + kBlock - 1) / kBlock)),
                     dim3(kBlock), 0, stream, src, dst, total, rows, K);
  return hipGetLastError();
}

hipError_t launch_combine(const FfnArgs& a, hipStream_t stream) {
  const dim3 grid((a.d + kBlock * 4 - 1) / (kBlock * 4), a.T), block(kBlock);
  hipLaunchKernelGGL(combine_kernel, grid, block, 0, stream, a);
  return hipGetLastError();
}

}  // namespace xs

// The block timeline of the last gate/up, down and persistent down launches (a profiling
// build); XSHARE_EUNSUPPORTED in the product build.  With `clear` the stamps are zeroed after
// the copy (hipMemsetAsync: a measurement call, not for graph capture).
extern "C" xshare_status xshare_block_times(uint64_t* gate_up, uint64_t* down,
                                            uint64_t* down_units, int32_t clear,
                                            hipStream_t stream) {
#if XS_BLOCK_TIMES
  if (!gate_up || !down || !down_units) return XSHARE_EINVAL;
  void* src[3] = {nullptr, nullptr, nullptr};
  if (hipGetSymbolAddress(&src[0], HIP_SYMBOL(xs::xs_times_gu)) != hipSuccess ||
      hipGetSymbolAddress(&src[1], HIP_SYMBOL(xs::xs_times_dn)) != hipSuccess ||
      hipGetSymbolAddress(&src[2], HIP_SYMBOL(xs::xs_times_seq)) != hipSuccess)
    return XSHARE_EHIP;
  uint64_t* dst[3] = {gate_up, down, down_units};
  const size_t bytes[3] = {sizeof(xs::xs_times_gu), sizeof(xs::xs_times_dn),
                           sizeof(xs::xs_times_seq)};
  for (int i = 0; i < 3; ++i) {
    if (hipMemcpyAsync(dst[i], src[i], bytes[i], hipMemcpyDeviceToDevice, stream) != hipSuccess)
      return XSHARE_EHIP;
    if (clear && hipMemsetAsync(src[i], 0, bytes[i], stream) != hipSuccess) return XSHARE_EHIP;
  }
  return XSHARE_OK;
#else
  (void)gate_up;
  (void)down;
  (void)down_units;
  (void)clear;
  (void)stream;
  return XSHARE_EUNSUPPORTED;
#endif
}
