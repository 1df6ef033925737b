// Expert selection for one MoE layer and one decode batch (XShare, arXiv 2602.07265):
// router scoring, batch scores, greedy selection (flat Algorithm 2 or per-request +
// batch Algorithms 3-4), refinement, and the token permutation consumed by the expert
// GEMMs.  For decode-sized batches (one_group_tokens) one workgroup of 1024 threads does all of
// it: the whole problem is a few thousand logits and is latency-, not throughput-bound, so the
// kernel avoids LDS round trips in its inner loops: wave reductions use DPP, rankings compare
// packed integer keys, and a token bitmask per expert turns every per-expert gather into
// popcounts.  Larger batches run four kernels over the whole GPU (route_tokens_kernel and the
// ones after it).
//
// Numerics: this translation unit is compiled with -ffp-contract=off; every fp32 step
// of the gates is a separate IEEE round-to-nearest operation in a fixed order, so the
// selected set and the per-token routing are reproducible bit for bit.
#pragma clang fp contract(off)

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "internal.h"

namespace xs {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr uint32_t kNoEntry = 0xFFFFu;   // empty slot of the per-token lists
#ifndef XS_HEAVY_ROWS
#define XS_HEAVY_ROWS 8
#endif
constexpr int kHeavyRows = XS_HEAVY_ROWS;   // active-list class boundary (routed rows)

// exp(x) for x <= 0 in fp32: n = rint(x log2 e); r = (x - n ln2_hi) - n ln2_lo with a
// 15-bit ln2_hi (Cody-Waite: n ln2_hi is exact); p = degree-7 Taylor polynomial of e^r
// (coefficients 1/i!) in Horner form; result p * 2^n.  Below -80 the result is 0.
__device__ __forceinline__ float exp_fixed(float x) {
  constexpr float kLog2e = (float)1.4426950408889634;
  constexpr float kLn2Hi = 0.693145751953125f;
  constexpr float kLn2Lo = (float)(0.6931471805599453 - 0.693145751953125);
  constexpr float c2 = 0.5f;
  constexpr float c3 = (float)(1.0 / 6.0);
  constexpr float c4 = (float)(1.0 / 24.0);
  constexpr float c5 = (float)(1.0 / 120.0);
  constexpr float c6 = (float)(1.0 / 720.0);
  constexpr float c7 = (float)(1.0 / 5040.0);
  if (x < -80.0f) return 0.0f;
  const float n = rintf(x * kLog2e);
  const float r = (x - n * kLn2Hi) - n * kLn2Lo;
  float p = c7;
  p = p * r + c6;
  p = p * r + c5;
  p = p * r + c4;
  p = p * r + c3;
  p = p * r + c2;
  p = p * r + 1.0f;
  p = p * r + 1.0f;
  return ldexpf(p, (int)n);
}

// Order-preserving map of finite fp32 values to uint32 (> 0); 0 marks "no value".
__device__ __forceinline__ uint32_t ord(float h) {
  const uint32_t b = __float_as_uint(h);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float unord(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// One DPP step of a reduction: the value of the lane that Ctrl names, or the reduction's
// identity in rows outside RowMask.  With the identity as the "old" operand the compiler
// folds the move into the reducing instruction (one v_max_u32_dpp / v_min_u32_dpp per step
// instead of two moves and the max).
template <int Ctrl, int RowMask, uint32_t Identity>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)Identity, (int)v, Ctrl, RowMask, 0xF, false);
}

// Wave-wide max / min of a uint32 with DPP (quad swaps, row mirrors, row broadcasts);
// lane 63 ends with the result, which is returned to every lane.
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  v = max(v, dpp<0xB1, 0xF, 0u>(v));   // quad_perm [1,0,3,2]
  v = max(v, dpp<0x4E, 0xF, 0u>(v));   // quad_perm [2,3,0,1]
  v = max(v, dpp<0x141, 0xF, 0u>(v));  // row_half_mirror
  v = max(v, dpp<0x140, 0xF, 0u>(v));  // row_mirror
  v = max(v, dpp<0x142, 0xA, 0u>(v));  // row_bcast:15
  v = max(v, dpp<0x143, 0xC, 0u>(v));  // row_bcast:31
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
  constexpr uint32_t kId = 0xFFFFFFFFu;
  v = min(v, dpp<0xB1, 0xF, kId>(v));
  v = min(v, dpp<0x4E, 0xF, kId>(v));
  v = min(v, dpp<0x141, 0xF, kId>(v));
  v = min(v, dpp<0x140, 0xF, kId>(v));
  v = min(v, dpp<0x142, 0xA, kId>(v));
  v = min(v, dpp<0x143, 0xC, kId>(v));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

__device__ __forceinline__ float lane_value(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// One round of a wave-wide selection over keys held Q per lane (expert lane + 64 q):
// returns the expert with the largest key, lowest index on equal keys (key 0 = not
// available), removes it from its lane, and reports its key; -1 if nothing is left.
// A second (min-index) reduction over the holders of the largest key finds the expert.
template <int Q>
__device__ __forceinline__ int wave_pick(uint32_t (&key)[Q], int lane, uint32_t& kbest) {
  uint32_t bk = 0;
  uint32_t bj = 0xFFFFFFFFu;
#pragma unroll
  for (int q = 0; q < Q; ++q) {  // strict: the lower q (lower index) wins inside a lane
    const bool up = key[q] > bk;
    bk = up ? key[q] : bk;
    bj = up ? (uint32_t)(lane + 64 * q) : bj;
  }
  kbest = wave_max(bk);
  if (kbest == 0) return -1;
  // the lowest expert index among the holders of the largest key
  const uint32_t jmin = wave_min(bk == kbest ? bj : 0xFFFFFFFFu);
  // the holder lane drops the key: selects, not a branch around the holder lane
  const bool mine = (int)(jmin & 63) == lane;
  const int qsel = (int)(jmin >> 6);
#pragma unroll
  for (int q = 0; q < Q; ++q) key[q] = (mine && q == qsel) ? 0u : key[q];
  return (int)jmin;
}

// Ranks [r0, k) of the available keys; lane r receives rank r as (logit, expert), or
// (-inf, -1) if fewer are available.  Lanes below r0 keep what they hold.
template <int Q>
__device__ __forceinline__ void wave_topk(uint32_t (&key)[Q], int r0, int k, int lane,
                                          float& my_h, int& my_j) {
  if (lane >= r0) {
    my_h = -INFINITY;
    my_j = -1;
  }
  for (int r = r0; r < k; ++r) {
    uint32_t kb;
    const int jb = wave_pick<Q>(key, lane, kb);
    if (jb < 0) break;
    const bool at = lane == r;
    my_h = at ? unord(kb) : my_h;
    my_j = at ? jb : my_j;
  }
}

// Gates of the ranked list held by lanes 0..k-1: e_r = exp(h_r - h_0), Z summed in rank
// order, g_r = e_r / Z (correctly rounded division).
__device__ __forceinline__ float ranked_gate(float my_h, int lane, int k) {
  const float m = lane_value(my_h, 0);
  const float e = lane < k ? exp_fixed(my_h - m) : 0.0f;
  float z = 0.0f;
  for (int r = 0; r < k; ++r) z = z + lane_value(e, r);
  return lane < k ? e / z : 0.0f;
}

// ---- Two tokens per wave: each 32-lane half ranks its own token (lane l of half h holds
//      experts l, l + 32, ... of token 2p + h), so one chain of dependent reductions
//      serves two tokens.  Used where a token's experts fit 8 per lane (N <= 256).

// Max / min over each 32-lane half (lanes 0-31 and 32-63), returned to every lane: four
// DPP steps give every lane its 16-lane row's value, then the two rows of each half
// exchange (v_permlane16_swap pairs rows 0 and 1, and rows 2 and 3).
__device__ __forceinline__ uint32_t half_max(uint32_t v) {
  v = max(v, dpp<0xB1, 0xF, 0u>(v));   // quad_perm [1,0,3,2]
  v = max(v, dpp<0x4E, 0xF, 0u>(v));   // quad_perm [2,3,0,1]
  v = max(v, dpp<0x141, 0xF, 0u>(v));  // row_half_mirror
  v = max(v, dpp<0x140, 0xF, 0u>(v));  // row_mirror
  const auto s = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return max((uint32_t)s[0], (uint32_t)s[1]);
}
__device__ __forceinline__ uint32_t half_min(uint32_t v) {
  constexpr uint32_t kId = 0xFFFFFFFFu;
  v = min(v, dpp<0xB1, 0xF, kId>(v));
  v = min(v, dpp<0x4E, 0xF, kId>(v));
  v = min(v, dpp<0x141, 0xF, kId>(v));
  v = min(v, dpp<0x140, 0xF, kId>(v));
  const auto s = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return min((uint32_t)s[0], (uint32_t)s[1]);
}

// wave_pick for both halves at once: each half takes its largest key (lowest expert index
// on equal keys), drops it and returns its expert (-1 if the half has no key left or is
// not active this round); kbest receives the half's largest key.  sl: lane within the half.
template <int Q2>
__device__ __forceinline__ int half_pick(uint32_t (&key)[Q2], int sl, bool act,
                                         uint32_t& kbest) {
  uint32_t bk = 0;
  uint32_t bj = 0xFFFFFFFFu;
#pragma unroll
  for (int q = 0; q < Q2; ++q) {  // strict: the lower q (lower index) wins inside a lane
    const bool up = key[q] > bk;
    bk = up ? key[q] : bk;
    bj = up ? (uint32_t)(sl + 32 * q) : bj;
  }
  const uint32_t kb = half_max(bk);
  kbest = kb;
  const bool got = act && kb != 0;
  // the lowest expert index among the half's holders of the largest key
  const uint32_t jb = half_min(got && bk == kb ? bj : 0xFFFFFFFFu);
  const bool mine = got && (int)(jb & 31) == sl;
  const int qsel = (int)(jb >> 5);
#pragma unroll
  for (int q = 0; q < Q2; ++q) key[q] = (mine && q == qsel) ? 0u : key[q];
  return got ? (int)jb : -1;
}

// wave_topk for both halves: ranks [r0, k) of each half's keys (r0 uniform within a half);
// lane sl of a half receives rank sl as (logit, expert).  Lanes below r0 keep what they hold.
template <int Q2>
__device__ __forceinline__ void half_topk(uint32_t (&key)[Q2], int r0, int k, int sl, int h,
                                          float& my_h, int& my_j) {
  if (sl >= r0) {
    my_h = -INFINITY;
    my_j = -1;
  }
  const int rs = min(__builtin_amdgcn_readlane(r0, 0), __builtin_amdgcn_readlane(r0, 32));
  for (int r = rs; r < k; ++r) {
    uint32_t kb;
    const int jb = half_pick<Q2>(key, sl, r >= r0, kb);
    const bool at = jb >= 0 && sl == r;
    my_h = at ? unord(kb) : my_h;
    my_j = at ? jb : my_j;
  }
}

// ranked_gate for both halves: e_r = exp(h_r - h_0), Z summed in rank order, g_r = e_r / Z.
__device__ __forceinline__ float half_gate(float my_h, int sl, int h, int k) {
  const float m = h ? lane_value(my_h, 32) : lane_value(my_h, 0);
  const float e = sl < k ? exp_fixed(my_h - m) : 0.0f;
  float z0 = 0.0f, z1 = 0.0f;
  for (int r = 0; r < k; ++r) {
    z0 = z0 + lane_value(e, r);
    z1 = z1 + lane_value(e, 32 + r);
  }
  const float z = h ? z1 : z0;
  return sl < k ? e / z : 0.0f;
}

// ---- Four tokens per wave: each 16-lane row ranks its own token (lane l of row r holds
//      experts l, l + 16, ... of token 4p + r).  Used where a token's experts fit 8 per lane
//      (N <= 128) and its k ranks fit in a row (k <= 16).

// Max / min over each 16-lane row, returned to every lane of the row (the first four steps
// of half_max).
__device__ __forceinline__ uint32_t row_max(uint32_t v) {
  v = max(v, dpp<0xB1, 0xF, 0u>(v));   // quad_perm [1,0,3,2]
  v = max(v, dpp<0x4E, 0xF, 0u>(v));   // quad_perm [2,3,0,1]
  v = max(v, dpp<0x141, 0xF, 0u>(v));  // row_half_mirror
  v = max(v, dpp<0x140, 0xF, 0u>(v));  // row_mirror
  return v;
}
__device__ __forceinline__ uint32_t row_min(uint32_t v) {
  constexpr uint32_t kId = 0xFFFFFFFFu;
  v = min(v, dpp<0xB1, 0xF, kId>(v));
  v = min(v, dpp<0x4E, 0xF, kId>(v));
  v = min(v, dpp<0x141, 0xF, kId>(v));
  v = min(v, dpp<0x140, 0xF, kId>(v));
  return v;
}

// The value of `v` in lane 16 r + c for this lane's row r (c uniform).
__device__ __forceinline__ int row_lane(int v, int r, int c) {
  const int v0 = __builtin_amdgcn_readlane(v, c);
  const int v1 = __builtin_amdgcn_readlane(v, 16 + c);
  const int v2 = __builtin_amdgcn_readlane(v, 32 + c);
  const int v3 = __builtin_amdgcn_readlane(v, 48 + c);
  return r < 2 ? (r == 0 ? v0 : v1) : (r == 2 ? v2 : v3);
}

// wave_pick for the four rows at once: each row takes its largest key (lowest expert index
// on equal keys), drops it and returns its expert (-1 if the row has no key left or is not
// active this round); kbest receives the row's largest key.  ql: lane within the row.
template <int Q4>
__device__ __forceinline__ int row_pick(uint32_t (&key)[Q4], int ql, bool act, uint32_t& kbest) {
  uint32_t bk = 0;
  uint32_t bj = 0xFFFFFFFFu;
#pragma unroll
  for (int q = 0; q < Q4; ++q) {  // strict: the lower q (lower index) wins inside a lane
    const bool up = key[q] > bk;
    bk = up ? key[q] : bk;
    bj = up ? (uint32_t)(ql + 16 * q) : bj;
  }
  const uint32_t kb = row_max(bk);
  kbest = kb;
  const bool got = act && kb != 0;
  // the lowest expert index among the row's holders of the largest key: a second row
  // reduction, cheaper than a ballot and a lane read per row
  const uint32_t jb = row_min(got && bk == kb ? bj : 0xFFFFFFFFu);
  const bool mine = got && (int)(jb & 15) == ql;
  const int qsel = (int)(jb >> 4);
#pragma unroll
  for (int q = 0; q < Q4; ++q) key[q] = (mine && q == qsel) ? 0u : key[q];
  return got ? (int)jb : -1;
}

// wave_topk for the four rows: ranks [r0, k) of each row's keys (r0 uniform within a row);
// lane ql of a row receives rank ql as (logit, expert).  Lanes below r0 keep what they hold.
template <int Q4>
__device__ __forceinline__ void row_topk(uint32_t (&key)[Q4], int r0, int k, int ql, int qr,
                                         float& my_h, int& my_j) {
  if (ql >= r0) {
    my_h = -INFINITY;
    my_j = -1;
  }
  const int rs = min(min(__builtin_amdgcn_readlane(r0, 0), __builtin_amdgcn_readlane(r0, 16)),
                     min(__builtin_amdgcn_readlane(r0, 32), __builtin_amdgcn_readlane(r0, 48)));
  for (int r = rs; r < k; ++r) {
    uint32_t kb;
    const int jb = row_pick<Q4>(key, ql, r >= r0, kb);
    const bool at = jb >= 0 && ql == r;
    my_h = at ? unord(kb) : my_h;
    my_j = at ? jb : my_j;
  }
}

// ranked_gate for the four rows: e_r = exp(h_r - h_0), Z summed in rank order, g_r = e_r / Z.
__device__ __forceinline__ float row_gate(float my_h, int ql, int qr, int k) {
  const float m = __int_as_float(row_lane(__float_as_int(my_h), qr, 0));
  const float e = ql < k ? exp_fixed(my_h - m) : 0.0f;
  float z0 = 0.0f, z1 = 0.0f, z2 = 0.0f, z3 = 0.0f;
  for (int r = 0; r < k; ++r) {
    z0 = z0 + lane_value(e, r);
    z1 = z1 + lane_value(e, 16 + r);
    z2 = z2 + lane_value(e, 32 + r);
    z3 = z3 + lane_value(e, 48 + r);
  }
  const float z = qr < 2 ? (qr == 0 ? z0 : z1) : (qr == 2 ? z2 : z3);
  return ql < k ? e / z : 0.0f;
}

// Raw logits of token quad p: lane ql of row qr holds experts ql, ql + 16, ... of token
// 4p + qr (0 beyond the batch or beyond N).
template <int Q4>
__device__ __forceinline__ void load_quad(const RouteArgs& a, int p, int ql, int qr,
                                          float (&raw)[Q4]) {
  const int i = 4 * p + qr;
  const size_t row = (size_t)i * a.N;
#pragma unroll
  for (int q = 0; q < Q4; ++q) {
    const int j = ql + 16 * q;
    raw[q] = (i < a.T && j < a.N) ? a.logits[row + j] : 0.0f;
  }
}

// Raw logits of token pair p: lane sl of half h holds experts sl, sl + 32, ... of token
// 2p + h (0 beyond the batch or beyond N).
template <int Q2>
__device__ __forceinline__ void load_pair(const RouteArgs& a, int p, int sl, int h,
                                          float (&raw)[Q2]) {
  const int i = 2 * p + h;
  const size_t row = (size_t)i * a.N;
#pragma unroll
  for (int q = 0; q < Q2; ++q) {
    const int j = sl + 32 * q;
    raw[q] = (i < a.T && j < a.N) ? a.logits[row + j] : 0.0f;
  }
}

// Raw logits of token i, lane l holding experts l, l + 64, ...
template <int Q>
__device__ __forceinline__ void load_row(const RouteArgs& a, int i, int lane, float (&raw)[Q]) {
  const size_t row = (size_t)i * a.N;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int j = lane + 64 * q;
    raw[q] = j < a.N ? a.logits[row + j] : 0.0f;
  }
}

// Canonicalised logits (h + 0.0 maps -0.0 to +0.0) and their keys.
template <int Q>
__device__ __forceinline__ void row_keys(const float (&raw)[Q], int N, int lane, float (&v)[Q],
                                         uint32_t (&key)[Q]) {
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int j = lane + 64 * q;
    v[q] = raw[q] + 0.0f;
    key[q] = j < N ? ord(v[q]) : 0u;
  }
}

template <int Q>
__device__ __forceinline__ void copy_keys(uint32_t (&dst)[Q], const uint32_t (&src)[Q]) {
#pragma unroll
  for (int q = 0; q < Q; ++q) dst[q] = src[q];
}

// Wave-wide inclusive prefix sum with DPP: shifts by 1, 2, 4 and 8 lanes inside each row
// of 16 (lanes without a source add 0), then each row's total added to the rows above it
// (row_bcast:15 into rows 1 and 3, row_bcast:31 into rows 2 and 3).
__device__ __forceinline__ int wave_incl_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return v;
}

// Block-wide exclusive prefix sum of one int per thread; every thread must call it.
__device__ int block_excl_scan(int v, int* s_wsum, int& total) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int inc = wave_incl_scan(v);
  if (lane == 63) s_wsum[wave] = inc;
  __syncthreads();
  int pre = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const int t = s_wsum[w];
    if (w < wave) pre += t;
    total += t;
  }
  __syncthreads();
  return pre + inc - v;
}

// Per-token list entry: bits 0-9 expert, bits 10-14 rank; kNoEntry = empty.

// Tokens of the one-workgroup selection (route_kernel), at most; one_group_tokens says which
// batches take it.  One token bitmask per expert turns the per-expert gathers (scores,
// per-request scores, permutation) into popcounts, and the keys of a wave's tokens stay in
// registers from the top-k to the refinement.  kFew: the instances for more tokens of at most
// kFewRanks ranks each, whose rankings are short (no dense scores).
constexpr int kFewRanks = 4;
template <int Q, bool kFew>
constexpr int max_tokens() {
  if (kFew) return Q == 1 ? 128 : Q == 2 ? 112 : Q == 4 ? 72 : Q == 8 ? 52 : 32;
  return Q <= 2 ? 64 : Q == 4 ? 40 : Q == 8 ? 24 : 16;
}
static_assert(max_tokens<1, true>() <= kSlotRows, "one slot holds all rows of an expert");

// Batches of up to this many tokens take the one-workgroup selection: one launch, where the four
// kernels need four and at least 15 us, but serial work that grows with T, k and N.  Measured, us
// a call, one workgroup / four kernels, queued behind other GPU work and then in a stream of
// selection calls alone (where four launches cost the host 24 us):
//   N=64   k=1 T=128 16 / 16, 17 / 24   k=4 T=80 18 / 18, 17 / 24   T=112 22 / 18, 19 / 24
//   N=128  k=1 T=112 17 / 16, 17 / 24   k=4 T=64 18 / 18, 17 / 24   T=80 21 / 19, 18 / 24
//          k=6 T=64 20 / 20, 19 / 24    k=8 T=64 23 / 21, 21 / 24
//   N=256  k=1 T=72 19 / 17, 17 / 24    k=2 T=56 18 / 18, 17 / 24   T=64 21 / 18, 19 / 24
//          k=6 T=40 22 / 21, 20 / 24    16 requests of 4, k=2: 23 / 19, 21 / 25
//   N=512  k=1 T=48 19 / 20, 18 / 24    k=4 T=33 23 / 22, 21 / 24   k=8 T=28 27 / 26, 25 / 24
//   N=1024 k=1 T=32 24 / 23, 22 / 23    k=4 T=20 28 / 28, 25 / 25   k=8 T=16 27 / 27, 25 / 25
// Picks per request add to the serial work like two more ranks.  Dense scores (a sum over all
// experts in order) are slower in one workgroup from 40 tokens on.
template <int Q>
int one_group_tokens(const RouteArgs& a) {
  const bool dense = a.score_mode == 1;
  const int k = a.k + (a.req_offsets && a.m_r > 0 ? 2 : 0);
  if (dense || k > kFewRanks) return Q == 2 && (dense || k > 6) ? 56 : max_tokens<Q, false>();
  constexpr int kStep = Q == 1 ? 12 : Q == 2 ? 16 : Q == 4 ? 12 : Q == 8 ? 8 : 4;
  return std::max(max_tokens<Q, true>() - kStep * (k - 1), max_tokens<Q, false>());
}

__device__ __forceinline__ uint64_t below(int i) { return i >= 64 ? ~0ull : ((1ull << i) - 1ull); }

// A set of tokens, kW words.
template <int kW>
struct TokenMask {
  uint64_t w[kW];
  __device__ void add(int i) {
    atomicOr(reinterpret_cast<unsigned long long*>(&w[kW > 1 ? i >> 6 : 0]), 1ull << (i & 63));
  }
  __device__ int count() const {
    int c = __popcll(w[0]);
    if constexpr (kW > 1) c += __popcll(w[1]);
    return c;
  }
  __device__ int count_below(int i) const {       // 0 <= i <= 64 kW
    int c = __popcll(w[0] & below(i));
    if constexpr (kW > 1) c += __popcll(w[1] & below(max(i - 64, 0)));
    return c;
  }
};

// Groups the entries by expert (ascending), tokens ascending inside: s_off[e] is the start
// of expert e's run in s_list, which holds entry indices p = i * k + r.  Needs s_occ zeroed;
// every thread must call.  Returns this thread's expert count (j = tid < N).
template <int kW>
__device__ int group_by_expert(const uint16_t* s_ent, TokenMask<kW>* s_occ, int* s_off,
                               uint16_t* s_list, int* s_wsum, int TK, int k, int N, int& total) {
  const int tid = threadIdx.x;
  for (int p = tid; p < TK; p += kThreads) {
    const uint32_t ent = s_ent[p];
    if (ent != kNoEntry) s_occ[ent & 1023u].add(p / k);
  }
  __syncthreads();
  const int cnt = tid < N ? s_occ[tid].count() : 0;
  const int off = block_excl_scan(cnt, s_wsum, total);
  if (tid < N) s_off[tid] = off;
  if (tid == N - 1) s_off[N] = off + cnt;
  __syncthreads();
  for (int p = tid; p < TK; p += kThreads) {
    const uint32_t ent = s_ent[p];
    if (ent == kNoEntry) continue;
    const int e = (int)(ent & 1023u);
    s_list[s_off[e] + s_occ[e].count_below(p / k)] = (uint16_t)p;
  }
  __syncthreads();
  return cnt;
}

// Tables of the greedy in LDS, one entry per expert (and a few block counters, zeroed by the
// caller with the tables).
struct GreedyTables {
  __align__(16) uint64_t key[kMaxExperts];   // keys of the candidates
  // GPU groups: warm-up experts per group, then |S| per group
  int gload[kMaxExperts];
  // GPU groups: candidates per group outside the warm-up set; threshold rule: scores by index
  __align__(16) int gcand[kMaxExperts];
  // GPU groups: takeable candidates per rank inside their group; threshold rule: scores by rank
  __align__(16) int hist[kMaxExperts];
  int wsum[kWaves];
  int cnt[8];
};

// The batch greedy (Algorithm 1 with a fixed budget; Algorithm 4's final stage; Algorithms 5
// and 6 with GPU groups) for expert j = threadIdx.x: whether it is selected.  Order (tier,
// score desc, index asc), keep the first budget_eff candidates.  Key: (3 - tier) << 42 |
// ord(score) << 10 | (1023 - j); candidates are compacted and each counts the candidates ahead
// of it.  Every thread of the block calls; MaxLoad(S) ends in sh.cnt[0] behind the caller's
// next barrier.
__device__ __forceinline__ bool select_set(const RouteArgs& a, GreedyTables& sh, bool tier1,
                                           float s, bool inU, bool inS0, int& n_s0, int& n_start,
                                           int& n_u, int& m_eff) {
  const int tid = threadIdx.x, j = tid;
  const int T = a.T, N = a.N, k = a.k;
  const bool dense = a.score_mode == 1;
  bool sel = false;
  if (a.G == 0) {
    int tier = 3;
    uint64_t mykey = 0;
    if (j < N) {
      const bool cand = dense ? (T > 0) : inU;
      tier = inS0 ? 0 : (tier1 ? 1 : (cand ? 2 : 3));
      if (tier < 3)
        mykey = ((uint64_t)(3 - tier) << 42) | ((uint64_t)ord(s) << 10) | (uint64_t)(1023 - j);
      if (tier == 0) atomicAdd(&sh.cnt[1], 1);
      if (tier <= 1) atomicAdd(&sh.cnt[2], 1);
      if (inU) atomicAdd(&sh.cnt[3], 1);
    }
    int n_cand = 0;
    const int cpos = block_excl_scan(mykey != 0 ? 1 : 0, sh.wsum, n_cand);
    if (mykey != 0) sh.key[cpos] = mykey;
    if (tid == 0 && (n_cand & 1)) sh.key[n_cand] = 0;
    __syncthreads();
    n_s0 = sh.cnt[1];
    n_start = sh.cnt[2];
    n_u = sh.cnt[3];
    int rank = 0;
    if (mykey != 0) {
      const ulonglong2* keys2 = reinterpret_cast<const ulonglong2*>(sh.key);
      const int n2 = (n_cand + 1) >> 1;
      for (int jj = 0; jj < n2; ++jj) {
        const ulonglong2 kk = keys2[jj];
        rank += (kk.x > mykey) + (kk.y > mykey);
      }
    }
    if (a.budget_mode == 3) {
      // Algorithm 1's threshold rule: the starting set (ranks below n_start) and then the
      // candidates in rank order join while f(S) < tau * f(E).  One thread replays the fp32
      // sums in the stated order: f(E) over every expert in index order, f(S) in rank order.
      float* const by_index = reinterpret_cast<float*>(sh.gcand);
      float* const by_rank = reinterpret_cast<float*>(sh.hist);
      if (j < N) by_index[j] = s;
      if (j >= N && j < ((N + 3) & ~3)) by_index[j] = 0.0f;   // pad to whole float4s
      if (mykey != 0) by_rank[rank] = s;
      __syncthreads();
      if (tid == 0) {
        // sequential fp32 sums; 16-byte LDS reads keep the loads ahead of the adds
        const float4* e4 = reinterpret_cast<const float4*>(by_index);
        float f_E = 0.0f;
#pragma unroll 4
        for (int q = 0; q < (N + 3) / 4; ++q) {
          const float4 v = e4[q];
          f_E = f_E + v.x;
          f_E = f_E + v.y;
          f_E = f_E + v.z;
          f_E = f_E + v.w;
        }
        const float target = a.tau * f_E;
        float f_S = 0.0f;
        for (int r = 0; r < n_start; ++r) f_S = f_S + by_rank[r];
        int m = n_start;
        while (m < n_cand && f_S < target) f_S = f_S + by_rank[m++];
        sh.cnt[6] = m;
      }
      __syncthreads();
      m_eff = max(sh.cnt[6], min(k, n_cand));
    } else {
      const int base = a.budget_mode == 0 ? a.budget : n_start + a.budget;
      m_eff = max(min(base, n_cand), min(k, n_cand));
    }
    sel = mykey != 0 && rank < m_eff;
  } else {
    // GPU groups (Algorithms 5 and 6).  Group g can take a_g = m_g - |S_0 on g| experts
    // (m_g caps every group's load, Eq. (5)), one per round, best first; its candidate of
    // rank r (score desc, index asc, among its candidates outside S_0) is taken in round
    // r + 1 if r < a_g.  The loop stops after the fewest rounds R that bring |S| to m_g * G,
    // or when no group can take more; so S = S_0 plus every takeable candidate of rank < R,
    // and R follows from a prefix count of the takeable candidates by rank.
    const int G = a.G, m_g = a.budget;
    const int gj = j < N ? (a.group ? a.group[j] : j / (N / G)) : 0;
    const bool cand = j < N && (dense ? (T > 0) : inU);
    const bool pick = cand && !inS0;
    if (j < N) {
      if (inS0) {
        atomicAdd(&sh.gload[gj], 1);
        atomicAdd(&sh.cnt[1], 1);
      }
      if (pick) atomicAdd(&sh.gcand[gj], 1);
      if (inU) atomicAdd(&sh.cnt[3], 1);
      if (cand) atomicAdd(&sh.cnt[5], 1);
    }
    // key: group << 44 | ord(score) << 10 | (1023 - j); the rank counts the group's keys above
    const uint64_t pkey =
        pick ? ((uint64_t)gj << 44) | ((uint64_t)ord(s) << 10) | (uint64_t)(1023 - j) : 0;
    int n_pick = 0;
    const int ppos = block_excl_scan(pick ? 1 : 0, sh.wsum, n_pick);
    if (pick) sh.key[ppos] = pkey;
    if (tid == 0 && (n_pick & 1)) sh.key[n_pick] = 0;
    __syncthreads();
    int rank = 0;
    bool takeable = false;
    if (pick) {
      const ulonglong2* keys2 = reinterpret_cast<const ulonglong2*>(sh.key);
      const uint64_t mine = (uint64_t)gj;
      const int n2 = (n_pick + 1) >> 1;
      for (int jj = 0; jj < n2; ++jj) {
        const ulonglong2 kk = keys2[jj];
        rank += ((kk.x >> 44) == mine && kk.x > pkey) + ((kk.y >> 44) == mine && kk.y > pkey);
      }
      takeable = rank < m_g - sh.gload[gj];
      if (takeable) atomicAdd(&sh.hist[rank], 1);
    }
    __syncthreads();
    n_s0 = sh.cnt[1];
    n_u = sh.cnt[3];
    const int n_cand = sh.cnt[5];
    const int need = m_g * G - n_s0;          // picks the rounds must reach
    static_assert(kThreads == kMaxExperts, "one rank of sh.hist per thread");
    const int at_rank = sh.hist[tid];
    int n_take = 0;
    const int before = block_excl_scan(at_rank, sh.wsum, n_take);
    if (need > 0 && before < need && before + at_rank >= need) sh.cnt[6] = tid + 1;
    __syncthreads();
    const int rounds = need <= 0 ? 0 : (n_take < need ? kMaxExperts : sh.cnt[6]);
    sel = inS0 || (takeable && rank < rounds);
    if (sel) atomicAdd(&sh.cnt[2], 1);
    __syncthreads();
    // fewer than k experts: the best remaining candidates join regardless of group
    const int n_loop = sh.cnt[2], want = min(k, n_cand);
    if (n_loop < want) {
      const bool rest = cand && !sel;
      const uint64_t fkey = rest ? ((uint64_t)ord(s) << 10) | (uint64_t)(1023 - j) : 0;
      int n_rest = 0;
      const int fpos = block_excl_scan(rest ? 1 : 0, sh.wsum, n_rest);
      if (rest) sh.key[fpos] = fkey;
      if (tid == 0 && (n_rest & 1)) sh.key[n_rest] = 0;
      __syncthreads();
      if (rest) {
        const ulonglong2* keys2 = reinterpret_cast<const ulonglong2*>(sh.key);
        int r2 = 0;
        const int n2 = (n_rest + 1) >> 1;
        for (int jj = 0; jj < n2; ++jj) {
          const ulonglong2 kk = keys2[jj];
          r2 += (kk.x > fkey) + (kk.y > fkey);
        }
        sel = r2 < want - n_loop;
      }
    }
    // Load_g(S) and MaxLoad(S) (Section 5.1)
    if (tid < G) sh.gload[tid] = 0;
    __syncthreads();
    if (sel) atomicAdd(&sh.gload[gj], 1);
    __syncthreads();
    if (tid < G) {
      if (a.group_load && blockIdx.x == 0) a.group_load[tid] = sh.gload[tid];
      atomicMax(&sh.cnt[0], sh.gload[tid]);
    }
    n_start = n_s0;
    m_eff = min(m_g * G, N);
  }
  return sel;
}

template <int Q, bool kFew>
__global__ __launch_bounds__(kThreads) void route_kernel(RouteArgs a) {
  constexpr int kTokens = max_tokens<Q, kFew>();
  constexpr int kEntries = kTokens * (kFew ? kFewRanks : kMaxTopK);
  constexpr int kW = (kTokens + 63) / 64;
  __shared__ __align__(16) uint16_t s_ent[kEntries];           // (token, rank) -> expert | rank
  __shared__ float s_g[kEntries];                              // vanilla gate of that entry
  __shared__ float s_vh[kEntries];                             // vanilla logit of that entry
  __shared__ uint16_t s_list[kEntries];                        // entries grouped by expert
  __shared__ __align__(16) TokenMask<kW> s_occ[kMaxExperts];   // tokens of each expert
  __shared__ GreedyTables sh;
  __shared__ int s_off[kMaxExperts + 1];
  __shared__ uint8_t s_tier1[kMaxExperts];                   // picked by some request
  __shared__ uint8_t s_sel[kMaxExperts];
  __shared__ uint32_t s_seed[kWaves][2 * kMaxTopK];          // refinement seeds per wave
  __shared__ float s_seed_h[kWaves][2 * kMaxTopK];            //   (and per half of a wave)

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int T = a.T, N = a.N, k = a.k, k0 = a.k0;
  const bool dense = a.score_mode == 1;
  const bool hier = a.req_offsets != nullptr;
  const bool ep = a.G > 0;
  const int TK = T * k;

  // Two tokens per wave (one per half) where a token's experts fit 8 per lane and the batch
  // gives a wave more than one token, except with dense scores (their softmax sums every
  // expert of the token in index order): token pairs p = wave, wave + 16, ..., pair p
  // holding tokens 2p and 2p + 1.  Measured (selection us, one token per wave -> halves):
  // DeepSeek T=32 25.8 -> 25.0, Qwen T=64 34.4 -> 30.7, speculative T=64 40.0 -> 37.5; with
  // at most one token per wave (T <= 16) the half-wave rounds only add: T=8 18.0 -> 19.5.
  // Four tokens per wave (one per 16-lane row) where a token's experts fit 8 per lane, its
  // ranks fit in a row and the batch gives a wave more than two tokens (token quads p = wave,
  // wave + 16, ...).  The keys left after the top-k stay in registers (1024 threads allow 128
  // each): tokens, pairs and quads per wave.
  constexpr bool kHalves = Q <= 4;
  constexpr int Q2 = 2 * Q;
  constexpr bool kQuads = Q <= 2;
  constexpr int Q4 = 4 * Q;
  // (kFew: only more than 16 tokens, so in pairs or quads where these are)
  static_assert(max_tokens<Q, false>() >= kWaves, "kFew: pairs or quads");
  constexpr int kCache = kFew && kHalves ? 0 : (kTokens + kWaves - 1) / kWaves;
  constexpr int kCacheP = (kTokens + 2 * kWaves - 1) / (2 * kWaves);
  constexpr int kCacheQ = (kTokens + 4 * kWaves - 1) / (4 * kWaves);
  const int n_quads = (T + 3) >> 2;
  const bool quads = kQuads && !dense && k <= 16 && T > 2 * kWaves;
  const bool halves = kHalves && !dense && T > kWaves && !quads;
  const int hh = lane >> 5, sl = lane & 31;
  const int qr = lane >> 4, ql = lane & 15;
  const int n_pairs = (T + 1) >> 1;
  uint32_t kc[kCache > 0 ? kCache : 1][Q];
  uint32_t kcp[kHalves ? kCacheP : 1][kHalves ? Q2 : 1];
  uint32_t kcq[kQuads ? kCacheQ : 1][kQuads ? Q4 : 1];
  float raw_next[Q];
  float rawp_next[kHalves ? Q2 : 1];
  float rawq_next[kQuads ? Q4 : 1];
  // the wave's first logits row is on its way while the workgroup clears its tables
  if (quads) {
    if constexpr (kQuads)
      if (wave < n_quads) load_quad<Q4>(a, wave, ql, qr, rawq_next);
  } else if (halves) {
    if constexpr (kHalves)
      if (wave < n_pairs) load_pair<Q2>(a, wave, sl, hh, rawp_next);
  } else if (wave < T) {
    load_row<Q>(a, wave, lane, raw_next);
  }

  if (tid < 8) sh.cnt[tid] = 0;
  for (int j = tid; j < kMaxExperts; j += kThreads) {
    s_tier1[j] = 0;
    s_occ[j] = TokenMask<kW>{};
    sh.gload[j] = 0;
    sh.gcand[j] = 0;
    sh.hist[j] = 0;
  }
  __syncthreads();

  // ---- request offsets must be 0 = o_0 < o_1 < ... < o_R = T and every expert's group must
  //      lie in [0, G) (checked in parallel); otherwise the call selects nothing
  if (hier) {
    const int R = a.R;
    for (int r = tid; r < R; r += kThreads) {
      const int lo = a.req_offsets[r], hi = a.req_offsets[r + 1];
      if (!(lo < hi) || lo < 0 || hi > T) atomicOr(&sh.cnt[7], 1);
    }
    if (tid == 0 && (a.req_offsets[0] != 0 || a.req_offsets[R] != T)) atomicOr(&sh.cnt[7], 1);
  }
  if (ep && a.group)
    for (int jj = tid; jj < N; jj += kThreads)
      if (a.group[jj] < 0 || a.group[jj] >= a.G) atomicOr(&sh.cnt[7], 1);
  if (hier || (ep && a.group)) {
    __syncthreads();
    if (sh.cnt[7]) {
      for (int j = tid; j < N; j += kThreads) a.sel_mask[j] = 0;
      for (int p = tid; p < TK; p += kThreads) {
        a.ids[p] = -1;
        a.w[p] = 0.0f;
      }
      for (int j = tid; j <= N; j += kThreads) a.offsets[j] = 0;
      if (a.group_load)
        for (int g = tid; g < a.G; g += kThreads) a.group_load[g] = 0;
      if (tid == 0) {
        a.counters[kCntActive] = 0;
        a.counters[kCntSelected] = 0;
        a.counters[kCntStatus] = 1;
        if (a.stats) {
          a.stats[0] = -1;
          for (int s = 1; s < 8; ++s) a.stats[s] = 0;
        }
        if (a.ledger) {
          a.ledger[0] += 1;
          a.ledger[4] += 1;
        }
      }
      return;
    }
  }

  // ---- (a) per token: plain top-k and its gates (Section 2.2); dense softmax if requested.
  //      The next token's row is loaded while the current one is ranked; the keys left after
  //      the top-k (all experts but the token's top-k) stay in registers for the refinement.
  // Token i: its plain top-k, gates and entries; `left` receives the keys that remain
  // after the top-k.  The wave's next row is loaded meanwhile.
  auto plain_topk = [&](int i, uint32_t (&left)[Q]) {
    float raw[Q], v[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) raw[q] = raw_next[q];
    if (i + kWaves < T) load_row<Q>(a, i + kWaves, lane, raw_next);
    row_keys<Q>(raw, N, lane, v, left);
    float my_h;
    int my_j;
    wave_topk<Q>(left, 0, k, lane, my_h, my_j);
    const float g = ranked_gate(my_h, lane, k);
    if (lane < k) {
      s_ent[i * k + lane] = (uint16_t)(my_j < 0 ? kNoEntry : (uint32_t)((lane << 10) | my_j));
      s_g[i * k + lane] = g;
      s_vh[i * k + lane] = my_h;
    }
    if (dense) {
      const float m = lane_value(my_h, 0);
      float e[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) e[q] = (lane + 64 * q < N) ? exp_fixed(v[q] - m) : 0.0f;
      float z = 0.0f;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int lim = min(64, N - 64 * q);
        for (int l = 0; l < lim; ++l) z = z + lane_value(e[q], l);
      }
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (lane + 64 * q < N) a.dense[(size_t)i * N + lane + 64 * q] = e[q] / z;
    }
  };
  // Token pair p (halves): the plain top-k of both tokens, as plain_topk.
  auto plain_topk_pair = [&](int p, uint32_t (&left)[kHalves ? Q2 : 1]) {
    if constexpr (kHalves) {
      float raw[Q2];
#pragma unroll
      for (int q = 0; q < Q2; ++q) raw[q] = rawp_next[q];
      if (p + kWaves < n_pairs) load_pair<Q2>(a, p + kWaves, sl, hh, rawp_next);
      const int i = 2 * p + hh;
      const bool valid = i < T;
#pragma unroll
      for (int q = 0; q < Q2; ++q)
        left[q] = (valid && sl + 32 * q < N) ? ord(raw[q] + 0.0f) : 0u;
      float my_h;
      int my_j;
      half_topk<Q2>(left, 0, k, sl, hh, my_h, my_j);
      const float g = half_gate(my_h, sl, hh, k);
      if (valid && sl < k) {
        s_ent[i * k + sl] = (uint16_t)(my_j < 0 ? kNoEntry : (uint32_t)((sl << 10) | my_j));
        s_g[i * k + sl] = g;
        s_vh[i * k + sl] = my_h;
      }
    }
  };
  // Token quad p (rows): the plain top-k of four tokens, as plain_topk.
  auto plain_topk_quad = [&](int p, uint32_t (&left)[kQuads ? Q4 : 1]) {
    if constexpr (kQuads) {
      float raw[Q4];
#pragma unroll
      for (int q = 0; q < Q4; ++q) raw[q] = rawq_next[q];
      if (p + kWaves < n_quads) load_quad<Q4>(a, p + kWaves, ql, qr, rawq_next);
      const int i = 4 * p + qr;
      const bool valid = i < T;
#pragma unroll
      for (int q = 0; q < Q4; ++q)
        left[q] = (valid && ql + 16 * q < N) ? ord(raw[q] + 0.0f) : 0u;
      float my_h;
      int my_j;
      row_topk<Q4>(left, 0, k, ql, qr, my_h, my_j);
      const float g = row_gate(my_h, ql, qr, k);
      if (valid && ql < k) {
        s_ent[i * k + ql] = (uint16_t)(my_j < 0 ? kNoEntry : (uint32_t)((ql << 10) | my_j));
        s_g[i * k + ql] = g;
        s_vh[i * k + ql] = my_h;
      }
    }
  };
  if (quads) {
    if constexpr (kQuads) {
#pragma unroll
      for (int it = 0; it < kCacheQ; ++it)
        if (wave + it * kWaves < n_quads) plain_topk_quad(wave + it * kWaves, kcq[it]);
    }
  } else if (halves) {
    if constexpr (kHalves) {
#pragma unroll
      for (int it = 0; it < kCacheP; ++it)
        if (wave + it * kWaves < n_pairs) plain_topk_pair(wave + it * kWaves, kcp[it]);
    }
  } else {
    // compile-time slots keep the cache in registers
#pragma unroll
    for (int it = 0; it < kCache; ++it)
      if (wave + it * kWaves < T) plain_topk(wave + it * kWaves, kc[it]);
  }
  __syncthreads();

  // ---- (b) per expert: batch score (ascending tokens), membership of U and S_0
  const int j = tid;
  float s = 0.0f;
  bool inU = false, inS0 = false;
  {
    int total;
    const int cnt = group_by_expert(s_ent, s_occ, s_off, s_list, sh.wsum, TK, k, N, total);
    if (j < N) {
      // eight entries' loads, then their adds in token order (the loads do not wait for the
      // sum, so a long list costs one LDS round trip per eight tokens)
      const int o = s_off[j];
      for (int q0 = 0; q0 < cnt; q0 += 8) {
        float gq[8];
        uint32_t eq[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int p = s_list[o + min(q0 + u, cnt - 1)];
          gq[u] = s_g[p];
          eq[u] = s_ent[p];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          if (q0 + u < cnt) {
            if (!dense) s = s + gq[u];
            if ((int)((eq[u] >> 10) & 31u) < k0) inS0 = true;
          }
        }
      }
      inU = cnt > 0;
    }
  }
  if (dense && j < N)
    for (int i = 0; i < T; ++i) s = s + a.dense[(size_t)i * N + j];

  // ---- (c) per request (Algorithm 3), one wave per request: S_0(r) plus the m_r best
  //      remaining experts of r under the request's own score
  if (hier && a.m_r > 0) {
    for (int r = wave; r < a.R; r += kWaves) {
      const int lo = a.req_offsets[r], hi = a.req_offsets[r + 1];
      float sr[Q];
      unsigned inUr = 0, inS0r = 0;
#pragma unroll
      for (int q = 0; q < Q; ++q) sr[q] = 0.0f;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int jq = lane + 64 * q;
        if (jq >= N) continue;
        const int before = s_occ[jq].count_below(lo);
        const int n = s_occ[jq].count_below(hi) - before;
        const int o = s_off[jq] + before;
        for (int t0 = 0; t0 < n; t0 += 8) {   // loads ahead of the ordered adds, as in (b)
          float gq[8];
          uint32_t eq[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int p = s_list[o + min(t0 + u, n - 1)];
            gq[u] = s_g[p];
            eq[u] = s_ent[p];
          }
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            if (t0 + u < n) {
              if ((int)((eq[u] >> 10) & 31u) < k0) inS0r |= 1u << q;
              if (!dense) sr[q] = sr[q] + gq[u];
            }
          }
        }
        if (n > 0) inUr |= 1u << q;
      }
      if (dense)
        for (int i = lo; i < hi; ++i)
#pragma unroll
          for (int q = 0; q < Q; ++q)
            if (lane + 64 * q < N) sr[q] = sr[q] + a.dense[(size_t)i * N + lane + 64 * q];
      uint32_t key[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const bool cand = (lane + 64 * q < N) && (dense || ((inUr >> q) & 1u)) &&
                          !((inS0r >> q) & 1u);
        key[q] = cand ? ord(sr[q]) : 0u;
      }
      for (int t = 0; t < a.m_r; ++t) {
        uint32_t kb;
        const int jb = wave_pick<Q>(key, lane, kb);
        if (jb < 0) break;
        if (lane == 0) s_tier1[jb] = 1;
      }
    }
  }
  __syncthreads();

  // ---- (d) batch greedy
  int max_load = 0, n_s0 = 0, n_start = 0, n_u = 0, m_eff = 0;
  const bool sel = select_set(a, sh, j < N && s_tier1[j], s, inU, inS0, n_s0, n_start, n_u, m_eff);
  if (j < N) {
    s_sel[j] = sel;
    a.sel_mask[j] = sel;
    if (sel) atomicAdd(&sh.cnt[4], 1);
  }
  __syncthreads();
  if (ep) max_load = sh.cnt[0];

  // ---- (e) refinement: every token to its top-k inside S, gates renormalised (Section 3.4).
  //      The token's plain top-k experts that are in S are its first refined ranks (in
  //      their order); only the remaining ranks are searched, among the other experts.
  // Token i: `key` holds its keys without its plain top-k.
  auto refine = [&](int i, uint32_t (&key)[Q]) {
    const uint32_t vent = lane < k ? (uint32_t)s_ent[i * k + lane] : kNoEntry;
    const int vid = vent == kNoEntry ? -1 : (int)(vent & 1023u);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int jq = lane + 64 * q;
      if (jq >= N || !s_sel[jq]) key[q] = 0;
    }
    const bool keep = vid >= 0 && s_sel[vid];
    const uint64_t kept = __ballot(keep);
    const int m = __popcll(kept);
    if (keep) {
      const int dst = __popcll(kept & below(lane));
      s_seed[wave][dst] = (uint32_t)vid;
      s_seed_h[wave][dst] = s_vh[i * k + lane];
    }
    float my_h = -INFINITY;
    int my_j = -1;
    if (lane < m) {
      my_j = (int)s_seed[wave][lane];
      my_h = s_seed_h[wave][lane];
    }
    wave_topk<Q>(key, m, k, lane, my_h, my_j);
    const float g = ranked_gate(my_h, lane, k);
    if (lane < k) {
      a.ids[i * k + lane] = my_j;
      a.w[i * k + lane] = g;
      s_ent[i * k + lane] = (uint16_t)(my_j < 0 ? kNoEntry : (uint32_t)((lane << 10) | my_j));
    }
  };
  // Token pair p (halves): as refine, each half with its own token and seeds.
  auto refine_pair = [&](int p, uint32_t (&key)[kHalves ? Q2 : 1]) {
    if constexpr (kHalves) {
      const int i = 2 * p + hh;
      const bool valid = i < T;
      const uint32_t vent = (valid && sl < k) ? (uint32_t)s_ent[i * k + sl] : kNoEntry;
      const int vid = vent == kNoEntry ? -1 : (int)(vent & 1023u);
#pragma unroll
      for (int q = 0; q < Q2; ++q) {
        const int jq = sl + 32 * q;
        if (jq >= N || !s_sel[jq]) key[q] = 0;
      }
      const bool keep = vid >= 0 && s_sel[vid];
      const uint64_t kept = __ballot(keep);
      const uint32_t kh = hh ? (uint32_t)(kept >> 32) : (uint32_t)kept;
      const int m = __popc(kh);
      if (keep) {
        const int dst = __popc(kh & ((1u << sl) - 1u));
        s_seed[wave][hh * kMaxTopK + dst] = (uint32_t)vid;
        s_seed_h[wave][hh * kMaxTopK + dst] = s_vh[i * k + sl];
      }
      float my_h = -INFINITY;
      int my_j = -1;
      if (sl < m) {
        my_j = (int)s_seed[wave][hh * kMaxTopK + sl];
        my_h = s_seed_h[wave][hh * kMaxTopK + sl];
      }
      half_topk<Q2>(key, m, k, sl, hh, my_h, my_j);
      const float g = half_gate(my_h, sl, hh, k);
      if (valid && sl < k) {
        a.ids[i * k + sl] = my_j;
        a.w[i * k + sl] = g;
        s_ent[i * k + sl] = (uint16_t)(my_j < 0 ? kNoEntry : (uint32_t)((sl << 10) | my_j));
      }
    }
  };
  // Token quad p (rows): as refine, each row with its own token and seeds.
  auto refine_quad = [&](int p, uint32_t (&key)[kQuads ? Q4 : 1]) {
    if constexpr (kQuads) {
      const int i = 4 * p + qr;
      const bool valid = i < T;
      const uint32_t vent = (valid && ql < k) ? (uint32_t)s_ent[i * k + ql] : kNoEntry;
      const int vid = vent == kNoEntry ? -1 : (int)(vent & 1023u);
#pragma unroll
      for (int q = 0; q < Q4; ++q) {
        const int jq = ql + 16 * q;
        if (jq >= N || !s_sel[jq]) key[q] = 0;
      }
      const bool keep = vid >= 0 && s_sel[vid];
      const uint64_t kept = __ballot(keep);
      const uint32_t kq = (uint32_t)(kept >> (16 * qr)) & 0xFFFFu;
      const int m = __popc(kq);
      if (keep) {
        const int dst = __popc(kq & ((1u << ql) - 1u));
        s_seed[wave][qr * 16 + dst] = (uint32_t)vid;
        s_seed_h[wave][qr * 16 + dst] = s_vh[i * k + ql];
      }
      float my_h = -INFINITY;
      int my_j = -1;
      if (ql < m) {
        my_j = (int)s_seed[wave][qr * 16 + ql];
        my_h = s_seed_h[wave][qr * 16 + ql];
      }
      row_topk<Q4>(key, m, k, ql, qr, my_h, my_j);
      const float g = row_gate(my_h, ql, qr, k);
      if (valid && ql < k) {
        a.ids[i * k + ql] = my_j;
        a.w[i * k + ql] = g;
        s_ent[i * k + ql] = (uint16_t)(my_j < 0 ? kNoEntry : (uint32_t)((ql << 10) | my_j));
      }
    }
  };
  if (quads) {
    if constexpr (kQuads) {
#pragma unroll
      for (int it = 0; it < kCacheQ; ++it)
        if (wave + it * kWaves < n_quads) refine_quad(wave + it * kWaves, kcq[it]);
    }
  } else if (halves) {
    if constexpr (kHalves) {
#pragma unroll
      for (int it = 0; it < kCacheP; ++it)
        if (wave + it * kWaves < n_pairs) refine_pair(wave + it * kWaves, kcp[it]);
    }
  } else {
#pragma unroll
    for (int it = 0; it < kCache; ++it)
      if (wave + it * kWaves < T) refine(wave + it * kWaves, kc[it]);
  }
  __syncthreads();

  // ---- (f) permutation: rows grouped by expert (ascending), tokens ascending inside
  int total = 0, off = 0;
  for (int jj = tid; jj < kMaxExperts; jj += kThreads) s_occ[jj] = TokenMask<kW>{};
  __syncthreads();
  const int cnt =
      group_by_expert(s_ent, s_occ, s_off, s_list, sh.wsum, TK, k, N, total);
  if (j < N) {
    off = s_off[j];
    for (int q = 0; q < cnt; ++q) a.perm[off + q] = s_list[off + q];
  }
  // with a local GPU group only that group's experts are listed for the expert GEMMs
  const bool listed = j < N && cnt > 0 &&
                      (a.local_group < 0 ||
                       (a.group ? a.group[j] : j / (N / a.G)) == a.local_group);
  // The active list puts experts with more than kHeavyRows routed rows first (in expert
  // order), then the others: their GEMM blocks run longest, so they start first instead of
  // trailing the launch.  One scan counts both classes (16 bits each).
  const bool heavy = listed && cnt > kHeavyRows;
  int packed_total = 0;
  const int packed = block_excl_scan(listed ? (heavy ? 1 : (1 << 16)) : 0, sh.wsum, packed_total);
  const int n_heavy = packed_total & 0xFFFF;
  const int n_active = n_heavy + (packed_total >> 16);
  const int arank = heavy ? (packed & 0xFFFF) : n_heavy + (packed >> 16);
  if (j < N) {
    a.offsets[j] = off;
    if (j == N - 1) a.offsets[N] = off + cnt;
    if (listed) a.active[arank] = make_int4(j, off, cnt, 0);
  }
  if (tid == 0) {
    a.counters[kCntActive] = n_active;
    a.counters[kCntSelected] = sh.cnt[4];
    a.counters[kCntStatus] = 0;
    if (a.stats) {
      a.stats[0] = sh.cnt[4];
      a.stats[1] = n_active;
      a.stats[2] = n_u;
      a.stats[3] = n_s0;
      a.stats[4] = n_start;
      a.stats[5] = m_eff;
      a.stats[6] = max_load;
      a.stats[7] = 0;
    }
    if (a.ledger) {   // running totals over the layers of a pass (global budget K)
      a.ledger[0] += 1;
      a.ledger[1] += sh.cnt[4];
      a.ledger[2] += n_active;
      a.ledger[3] += n_u;
      a.ledger[5] = max(a.ledger[5], sh.cnt[4]);
    }
  }
}

// ---- Batches past the one-workgroup kernel's limit: the same steps as four kernels over the
// whole GPU.  Only the greedy needs every expert's score in one place, and it is cheap, so
// each block of the third kernel repeats it for the tokens it refines.
//   route_tokens_kernel  (a)      one wave per token: its plain top-k and gates
//   route_scores_kernel  (b), (c) one wave per expert: its batch score, tokens ascending; one
//                                 wave per request: its picks
//   route_refine_kernel  (d), (e) per block the greedy, then one wave per token
//   route_lists_kernel   (f)      per block the expert counts, then one wave per expert
// One workgroup, where a thread per expert walked all T * k entries, took 6 to 22 times as long
// (us a call in a stream of them, one workgroup -> four kernels): N=256 k=8 T=128 151 -> 26, T=512
// 585 -> 35, T=1024 1157 -> 52; N=128 T=256 287 -> 27; N=8 k=2 T=1024 353 -> 27.  What is left is
// four launches and the latency of each one's dependent loads.  Between the kernels the plain
// top-k entries lie in `perm` (rank << 10 | expert, -1 = none) and their gates in `w`, both
// overwritten with the results later; an expert's score and flags in its `active` record.
constexpr int kTokThreads = 256;
constexpr int kTokWaves = kTokThreads / 64;
constexpr uint32_t kFlagU = 1, kFlagS0 = 2;

__device__ __forceinline__ int rank_before(uint64_t m) {   // set bits of m in lanes below
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

// s + v(lane 0) + v(lane 1) + ... in lane order; lanes past the data hold +0.0 (s >= 0 stays
// as it is).  n: lanes that hold data, for an early end.
__device__ __forceinline__ float add_lanes(float s, float v, int n) {
  for (int l0 = 0; l0 < n; l0 += 8) {
#pragma unroll
    for (int l = 0; l < 8; ++l) s = s + lane_value(v, l0 + l);
  }
  return s;
}

template <int Q>
__global__ __launch_bounds__(kTokThreads) void route_tokens_kernel(RouteArgs a) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int T = a.T, N = a.N, k = a.k;
  // the first block also clears the picks and checks the offsets and the group map (as
  // route_kernel does); the later kernels read the status
  if (blockIdx.x == 0) {
    __shared__ int s_bad;
    if (tid == 0) s_bad = 0;
    __syncthreads();
    for (int j = tid; j < N; j += kTokThreads) a.active[j] = make_int4(0, 0, 0, 0);
    bool bad = false;
    if (a.req_offsets) {
      for (int r = tid; r < a.R; r += kTokThreads) {
        const int lo = a.req_offsets[r], hi = a.req_offsets[r + 1];
        bad = bad || !(lo < hi) || lo < 0 || hi > T;
      }
      if (tid == 0) bad = bad || a.req_offsets[0] != 0 || a.req_offsets[a.R] != T;
    }
    if (a.G > 0 && a.group)
      for (int j = tid; j < N; j += kTokThreads)
        bad = bad || a.group[j] < 0 || a.group[j] >= a.G;
    if (bad) atomicOr(&s_bad, 1);
    __syncthreads();
    if (tid == 0) a.counters[kCntStatus] = s_bad;
  }
  const int i = blockIdx.x * kTokWaves + wave;
  if (i >= T) return;
  float raw[Q], v[Q];
  uint32_t key[Q];
  load_row<Q>(a, i, lane, raw);
  row_keys<Q>(raw, N, lane, v, key);
  float my_h;
  int my_j;
  wave_topk<Q>(key, 0, k, lane, my_h, my_j);
  const float g = ranked_gate(my_h, lane, k);
  if (lane < k) {
    a.perm[i * k + lane] = my_j < 0 ? -1 : (lane << 10) | my_j;
    a.w[i * k + lane] = g;
  }
  if (a.score_mode == 1) {
    const float m = lane_value(my_h, 0);
    float e[Q];
    float z = 0.0f;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      e[q] = (lane + 64 * q < N) ? exp_fixed(v[q] - m) : 0.0f;
      z = add_lanes(z, e[q], min(64, N - 64 * q));
    }
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (lane + 64 * q < N) a.dense[(size_t)i * N + lane + 64 * q] = e[q] / z;
  }
}

// One wave: expert j's entries in token order are gathered into the wave's LDS list (ballots
// give each entry its place), then their gates are loaded 64 at a time and added in order.
template <int Q>
__global__ __launch_bounds__(kTokThreads) void route_scores_kernel(RouteArgs a) {
  __shared__ uint16_t s_list[kTokWaves][kMaxTokens];   // an expert holds a token at most once
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int T = a.T, N = a.N, k = a.k, k0 = a.k0, TK = T * k;
  const bool dense = a.score_mode == 1;
  const int unit = blockIdx.x * kTokWaves + wave;
  if (unit < N) {
    const int j = unit;
    uint16_t* const list = s_list[wave];
    int cnt = 0;
    const int4* const ents = reinterpret_cast<const int4*>(a.perm);
    constexpr int kAhead = 4;                          // 256-entry pieces loaded together
    for (int b0 = 0; b0 < TK; b0 += 256 * kAhead) {
      int4 e4[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int p = b0 + 256 * u + 4 * lane;
        e4[u] = p < TK ? ents[p >> 2] : make_int4(-1, -1, -1, -1);
      }
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int p = b0 + 256 * u + 4 * lane;
        const int en[4] = {e4[u].x, e4[u].y, e4[u].z, e4[u].w};
        bool hit[4];
        int before = 0, all = 0, mine = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          hit[c] = p + c < TK && (en[c] & 0x800003FF) == j;
          const uint64_t m = __ballot(hit[c]);
          before += rank_before(m);
          all += __popcll(m);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (hit[c]) list[cnt + before + mine++] = (uint16_t)(p + c);
        cnt += all;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    float s = 0.0f;
    bool s0 = false;
    for (int q0 = 0; q0 < cnt; q0 += 64) {
      const int p = list[min(q0 + lane, cnt - 1)];
      const float g = q0 + lane < cnt ? a.w[p] : 0.0f;
      s0 = s0 || p % k < k0;
      if (!dense) s = add_lanes(s, g, min(64, cnt - q0));
    }
    if (dense) {
      for (int i0 = 0; i0 < T; i0 += 64) {
        const float g = i0 + lane < T ? a.dense[(size_t)(i0 + lane) * N + j] : 0.0f;
        s = add_lanes(s, g, min(64, T - i0));
      }
    }
    const bool inS0 = __ballot(s0) != 0;
    if (lane == 0) {
      a.active[j].x = __float_as_int(s);
      a.active[j].y = (int)((cnt > 0 ? kFlagU : 0) | (inS0 ? kFlagS0 : 0));
    }
    return;
  }
  // per request: S_0(r) plus the m_r best remaining experts of r under the request's own score
  const int r = unit - N;
  if (!a.req_offsets || a.m_r <= 0 || r >= a.R || a.counters[kCntStatus]) return;
  const int lo = a.req_offsets[r], hi = a.req_offsets[r + 1];
  float sr[Q];
  unsigned inUr = 0, inS0r = 0;
#pragma unroll
  for (int q = 0; q < Q; ++q) sr[q] = 0.0f;
  for (int p0 = lo * k; p0 < hi * k; p0 += 64) {
    const int p = p0 + lane;
    const int my_ent = p < hi * k ? a.perm[p] : -1;
    const float my_g = p < hi * k ? a.w[p] : 0.0f;
    const int n = min(64, hi * k - p0);
    for (int l = 0; l < n; ++l) {
      const int ent = __builtin_amdgcn_readlane(my_ent, l);
      if (ent < 0) continue;
      const float g = lane_value(my_g, l);
      const bool here = (ent & 63) == lane;
      const int qe = (ent & 1023) >> 6;
      const bool warm = ((ent >> 10) & 31) < k0;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        if (here && q == qe) {
          inUr |= 1u << q;
          if (warm) inS0r |= 1u << q;
          if (!dense) sr[q] = sr[q] + g;
        }
      }
    }
  }
  if (dense)
    for (int i = lo; i < hi; ++i)
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (lane + 64 * q < N) sr[q] = sr[q] + a.dense[(size_t)i * N + lane + 64 * q];
  uint32_t key[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const bool cand = (lane + 64 * q < N) && (dense || ((inUr >> q) & 1u)) &&
                      !((inS0r >> q) & 1u);
    key[q] = cand ? ord(sr[q]) : 0u;
  }
  for (int t = 0; t < a.m_r; ++t) {
    uint32_t kb;
    const int jb = wave_pick<Q>(key, lane, kb);
    if (jb < 0) break;
    if (lane == 0) a.active[jb].z = 1;     // several requests may store the same 1
  }
}

template <int Q>
__global__ __launch_bounds__(kThreads) void route_refine_kernel(RouteArgs a) {
  __shared__ GreedyTables sh;
  __shared__ uint8_t s_sel[kMaxExperts];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int T = a.T, N = a.N, k = a.k, j = tid;
  const int i = blockIdx.x * kWaves + wave;
  const bool first = blockIdx.x == 0;
  if (a.counters[kCntStatus]) {            // invalid offsets or groups: nothing is selected
    if (i < T && lane < k) {
      a.ids[i * k + lane] = -1;
      a.w[i * k + lane] = 0.0f;
    }
    if (first) {
      if (j < N) a.sel_mask[j] = 0;
      if (a.group_load && tid < a.G) a.group_load[tid] = 0;
    }
    return;
  }
  float raw[Q];
  if (i < T) load_row<Q>(a, i, lane, raw);
  const int4 rec = j < N ? a.active[j] : make_int4(0, 0, 0, 0);
  if (tid < 8) sh.cnt[tid] = 0;
  sh.gload[tid] = 0;
  sh.gcand[tid] = 0;
  sh.hist[tid] = 0;
  __syncthreads();
  int n_s0 = 0, n_start = 0, n_u = 0, m_eff = 0;
  const bool sel = select_set(a, sh, rec.z != 0, __int_as_float(rec.x), (rec.y & kFlagU) != 0,
                              (rec.y & kFlagS0) != 0, n_s0, n_start, n_u, m_eff);
  if (j < N) {
    s_sel[j] = sel;
    if (first) a.sel_mask[j] = sel;
    if (sel) atomicAdd(&sh.cnt[4], 1);
  }
  __syncthreads();
  if (first && tid == 0) {
    a.counters[kCntSelected] = sh.cnt[4];
    a.counters[kCntU] = n_u;
    a.counters[kCntS0] = n_s0;
    a.counters[kCntStart] = n_start;
    a.counters[kCntBudget] = m_eff;
    a.counters[kCntMaxLoad] = a.G > 0 ? sh.cnt[0] : 0;
  }
  if (i >= T) return;
  uint32_t key[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int jq = lane + 64 * q;
    key[q] = jq < N && s_sel[jq] ? ord(raw[q] + 0.0f) : 0u;
  }
  float my_h;
  int my_j;
  wave_topk<Q>(key, 0, k, lane, my_h, my_j);
  const float g = ranked_gate(my_h, lane, k);
  if (lane < k) {
    a.ids[i * k + lane] = my_j;
    a.w[i * k + lane] = g;
  }
}

// Every block counts the rows of all experts (LDS atomics) and scans the counts, so each knows
// where its experts' rows start; a wave then writes one expert's rows in order.
__global__ __launch_bounds__(kThreads) void route_lists_kernel(RouteArgs a) {
  __shared__ __align__(16) uint16_t s_ent[kMaxAssignments];
  __shared__ int s_cnt[kMaxExperts];
  __shared__ int s_off[kMaxExperts];
  __shared__ int s_wsum[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = tid;
  const int N = a.N, TK = a.T * a.k;
  const bool first = blockIdx.x == 0;
  if (a.counters[kCntStatus]) {
    if (!first) return;
    for (int e = tid; e <= N; e += kThreads) a.offsets[e] = 0;
    if (tid == 0) {
      a.counters[kCntActive] = 0;
      a.counters[kCntSelected] = 0;
      if (a.stats) {
        a.stats[0] = -1;
        for (int s = 1; s < 8; ++s) a.stats[s] = 0;
      }
      if (a.ledger) {
        a.ledger[0] += 1;
        a.ledger[4] += 1;
      }
    }
    return;
  }
  s_cnt[tid] = 0;
  __syncthreads();
  const int TK8 = (TK + 7) & ~7;           // <= kMaxAssignments, a multiple of 8
  for (int p = tid; p < TK8; p += kThreads) {
    const int e = p < TK ? a.ids[p] : -1;
    s_ent[p] = e < 0 ? (uint16_t)kNoEntry : (uint16_t)e;
    if (e >= 0) atomicAdd(&s_cnt[e], 1);
  }
  __syncthreads();
  const int cnt = s_cnt[j];                // 0 past N
  int total = 0;
  const int off = block_excl_scan(cnt, s_wsum, total);
  s_off[j] = off;
  __syncthreads();
  if (first) {
    // as route_kernel's list, but an expert of more than kSlotRows rows takes several slots
    // of nearly equal size
    const bool listed = cnt > 0 && (a.local_group < 0 ||
                                    (a.group ? a.group[j] : j / (N / a.G)) == a.local_group);
    const bool heavy = listed && cnt > kHeavyRows;
    const int parts = (cnt + kSlotRows - 1) / kSlotRows;
    int packed_total = 0;
    const int packed =
        block_excl_scan(listed ? (heavy ? parts : (1 << 16)) : 0, s_wsum, packed_total);
    const int n_heavy = packed_total & 0xFFFF;
    const int at = heavy ? (packed & 0xFFFF) : n_heavy + (packed >> 16);
    if (j < N) a.offsets[j] = off;
    if (j == N - 1) a.offsets[N] = off + cnt;
    if (listed) {
      for (int c = 0; c < parts; ++c) {
        const int lo = cnt * c / parts, hi = cnt * (c + 1) / parts;
        a.active[at + c] = make_int4(j, off + lo, hi - lo, (parts - 1) << 16 | c);
      }
    }
    block_excl_scan(listed ? 1 : 0, s_wsum, total);     // total: the active experts
    if (tid == 0) {
      const int n_sel = a.counters[kCntSelected], n_u = a.counters[kCntU];
      a.counters[kCntActive] = n_heavy + (packed_total >> 16);
      if (a.stats) {
        a.stats[0] = n_sel;
        a.stats[1] = total;
        a.stats[2] = n_u;
        a.stats[3] = a.counters[kCntS0];
        a.stats[4] = a.counters[kCntStart];
        a.stats[5] = a.counters[kCntBudget];
        a.stats[6] = a.counters[kCntMaxLoad];
        a.stats[7] = 0;
      }
      if (a.ledger) {
        a.ledger[0] += 1;
        a.ledger[1] += n_sel;
        a.ledger[2] += total;
        a.ledger[3] += n_u;
        a.ledger[5] = max(a.ledger[5], n_sel);
      }
    }
  }
  const int e = blockIdx.x * kWaves + wave;
  if (e >= N || s_cnt[e] == 0) return;
  int at = s_off[e];
  for (int b0 = 0; b0 < TK8; b0 += 512) {
    const int p = b0 + 8 * lane;
    uint4 v = make_uint4(~0u, ~0u, ~0u, ~0u);
    if (p < TK8) v = *reinterpret_cast<const uint4*>(s_ent + p);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    bool hit[8];
    int before = 0, all = 0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      hit[c] = ((w[c >> 1] >> (16 * (c & 1))) & 0xFFFFu) == (uint32_t)e;
      const uint64_t m = __ballot(hit[c]);
      before += rank_before(m);
      all += __popcll(m);
    }
    int mine = at + before;
#pragma unroll
    for (int c = 0; c < 8; ++c)
      if (hit[c]) a.perm[mine++] = p + c;
    at += all;
  }
}

template <int Q>
hipError_t launch_route_q(const RouteArgs& a, hipStream_t stream) {
  if (a.T <= one_group_tokens<Q>(a)) {
    if (a.T <= max_tokens<Q, false>())
      hipLaunchKernelGGL((route_kernel<Q, false>), dim3(1), dim3(kThreads), 0, stream, a);
    else
      hipLaunchKernelGGL((route_kernel<Q, true>), dim3(1), dim3(kThreads), 0, stream, a);
    return hipGetLastError();
  }
  const int units = a.N + (a.req_offsets && a.m_r > 0 ? a.R : 0);
  hipLaunchKernelGGL(route_tokens_kernel<Q>, dim3((a.T + kTokWaves - 1) / kTokWaves),
                     dim3(kTokThreads), 0, stream, a);
  hipLaunchKernelGGL(route_scores_kernel<Q>, dim3((units + kTokWaves - 1) / kTokWaves),
                     dim3(kTokThreads), 0, stream, a);
  hipLaunchKernelGGL(route_refine_kernel<Q>, dim3((a.T + kWaves - 1) / kWaves), dim3(kThreads), 0,
                     stream, a);
  hipLaunchKernelGGL(route_lists_kernel, dim3((a.N + kWaves - 1) / kWaves), dim3(kThreads), 0,
                     stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_route(const RouteArgs& a, hipStream_t stream) {
  if (a.N <= 64) return launch_route_q<1>(a, stream);
  if (a.N <= 128) return launch_route_q<2>(a, stream);
  if (a.N <= 256) return launch_route_q<4>(a, stream);
  if (a.N <= 512) return launch_route_q<8>(a, stream);
  return launch_route_q<16>(a, stream);
}

}  // namespace xs
