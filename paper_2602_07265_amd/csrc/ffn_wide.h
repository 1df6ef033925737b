// GEMMs of large batches: part of ffn.hip, inside its namespaces.
//
// An expert's rows (up to kSlotRows of them, one slot) share one pass over its weights, so that
// weights stream once; the staged pass of ffn.hip reads them again for every 32 rows.
// Both operands go through LDS: weights loaded straight into the B operand, as there, touch 64
// cache lines per 64 lanes, and past 32 rows the L1's line rate (one a cycle), not the matrix
// cores, sets the time (Mixtral T=1024 gate/up took 1000 us so, 80 % of the L1's cycles in weight
// loads).  Here eight lanes read a row's 128 bytes.
//   A block of 2 NW threads holds NW weight rows; its waves (two a SIMD, so that one's LDS and
// address work runs under the other's MFMAs; one wave a SIMD with twice the tile measured 930 us
// against 720) take 64 of them and half of the token tiles each, or, up to 64 token rows, 32 of
// them and all token tiles.
//   A step is KB elements: its pieces are loaded into registers two steps (kSets) before they are
// written into one of two LDS buffers, one step before their MFMAs.
//   A region is the MFMAs of 32 elements (of the hi or of the lo chunks in the down GEMM); the
// operands of the next region are read during it.  One barrier a step, before its last region.
// sched_barrier keeps a region's loads in it: left alone the compiler sank them to the end of
// the step, next to their waits.
//   LDS rows have no padding; 16-byte piece c of row r lies at piece c ^ sw(r), which puts any 16
// lanes of a read into distinct banks (rows 16 bytes apart instead cost 4 conflict cycles a read).
//   bf16: lane group g's elements of group u are 32u + 8g; FP8 and MXFP4: 16g + 8u of each 64, one
// read for both groups.
// Measured, us (staged pass -> this one): Mixtral T=1024 gate/up 2605 -> 700 (0.48 TFLOP, 687
// TFLOP/s; a large library product reaches 1220 on this card, which clocks down to 1.9 GHz), down
// 1506 -> 588 (0.48 TFLOP with hi and lo); DeepSeek T=512 M=96 gate/up 1983 -> 992 (5.6 GB of
// weights, 5.7 TB/s), down 1149 -> 576 (2.8 GB, 4.9 TB/s).
template <int kW, bool kDown, int NW>
struct Wide {
  static constexpr int kThreads = 2 * NW;
  static constexpr int AS = kDown ? 2 : 1;               // staged elements of x per element
  // elements per step; codes take twice as many where LDS has room, for the bytes in flight
  static constexpr int KB = kW != kBf16 && !kDown && NW == 256 ? 128 : 64;
  static constexpr int G = KB / 32 * AS;                 // regions per step
  static constexpr int XP = AS * KB / 8;                 // 16-byte pieces of an x row
  static constexpr int XR = kThreads / XP;               // x rows that the block's threads cover
  static constexpr int kXBytes = kSlotRows * XP * 16;    // of a buffer
  static constexpr int WP = KB / (kW == kBf16 ? 8 : (kW == kFp8 ? 16 : 32));   // of a weight row
  static constexpr int WR = kThreads / WP;
  static constexpr int NL = NW / WR;                     // weight pieces per thread and step
  static_assert(NW % WR == 0, "every thread loads weights");
  static constexpr int kBuf = kXBytes + NW * WP * 16;    // bytes of a buffer
  static constexpr int RB = KB / (kW == kBf16 ? 32 : 64);  // B reads per step and tile
  static constexpr int LG = kW == kBf16 ? 8 : 16;        // elements between lane groups
  // element of lane group g's piece in 32-element group u
  __device__ static int element(int g, int u) {
    return kW == kBf16 ? 32 * u + 8 * g : 64 * (u >> 1) + 16 * g + 8 * (u & 1);
  }
  static constexpr int kCodes = kW == kMx4 ? 2 : 1;      // elements per weight byte, for codes
  // swizzles of 8, 4 and 2 pieces a row, and of 16
  __device__ static int sw(int pieces, int r) {
    return pieces == 16  ? r & 15
           : pieces == 8 ? (r >> 1) & 7
           : pieces == 4 ? (r >> 2) & 3
                         : (r >> 3) & 1;
  }
  __device__ static int xsw(int r) { return sw(XP, r); }
  __device__ static int wsw(int r) { return sw(WP, r); }
  __device__ static size_t wbytes(size_t elements) {     // bytes of that many weights
    return kW == kBf16 ? 2 * elements : elements / kCodes;
  }
};
// acc[m][rt] += the wave's NT token tiles against its NM weight tiles over K elements; MW waves
// share a weight tile and split the token tiles.  wrow(q, r): address of the first weight of this
// block's range in row r of 16-row tile q of the block (wave group w has tiles NM w to
// NM w + NM - 1); sc[m], sk: MXFP4, the lane's scale rows of its wave's tiles and its first input.
// x rows: x + tok[r] * ld, r < R; LDS rows past R hold the last row again.
template <int kW, bool kDown, int NW, int MW, int NM, int NT, typename F>
__device__ __forceinline__ void wide_pass(const uint16_t* x, size_t ld, const int* tok, int R,
                                          F wrow, const uint8_t* const (&sc)[NM], int sk, int K,
                                          floatx4 (&acc)[NM][NT], char* lds) {
  using W = Wide<kW, kDown, NW>;
  constexpr int KB = W::KB, AS = W::AS, G = W::G, NL = W::NL, kBuf = W::kBuf;
  constexpr int NX = (MW * NT * 16 + W::XR - 1) / W::XR;   // x pieces per thread and step
  constexpr int kSets = 2;
  static_assert(NM * 16 * 2 * NW / 64 / MW == NW, "the waves hold the block's weight rows");
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const int n = lane & 15, g = lane >> 4;

  // this thread's pieces: where they come from, and their place in a buffer
  const char* xsrc[NX];
  const char* wsrc[NL];
  const int xr = t / W::XP, xc = (t % W::XP) ^ W::xsw(xr);   // the swizzles repeat every 16 rows
  const int wr = t / W::WP, wc = (t % W::WP) ^ W::wsw(wr);
#pragma unroll
  for (int i = 0; i < NX; ++i)
    xsrc[i] =
        reinterpret_cast<const char*>(x + (size_t)tok[min(i * W::XR + xr, R - 1)] * ld) + 16 * xc;
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int r = i * W::WR + wr;
    wsrc[i] = wrow(r >> 4, r & 15) + 16 * wc;
  }
  char* const wx = lds + t * 16;
  // this lane's operands
  const char* const ax = lds + (wave % MW * NT * 16 + n) * (W::XP * 16);
  const char* const bx = lds + W::kXBytes + (wave / MW * NM * 16 + n) * (W::WP * 16);

  u32x4 v[kSets][NX], w[kSets][NL];
  const int steps = K / (2 * KB) * 2, last = (steps - 1) * KB;
  auto load = [&](int h, int k) {
    k = min(k, last);
#pragma unroll
    for (int i = 0; i < NX; ++i)
      v[h][i] = *reinterpret_cast<const u32x4*>(xsrc[i] + (size_t)(2 * AS) * k);
#pragma unroll
    for (int i = 0; i < NL; ++i)
      w[h][i] = *reinterpret_cast<const u32x4*>(wsrc[i] + W::wbytes(k));
  };
  auto store = [&](int h, int buf) {
#pragma unroll
    for (int i = 0; i < NX; ++i)
      *reinterpret_cast<u32x4*>(wx + buf * kBuf + i * (W::kThreads * 16)) = v[h][i];
#pragma unroll
    for (int i = 0; i < NL; ++i)
      *reinterpret_cast<u32x4*>(wx + W::kXBytes + buf * kBuf + i * (W::kThreads * 16)) = w[h][i];
  };
  // A operand of tile rt and B operands in region i of buffer buf: weight group i (down: i / 2)
  auto read_a = [&](int rt, int buf, int i) {
    const int u = kDown ? i >> 1 : i;
    const int e = W::element(g, u);
    const int c = kDown ? 2 * (e >> 3) + (i & 1) : e >> 3;
    return *reinterpret_cast<const bf16x8*>(ax + buf * kBuf + rt * (W::XP * 256) +
                                            16 * (c ^ W::xsw(n)));
  };
  using Codes = typename std::conditional<kW == kFp8, uint4, uint2>::type;
  using BR = typename std::conditional<kW == kBf16, bf16x8, Codes>::type;
  auto read_b = [&](BR (&r)[NM], int buf, int p) {   // read p of the step
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const char* const row = bx + buf * kBuf + m * (W::WP * 256);
      if constexpr (kW == kMx4)
        r[m] = *reinterpret_cast<const BR*>(row + 16 * ((2 * p + (g >> 1)) ^ W::wsw(n)) +
                                            8 * (g & 1));
      else
        r[m] = *reinterpret_cast<const BR*>(row + 16 * ((4 * p + g) ^ W::wsw(n)));
    }
  };
  auto read_e = [&](uint8_t (&e)[W::RB][NM], int k) {
    if constexpr (kW == kMx4) {
#pragma unroll
      for (int p = 0; p < W::RB; ++p)
#pragma unroll
        for (int m = 0; m < NM; ++m) e[p][m] = (uint8_t)load_mx_scales<1>(sc[m], sk + k + 64 * p);
    }
  };
  auto operand = [&](const BR& r, uint32_t e, int u) {
    if constexpr (kW == kBf16) return r;
    else if constexpr (kW == kFp8)
      return fp8x8_to_bf16(u ? make_uint2(r.z, r.w) : make_uint2(r.x, r.y));
    else return fp4x8_to_bf16(u ? r.y : r.x, e8m0_scale(e));
  };

  if (steps > 0) {
    bf16x8 xa[NT];
    BR b[2][NM];
    uint8_t e[kSets][W::RB][NM];
#pragma unroll
    for (int h = 0; h < kSets; ++h) load(h, h * KB);
#pragma unroll
    for (int h = 0; h < kSets; ++h) read_e(e[h], min(h * KB, last));
    store(0, 0);
    load(0, kSets * KB);
    __syncthreads();
    read_b(b[0], 0, 0);
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) xa[rt] = read_a(rt, 0, 0);
    // step k from buffer h; the set that holds step k + KB is written into the other buffer and
    // loaded with step k + (kSets + 1) KB
    auto step = [&](auto half, int k) {
      constexpr int h = decltype(half)::value;
#pragma unroll
      for (int i = 0; i < G; ++i) {
        const int nb = i < G - 1 ? h : h ^ 1, ni = (i + 1) % G;       // the next region
        const int u = kDown ? i >> 1 : i, nu = kDown ? ni >> 1 : ni;
        constexpr int kPair = kW == kBf16 ? 1 : 2;                    // groups of a B read
        const int r = u / kPair, nr = nu / kPair;
        __builtin_amdgcn_sched_barrier(0);
        if (i == (G > 2 ? 1 : 0)) {
          store(h ^ 1, h ^ 1);
          load(h ^ 1, k + (kSets + 1) * KB);
        }
        // b[parity of the read, counted over two steps]
        if (nr != r || i == G - 1)
          read_b(b[W::RB % 2 ? (i == G - 1 ? h ^ 1 : h) : nr & 1], nb, nr);
        bf16x8 bv[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m)
          bv[m] = operand(b[W::RB % 2 ? h : r & 1][m], e[h][r][m], u & 1);
#pragma unroll
        for (int rt = 0; rt < NT; ++rt) {
#pragma unroll
          for (int m = 0; m < NM; ++m) acc[m][rt] = mfma(xa[rt], bv[m], acc[m][rt]);
          xa[rt] = read_a(rt, nb, ni);
        }
        if (i == G - 2) {
          __builtin_amdgcn_sched_barrier(0);
          __syncthreads();
        }
      }
      read_e(e[h], min(k + 2 * KB, last));
    };
    for (int k = 0; k < last; k += 2 * KB) {     // in pairs: registers are named by parity
      step(std::integral_constant<int, 0>(), k);
      step(std::integral_constant<int, 1>(), k + KB);
    }
    __syncthreads();
  }
  // the rest of the reduction, not overlapped: up to KB elements' loads, then their MFMAs.  A
  // piece past the row reads the row's start; no MFMA takes it.
  for (int kr = steps * KB; kr < K; kr += KB) {
    const int len = min(KB, K - kr);
    u32x4 vx[NX], vw[NL];
#pragma unroll
    for (int i = 0; i < NX; ++i)
      vx[i] = *reinterpret_cast<const u32x4*>(
          xsrc[i] + (16 * xc < 2 * AS * len ? 2 * AS * kr : -16 * xc));
#pragma unroll
    for (int i = 0; i < NL; ++i)
      vw[i] = *reinterpret_cast<const u32x4*>(
          wsrc[i] + (16 * wc < (int)W::wbytes(len) ? (long)W::wbytes(kr) : -16L * wc));
#pragma unroll
    for (int i = 0; i < NX; ++i) *reinterpret_cast<u32x4*>(wx + i * (W::kThreads * 16)) = vx[i];
#pragma unroll
    for (int i = 0; i < NL; ++i)
      *reinterpret_cast<u32x4*>(wx + W::kXBytes + i * (W::kThreads * 16)) = vw[i];
    __syncthreads();
    for (int u = 0; u < len / 32; ++u) {
      const int el = 32 * u + 8 * g;             // this lane's elements of the step, all formats
      bf16x8 bv[NM];
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        const char* const row = bx + m * (W::WP * 256);
        const int c = (int)W::wbytes(el) >> 4, o = (int)W::wbytes(el) & 15;
        const char* const at = row + 16 * (c ^ W::wsw(n)) + o;
        if constexpr (kW == kBf16) bv[m] = *reinterpret_cast<const bf16x8*>(at);
        else if constexpr (kW == kFp8) bv[m] = fp8x8_to_bf16(*reinterpret_cast<const uint2*>(at));
        else
          bv[m] = fp4x8_to_bf16(*reinterpret_cast<const uint32_t*>(at),
                                e8m0_scale(load_mx_scales<1>(sc[m], sk - W::LG * g + kr + el)));
      }
#pragma unroll
      for (int hl = 0; hl < AS; ++hl)
#pragma unroll
        for (int rt = 0; rt < NT; ++rt) {
          const int c = kDown ? 2 * (el >> 3) + hl : el >> 3;
          const bf16x8 a = *reinterpret_cast<const bf16x8*>(ax + rt * (W::XP * 256) +
                                                            16 * (c ^ W::xsw(n)));
#pragma unroll
          for (int m = 0; m < NM; ++m) acc[m][rt] = mfma(a, bv[m], acc[m][rt]);
        }
    }
    __syncthreads();
  }
}

// The instance for R rows: f(MW, NM, NT).
template <typename F>
__device__ __forceinline__ void wide_tiles(int R, F f) {
  using std::integral_constant;
  constexpr integral_constant<int, 1> c1{};
  constexpr integral_constant<int, 2> c2{};
  constexpr integral_constant<int, 3> c3{};
  constexpr integral_constant<int, 4> c4{};
  if (R <= 16) f(c1, c2, c1);
  else if (R <= 32) f(c1, c2, c2);
  else if (R <= 48) f(c1, c2, c3);
  else if (R <= 64) f(c1, c2, c4);
  else if (R <= 96) f(c2, c4, c3);
  else f(c2, c4, c4);
}

// (slot, column block) of block L.  The parts of an expert that takes several slots run side by
// side on one XCD, column block by column block (consecutive workgroups go to the 8 XCDs in
// turn), so that its L2 serves their weights once.
__device__ __forceinline__ void wide_unit(const FfnArgs& a, int L, int CB, int& slot, int& bx) {
  slot = L / CB;
  bx = L % CB;
  int parts = 1, part = 0;
  if (slot < a.shared_slots) {
    parts = a.shared_parts;
    part = slot % parts;
  } else if (slot - a.shared_slots < a.counters[kCntActive]) {
    const int w = a.active[slot - a.shared_slots].w;
    parts = (w >> 16) + 1;
    part = w & 0xFFFF;
  }
  if (parts == 1) return;
  const int s0 = slot - part, CB8 = CB & ~7;
  int l = L - s0 * CB;
  if (l < CB8 * parts) {
    part = (l >> 3) % parts;
    bx = (l >> 3) / parts * 8 + (l & 7);
  } else {
    l -= CB8 * parts;
    part = l / (CB - CB8);
    bx = CB8 + l % (CB - CB8);
  }
  slot = s0 + part;
}

// Gate/up for one slot and NW / 2 columns (NW weight rows: W1's and W3's), as gate_up_kernel.
template <int kW, int NW>
__global__ __attribute__((amdgpu_waves_per_eu(2)))
__launch_bounds__(2 * NW) void gate_up_wide_kernel(FfnArgs a) {
  using W = Wide<kW, false, NW>;
  SlotWork sw;
  int slot, bx;
  wide_unit(a, blockIdx.x + gridDim.x * blockIdx.y, gridDim.x, slot, bx);
  if (!slot_work<kW>(a, slot, sw)) return;
  XS_TIME(xs_times_gu, 2 * block_id3(), 2u * kTimeBlocks);
  sw.e = __builtin_amdgcn_readfirstlane(sw.e);
  const int p0 = sw.p0, te = sw.te;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int n = lane & 15, g = lane >> 4;
  const int d = a.d, f = a.f;
  const int Kg = d / a.gu_splits;
  const size_t kbase = (size_t)blockIdx.z * Kg;
  const int jb = bx * (NW / 2);                  // the block's first column
  const char *m1, *m3;                           // the expert's W1 and W3
  if constexpr (kW == kBf16) {
    m1 = reinterpret_cast<const char*>(slot_w(a, sw, a.w1, a.sw1));
    m3 = reinterpret_cast<const char*>(slot_w(a, sw, a.w3, a.sw3));
  } else {
    m1 = reinterpret_cast<const char*>(a.q1) + W::wbytes((size_t)sw.e * f * d);
    m3 = reinterpret_cast<const char*>(a.q3) + W::wbytes((size_t)sw.e * f * d);
  }
  // tiles 2q and 2q + 1: the block's column tile q of W1 and of W3
  auto wrow = [&](int q, int r) {
    const size_t c = min(jb + 16 * (q >> 1), f - 16) + r;
    return ((q & 1) ? m3 : m1) + W::wbytes(c * d + kbase);
  };
  __shared__ __align__(16) char stage[2 * W::kBuf];
  __shared__ int s_tok[kSlotRows];
  if (threadIdx.x < te)
    s_tok[threadIdx.x] = sw.shared ? p0 - a.T * (a.k + sw.e) + threadIdx.x
                                   : a.perm[p0 + threadIdx.x] / a.k;
  __syncthreads();
  wide_tiles(te, [&](auto mw, auto nm, auto nt) {
    constexpr int MW = decltype(mw)::value, NM = decltype(nm)::value, NT = decltype(nt)::value;
    const int j0 = jb + wave / MW * (NM / 2) * 16;          // the wave's first column
    const uint8_t* sc[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      sc[m] = nullptr;
      if constexpr (kW == kMx4) {
        const int G = mx_granules(d);
        sc[m] = mx_row(((m & 1) ? a.e3 : a.e1) + (size_t)sw.e * f * G * 8,
                       min(j0 + 16 * (m >> 1), f - 16) + n, G);
      }
    }
    floatx4 acc[NM][NT];
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int rt = 0; rt < NT; ++rt) acc[m][rt] = floatx4{0.f, 0.f, 0.f, 0.f};
    wide_pass<kW, false, NW, MW, NM, NT>(a.x + kbase, d, s_tok, te, wrow, sc,
                                         (int)kbase + W::LG * g, Kg, acc, stage);
    const size_t plane = (size_t)a.part_rows * f;
    float* const part = a.gpart + 2 * blockIdx.z * plane;
#pragma unroll
    for (int ct = 0; ct < NM / 2; ++ct) {
      if (j0 + 16 * ct >= f) break;
      const int col = j0 + 16 * ct + n;
      const float s1 = kW == kFp8 ? a.s1[(size_t)sw.e * f + col] : 1.0f;
      const float s3 = kW == kFp8 ? a.s3[(size_t)sw.e * f + col] : 1.0f;
#pragma unroll
      for (int rt = 0; rt < NT; ++rt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int t = (wave % MW * NT + rt) * 16 + 4 * g + i;
          if (t >= te) continue;
          const float h1 = acc[2 * ct][rt][i] * s1;
          const float h3 = acc[2 * ct + 1][rt][i] * s3;
          if (a.gu_splits == 1) {
            store_hilo(a.h, p0 + t, col, f, h1 / (1.0f + __expf(-h1)) * h3);
          } else {
            const size_t at = (size_t)(p0 + t) * f + col;
            part[at] = h1;
            part[plane + at] = h3;
          }
        }
    }
  });
  XS_TIME(xs_times_gu, 2 * block_id3() + 1, 2u * kTimeBlocks);
}

// Down for one slot and NW output rows, as down_kernel.
template <int kW, int NW>
__global__ __attribute__((amdgpu_waves_per_eu(2)))
__launch_bounds__(2 * NW) void down_wide_kernel(FfnArgs a) {
  using W = Wide<kW, true, NW>;
  SlotWork sw;
  int slot, bx;
  wide_unit(a, blockIdx.x + gridDim.x * blockIdx.y, gridDim.x, slot, bx);
  if (!slot_work<kW>(a, slot, sw)) return;
  XS_TIME(xs_times_dn, 2 * block_id3(), 2u * kTimeBlocks);
  sw.e = __builtin_amdgcn_readfirstlane(sw.e);
  const int p0 = sw.p0, te = sw.te;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int n = lane & 15, g = lane >> 4;
  const int d = a.d, f = a.f;
  const int Ks = f / a.splits;
  const size_t kbase = (size_t)blockIdx.z * Ks;
  const int nb = bx * NW;                        // the block's first output row
  const char* m2;                                // the expert's W2
  if constexpr (kW == kBf16) m2 = reinterpret_cast<const char*>(slot_w(a, sw, a.w2, a.sw2));
  else m2 = reinterpret_cast<const char*>(a.q2) + W::wbytes((size_t)sw.e * d * f);
  auto wrow = [&](int q, int r) {
    const size_t row = min(nb + 16 * q, d - 16) + r;
    return m2 + W::wbytes(row * f + kbase);
  };
  __shared__ __align__(16) char stage[2 * W::kBuf];
  __shared__ int s_tok[kSlotRows], s_out[kSlotRows];
  if (threadIdx.x < te) {
    s_tok[threadIdx.x] = p0 + threadIdx.x;
    s_out[threadIdx.x] = sw.shared ? p0 + threadIdx.x : a.perm[p0 + threadIdx.x];
  }
  __syncthreads();
  float* const ypart = a.yslot + (size_t)blockIdx.z * a.rows * d;
  wide_tiles(te, [&](auto mw, auto nm, auto nt) {
    constexpr int MW = decltype(mw)::value, NM = decltype(nm)::value, NT = decltype(nt)::value;
    const int n0 = nb + wave / MW * NM * 16;     // the wave's first output row
    const uint8_t* sc[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      sc[m] = nullptr;
      if constexpr (kW == kMx4) {
        const int G = mx_granules(f);
        sc[m] = mx_row(a.e2 + (size_t)sw.e * d * G * 8, min(n0 + 16 * m, d - 16) + n, G);
      }
    }
    floatx4 acc[NM][NT];
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int rt = 0; rt < NT; ++rt) acc[m][rt] = floatx4{0.f, 0.f, 0.f, 0.f};
    wide_pass<kW, true, NW, MW, NM, NT>(a.h + 2 * kbase, 2 * (size_t)f, s_tok, te, wrow, sc,
                                        (int)kbase + W::LG * g, Ks, acc, stage);
    float sc2[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m)
      sc2[m] = kW == kFp8 ? a.s2[(size_t)sw.e * d + min(n0 + 16 * m, d - 16) + n] : 1.0f;
#pragma unroll
    for (int rt = 0; rt < NT; ++rt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = (wave % MW * NT + rt) * 16 + 4 * g + i;
        if (t >= te) continue;
        float* const yrow = ypart + (size_t)s_out[t] * d;
#pragma unroll
        for (int m = 0; m < NM; ++m)
          if (n0 + 16 * m < d) yrow[n0 + 16 * m + n] = acc[m][rt][i] * sc2[m];
      }
  });
  XS_TIME(xs_times_dn, 2 * block_id3() + 1, 2u * kTimeBlocks);
}
