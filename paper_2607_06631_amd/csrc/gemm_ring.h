// The GEMM kernel for every problem but the largest plain bf16 ones (those run
// gemm.hip's 256 x 256 kernel): one kernel over a family of tile shapes, so
// that a problem of any size is cut into about a whole number of tiles per CU.
//
// What bounds it: a k-tile of a 256 x 256 tile kept too few workgroups in
// flight for small problems, each waiting out a memory round trip per k-tile
// (1.2-1.4 us per 64-deep k-tile whatever the load: 87.7 us for 390 x 5120 x
// 4096, 129 us for 1560 x 1536 x 6720).  Here the operand tiles sit in a ring
// of NST LDS slots, NST - 1 tiles in flight, and each k-tile has one barrier,
// in its middle, behind which the next tile's first fragments are read under
// MFMAs that need none of them: 30.8 us and 40.3 us for the two, 141 us
// against 207 us for 1560 x 10368 x 5120 (bf16).
//
// k-tiles are 128 bytes per row as in gemm.hip (same operand layout, swizzle,
// gather modes and order of the reduction: the two kernels give the same
// bits).  float32 uses v_mfma_f32_16x16x4_f32, whose rate (256 flops per clock
// and CU) bounds every tile shape: 8000 x 3456 x 1536 at 144 TFLOP/s, 118 on
// 256 x 256 tiles.
#pragma once
#include <type_traits>

#include "gemm.h"

namespace dif {

template <typename T>
__device__ __forceinline__ void mma16(f32x4& acc, const u32x4& a, const u32x4& b) {
  if constexpr (sizeof(T) == 2) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                  __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
  } else {
    const f32x4 fa = __builtin_bit_cast(f32x4, a), fb = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[e], fb[e], acc, 0, 0, 0);
  }
}

template <typename T, typename OutT, int EPI, int GA, int WGM, int WGN, int AM, int AN, int NST, int OCC>
__global__ __launch_bounds__(64 * WGM * WGN, OCC) void gemm_ring_kernel(GemmParams<T, OutT> p) {
  constexpr int NW = WGM * WGN;
  constexpr int BM = WGM * AM * 16, BN = WGN * AN * 16;
  constexpr int VEC = Chunk<T>::VEC, BK = G_BKC * VEC;
  constexpr int GA8 = BM / 8, G8 = (BM + BN) / 8;   // 8-row load groups: of A, of both
  constexpr int LPT = (G8 + NW - 1) / NW;           // load instructions per wave and k-tile
  static_assert(BM % 16 == 0 && BN % 16 == 0 && G8 >= NW && NW % 2 == 0, "load split");
  static_assert(NST >= 2 && NST <= 6 && (NST - 1) * LPT < 64, "ring depth");
  // one LDS variable per ring slot: the compiler tells loads into one slot
  // from reads of another only across distinct variables
  __shared__ u32x4 s0_[BM + BN][G_BKC], s1_[BM + BN][G_BKC];
  __shared__ u32x4 s2_[NST > 2 ? BM + BN : 1][G_BKC], s3_[NST > 3 ? BM + BN : 1][G_BKC];
  __shared__ u32x4 s4_[NST > 4 ? BM + BN : 1][G_BKC], s5_[NST > 5 ? BM + BN : 1][G_BKC];
  auto slot = [&](auto st_c) __attribute__((always_inline)) -> u32x4(*)[G_BKC] {
    constexpr int st = decltype(st_c)::value;
    if constexpr (st == 0) return s0_;
    else if constexpr (st == 1) return s1_;
    else if constexpr (st == 2) return s2_;
    else if constexpr (st == 3) return s3_;
    else if constexpr (st == 4) return s4_;
    else return s5_;
  };
  extern __shared__ uint16_t kch_lds[];   // GA_KCH: source chunk of each K chunk

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const int g = lane >> 4, col = lane & 15;

  const int nbm = (p.M + BM - 1) / BM, nbn = (p.N + BN - 1) / BN;
  int mt, nt;
  tile_of(blockIdx.x, nbm, nbn * p.nseg, mt, nt);
  const int m0 = mt * BM;
  const int sg = nt / nbn;
  const int n0 = (nt - sg * nbn) * BN;
  const T* Bsg = p.Bs[sg];
  const float* bias_sg = p.biases[sg];
  OutT* Csg = p.C + (int64_t)sg * p.N;

  constexpr uint32_t kRsrcWord3 = 0x00020000u;
  constexpr int64_t ES = sizeof(T);
  const uint32_t a_bytes = (uint32_t)(min(BM, p.M - m0) * p.lda * ES);
  const uint32_t b_bytes = GA == GA_ROWS ? (uint32_t)((int64_t)p.b_rows * p.ldb * ES)
                                         : (uint32_t)(min(BN, p.N - n0) * p.ldb * ES);
  const T* b_base = GA == GA_ROWS ? Bsg : Bsg + (int64_t)n0 * p.ldb;
  const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<T*>(p.A + (int64_t)m0 * p.lda), (short)0, a_bytes, kRsrcWord3);
  const __amdgpu_buffer_rsrc_t b_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(b_base), (short)0, b_bytes, kRsrcWord3);
  // Load instruction i of wave w fills the eight LDS rows of group i * NW + w
  // (A's groups, then B's; past the last group the wave repeats its previous
  // one): lane l row + l / 8, physical chunk l % 8, fetching the logical chunk
  // that the swizzle places there, which is the same for all i (the swizzle
  // sees row bits 0..3: l / 8 and the group's parity, which is the wave's).
  const int wave_s = __builtin_amdgcn_readfirstlane(wave) & (NW - 1);
  const int lrow = lane / 8;
  const int dchunk = swz<G_BKC>((wave & 1) * 8 + lrow, lane % 8);
  auto group = [&](int i) __attribute__((always_inline)) {
    const int q = i * NW + wave_s;
    return (i + 1) * NW <= G8 || q < G8 ? q : q - NW;
  };
  // lane offsets without the k offset: row * ld + chunk of load instruction 0,
  // plus i times NW * 8 rows (A's; B's start BM rows in, modulo 2^32); gathered
  // B rows need an offset per instruction
  const uint32_t a_ld = (uint32_t)(p.lda * ES), b_ld = (uint32_t)(p.ldb * ES);
  const uint32_t lr0 = (uint32_t)(wave * 8 + lrow);
  const uint32_t a_off = lr0 * a_ld + dchunk * 16;
  const uint32_t b_off = (lr0 - BM) * b_ld + (GA == GA_KCH ? 0 : dchunk * 16);
  uint32_t r_off[GA == GA_ROWS ? LPT : 1];
  if constexpr (GA == GA_ROWS) {
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      const int q = group(i), n = n0 + q * 8 + lrow - BM;
      const int r = q >= GA8 && n < p.N ? p.rows[n] : -1;
      r_off[i] = r >= 0 ? (uint32_t)((r * p.ldb + dchunk * VEC) * ES) : kMasked;
    }
  }
  const int nk = p.K / BK;
  if constexpr (GA == GA_KCH) {   // (the host keeps chunk numbers below 65535)
    for (int c = tid; c < p.K / VEC; c += 64 * NW) kch_lds[c] = (uint16_t)p.kch[c];
    __syncthreads();
  }
  // load instruction i of tile kt into its slot
  // GA_KCH: byte offset of this lane's chunk of a tile, from the chunk table in
  // LDS (16-bit entries, so that three 160 x 256 slots leave room for it).  Read
  // half a tile ahead, in order with the fragment reads.  (A scalar load of the
  // tile's eight entries makes every wait for a fragment wait for it as well:
  // 13608 x 5120 x 2432 took 407 us on 256 x 256 tiles, 328 with the table.)
  uint32_t kb = 0, ke = 0;
  auto kb_load = [&](int kt) __attribute__((always_inline)) {
    if constexpr (GA == GA_KCH) ke = kch_lds[kt * G_BKC + dchunk];
  };
  auto kb_pick = [&]() __attribute__((always_inline)) {
    if constexpr (GA == GA_KCH) kb = ke != 0xffffu ? ke * 16u : kMasked;
  };
  auto issue_one = [&](int kt, auto st_c, int i) __attribute__((always_inline)) {
#if defined(__HIP_DEVICE_COMPILE__)
    typedef __attribute__((address_space(3))) void lds_t;
    const int koff = kt * BK * (int)ES;
    const int q = group(i);
    const uint32_t at = (uint32_t)(q & ~(NW - 1)) * 8;   // rows of instruction i past the first's
    lds_t* dst = (lds_t*)&slot(st_c)[q * 8][0];
    uint32_t a0 = a_off, b0 = b_off;
    // (opaque copies: formed here, not kept per instruction, for which the
    // chunk table's values leave no registers on the 224-row tile)
    if constexpr (GA == GA_KCH) asm volatile("" : "+v"(a0), "+v"(b0));
    const uint32_t oa = a0 + at * a_ld;
    uint32_t ob;
    if constexpr (GA == GA_ROWS) ob = r_off[i];
    else ob = b0 + at * b_ld + kb;
    constexpr bool KOFF = GA != GA_KCH;   // (a gathered chunk's offset is in kb)
    if ((i + 1) * NW <= GA8) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, dst, 16, oa, koff, 0, 0);
    } else if (i * NW >= GA8) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(b_rsrc, dst, 16, ob, KOFF ? koff : 0, 0, 0);
    } else {   // some waves' groups are A's, the others' B's
      const bool is_a = q < GA8;
      const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<T*>(is_a ? p.A + (int64_t)m0 * p.lda : b_base), (short)0, is_a ? a_bytes : b_bytes,
          kRsrcWord3);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst, 16, is_a ? oa : ob, is_a || KOFF ? koff : 0, 0, 0);
    }
#endif
  };
  auto issue = [&](int kt, auto st_c) __attribute__((always_inline)) {
    kb_load(kt);
    kb_pick();
#pragma unroll
    for (int i = 0; i < LPT; ++i) issue_one(kt, st_c, i);
  };

  f32x4 acc[AM][AN];
#pragma unroll
  for (int i = 0; i < AM; ++i)
#pragma unroll
    for (int j = 0; j < AN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // one load behind every second MFMA where there are enough (1 % over one
  // behind each, on 256 x 256 tiles)
  constexpr int LSTEP = AM * AN >= 2 * LPT ? 2 : 1;
  // Fragments of the two k-steps of a tile, each read from LDS while the
  // other's MFMAs issue: one read behind each MFMA, in the order the MFMAs
  // first use them (scheduling barriers keep that order).
  u32x4 fa[2][AM], fb[2][AN];
  constexpr FirstUse<AM, AN> fu = first_use_table<AM, AN>();
  auto frag_one = [&](auto st_c, int ks, int r) __attribute__((always_inline)) {
    const int c = swz<G_BKC>(col, 4 * ks + g);
    if (r < AM) fa[ks][r] = slot(st_c)[(wm * AM + r) * 16 + col][c];
    else fb[ks][r - AM] = slot(st_c)[BM + (wn * AN + r - AM) * 16 + col][c];
  };
  // Publishes tile kt: this wave's loads of it have landed (those of the tiles
  // after it, up to `ahead` of them, may be in flight) and its reads of the
  // tile before it are done; then everyone's.
  auto publish = [&](auto full_c) __attribute__((always_inline)) {
    constexpr int n = decltype(full_c)::value ? (NST - 2) * LPT : 0;
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((n & 15) | ((n >> 4) << 14) | (7 << 4) | (0 << 8));   // vmcnt(n) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // One k-tile, whose first k-step's fragments are in registers.  Half 0: its
  // MFMAs, and the second k-step's fragment reads behind them.  Then tile
  // kt + 1 is published, which also frees this tile's slot: half 1 loads tile
  // kt + NST into it and reads tile kt + 1's first fragments behind its MFMAs.
  // MAIN: tiles kt + 1 .. kt + NST exist.
  auto ktile = [&](int kt, auto st_c, auto main_c) __attribute__((always_inline)) {
    constexpr int st = decltype(st_c)::value;
    constexpr bool MAIN = decltype(main_c)::value;
    using NS = std::integral_constant<int, (st + 1) % NST>;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const bool next = MAIN || kt + 1 < nk, load = MAIN || kt + NST < nk;
      if (ks == 0) {
        if (load) kb_load(kt + NST);
      } else {
        if (next) {
          if (MAIN || kt + NST - 1 < nk) publish(std::true_type{});
          else publish(std::false_type{});
        }
        if (MAIN) kb_pick();
        if (!MAIN) {
          if (load) {
            kb_pick();
#pragma unroll
            for (int i = 0; i < LPT; ++i) issue_one(kt + NST, st_c, i);
          }
          if (next) {
#pragma unroll
            for (int r = 0; r < AM + AN; ++r) frag_one(NS{}, 0, fu.v[r]);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < AM * AN; ++i) {
        mma16<T>(acc[i / AN][i % AN], fa[ks][i / AN], fb[ks][i % AN]);
        if (ks == 0) {
          if (i < AM + AN) frag_one(st_c, 1, fu.v[i]);
        } else if (MAIN) {
          if (i < AM + AN) frag_one(NS{}, 0, fu.v[i]);
          if (i % LSTEP == 0 && i / LSTEP < LPT) issue_one(kt + NST, st_c, i / LSTEP);
        }
        if (i == AM * AN - 1) {   // (more reads or loads than MFMAs)
          if (ks == 0 || MAIN) {
#pragma unroll
            for (int r = AM * AN; r < AM + AN; ++r)
              if (ks == 0) frag_one(st_c, 1, fu.v[r]);
              else frag_one(NS{}, 0, fu.v[r]);
          }
          if (ks == 1 && MAIN) {
#pragma unroll
            for (int r = AM * AN / LSTEP; r < LPT; ++r) issue_one(kt + NST, st_c, r);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  using I4 = std::integral_constant<int, 4>;
  using I5 = std::integral_constant<int, 5>;
  auto prologue = [&](int n) __attribute__((always_inline)) {   // tiles 0 .. n-1, n <= NST
    if (n > 0) issue(0, I0{});
    if (n > 1) issue(1, I1{});
    if constexpr (NST > 2) if (n > 2) issue(2, I2{});
    if constexpr (NST > 3) if (n > 3) issue(3, I3{});
    if constexpr (NST > 4) if (n > 4) issue(4, I4{});
    if constexpr (NST > 5) if (n > 5) issue(5, I5{});
  };
  auto first = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < AM + AN; ++r) frag_one(I0{}, 0, fu.v[r]);
  };
  if (nk > 0) {
    using Y = std::true_type;
    using N = std::false_type;
    int kt = 0;
    if (nk >= 2 * NST) {
      // (no branch between the loads of this part: the compiler then counts
      // the loads in flight exactly and adds no waits of its own)
      prologue(NST);
      wait_vmcnt<(NST - 1) * LPT>();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      first();
      for (; kt + 2 * NST <= nk; kt += NST) {
        ktile(kt, I0{}, Y{});
        ktile(kt + 1, I1{}, Y{});
        if constexpr (NST > 2) ktile(kt + 2, I2{}, Y{});
        if constexpr (NST > 3) ktile(kt + 3, I3{}, Y{});
        if constexpr (NST > 4) ktile(kt + 4, I4{}, Y{});
        if constexpr (NST > 5) ktile(kt + 5, I5{}, Y{});
      }
    } else {
      prologue(min(nk, NST));
      wait_vmcnt<0>();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      first();
    }
    // the last 2 NST - 1 tiles or fewer
    for (; kt < nk; kt += NST) {
      ktile(kt, I0{}, N{});
      if (kt + 1 < nk) ktile(kt + 1, I1{}, N{});
      if constexpr (NST > 2) if (kt + 2 < nk) ktile(kt + 2, I2{}, N{});
      if constexpr (NST > 3) if (kt + 3 < nk) ktile(kt + 3, I3{}, N{});
      if constexpr (NST > 4) if (kt + 4 < nk) ktile(kt + 4, I4{}, N{});
      if constexpr (NST > 5) if (kt + 5 < nk) ktile(kt + 5, I5{}, N{});
    }
  }

  // Epilogue.  A lane holds four consecutive rows 4 g + r of column lane % 16
  // of each 16 x 16 tile.
  constexpr int WN = AN * 16;
  const int mw = m0 + wm * AM * 16, nw = n0 + wn * WN;   // the wave's block
  float colv[AN], gatev[AN];
#pragma unroll
  for (int j = 0; j < AN; ++j) {
    const int n = nw + j * 16 + col;
    colv[j] = 0.f;
    gatev[j] = 1.f;
    if (n < p.N) {
      if constexpr (GA == GA_ROWS) {
        const int r = p.rows[n];
        if (bias_sg && r >= 0) colv[j] = bias_sg[r];
      } else {
        if (bias_sg) colv[j] = bias_sg[n];
      }
      if (EPI == EPI_RESIDUAL && p.gate0) gatev[j] = p.gate0[n] + (p.gate1 ? p.gate1[n] : 0.f);
    }
  }
  if constexpr (EPI == EPI_STORE) {
    // transposed columns: the four rows are four consecutive tokens of one
    // dim, stored from the registers (a dim's 16 tokens are 32 contiguous
    // bytes of an instruction; the L2 merges the lines)
    if (p.vt && sg * p.N + n0 >= p.vt_col0) {
#pragma unroll
      for (int i = 0; i < AM; ++i) {
        const int m = mw + i * 16 + 4 * g;
#pragma unroll
        for (int j = 0; j < AN; ++j) {
          const int n = nw + j * 16 + col;
          if (n >= p.N || m >= p.M) continue;
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = acc[i][j][e] + colv[j];
          store_vt4(p, m, sg * p.N + n - p.vt_col0, v);
        }
      }
      return;
    }
  }
  // Otherwise through LDS, 16 rows at a time in the wave's own region of slot
  // 0 (rows padded by four floats: the four lane groups' rows fall in distinct
  // banks), so that a lane moves four consecutive elements of a row.
  constexpr int SW = WN + 4;
  static_assert((size_t)NW * 16 * SW * sizeof(float) <= sizeof(s0_), "epilogue staging");
  constexpr int LPR = WN / 4, RPT = 64 / LPR, NTR = 16 / RPT;   // lanes per row, rows per access
  float* stage = reinterpret_cast<float*>(&s0_[0][0]) + wave * (16 * SW);
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  const int nb = nw + (lane % LPR) * 4;
  const bool full4 = p.vec4 && nb + 4 <= p.N;
  // the residual's rows, all requested before the staging (unconditional
  // buffer loads; rows past M and ragged columns read zero)
  typedef typename std::conditional<std::is_same<OutT, float>::value, f32x4, bf16x4>::type Out4;
  constexpr bool RES = EPI == EPI_RESIDUAL;
  Out4 xres[RES ? AM : 1][RES ? NTR : 1];
  if constexpr (RES) {
    const __amdgpu_buffer_rsrc_t c_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        Csg + (int64_t)m0 * p.ldc, (short)0,
        (uint32_t)((int64_t)min(BM, p.M - m0) * p.ldc * (int64_t)sizeof(OutT)), kRsrcWord3);
    const uint32_t base = full4 ? (uint32_t)nb * (uint32_t)sizeof(OutT) : kMasked;
    const uint32_t row_bytes = (uint32_t)p.ldc * (uint32_t)sizeof(OutT);
#pragma unroll
    for (int i = 0; i < AM; ++i)
#pragma unroll
      for (int t = 0; t < NTR; ++t) {
        const uint32_t off = base + (uint32_t)(wm * AM * 16 + i * 16 + t * RPT + lane / LPR) * row_bytes;
        if constexpr (sizeof(Out4) == 8)
          xres[i][t] = __builtin_bit_cast(Out4, __builtin_amdgcn_raw_buffer_load_b64(c_rsrc, off, 0, 0));
        else
          xres[i][t] = __builtin_bit_cast(Out4, __builtin_amdgcn_raw_buffer_load_b128(c_rsrc, off, 0, 0));
      }
  }
  __syncthreads();   // slot 0 is free
#pragma unroll
  for (int i = 0; i < AM; ++i) {
#pragma unroll
    for (int j = 0; j < AN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float v = acc[i][j][r] + colv[j];
        if (EPI == EPI_GELU) v = gelu_tanh(v);
        if (EPI == EPI_RESIDUAL) v *= gatev[j];
        stage[(4 * g + r) * SW + j * 16 + col] = v;
      }
    wave_sync();
#pragma unroll
    for (int t = 0; t < NTR; ++t) {
      const int rl = t * RPT + lane / LPR;
      const int m = mw + i * 16 + rl;
      const f32x4 sv = *reinterpret_cast<const f32x4*>(&stage[rl * SW + (lane % LPR) * 4]);
      float v[4] = {sv[0], sv[1], sv[2], sv[3]};
      if (m >= p.M || nb >= p.N) continue;
      OutT* dst = Csg + (int64_t)m * p.ldc + nb;
      if (full4) {
        if constexpr (RES) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += (float)xres[i][t][e];
        }
        store4(dst, v);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (nb + e < p.N) {
            if (RES) v[e] += to_f32(dst[e]);
            dst[e] = from_f32<OutT>(v[e]);
          }
      }
    }
    if (i + 1 < AM) wave_sync();
  }
}

// ---------------------------------------------------------------------------
// Choice of the tile
// ---------------------------------------------------------------------------
// Tile shapes, largest first.  c1: microseconds per k-tile of a lone workgroup
// on each CU; cn: the same divided among several per CU; f: fixed cost of a
// round of tiles (prologue, first loads, epilogue); occ: workgroups a CU
// holds.  Measured on 128 .. 1024 tiles at K = 1024 and 4096 (bf16), 512 and
// 2048 (float32).  g: what a k-tile costs more in several rounds of a long
// reduction, where workgroups drift apart and share less of the L2 (bf16,
// 6000-24000 rows at K = 5120-12736; nothing at K = 1536).
struct TileShape {
  int bm, bn, occ;
  float c1, cn, f, g;
};
enum { TS_256 = 0, TS_224, TS_192, TS_160, TS_128W, TS_96W, TS_128, TS_96, TS_64, TS_64S, TS_32, TS_COUNT,
       TS_128D /* 128 x 128 in two slots, by a rule of its own */ };
template <typename T>
inline const TileShape* tile_shapes() {
  static constexpr TileShape bf[TS_COUNT] = {
      {256, 256, 1, 1.38f, 1.38f, 13.f, .10f},   {224, 256, 1, 1.23f, 1.23f, 11.f, .18f},
      {192, 256, 1, 1.075f, 1.075f, 10.f, .15f}, {160, 256, 1, 0.91f, 0.91f, 9.f, .13f},
      {128, 256, 1, 0.74f, 0.74f, 8.f, .21f},    {96, 256, 1, 0.605f, 0.605f, 7.f, .27f},
      {128, 128, 1, 0.475f, 0.475f, 7.5f, .25f}, {96, 128, 1, 0.36f, 0.36f, 6.f, .25f},
      {64, 128, 2, 0.31f, 0.31f, 5.f, .25f},     {64, 64, 2, 0.165f, 0.165f, 4.5f, .25f},
      {32, 32, 3, 0.075f, 0.07f, 5.f, .25f}};
  // (the wide tiles gain float32 nothing: the matrix rate bounds it)
  static constexpr TileShape f32[TS_COUNT] = {
      {}, {}, {}, {}, {}, {}, {}, {96, 128, 2, 1.33f, 1.30f, 6.f, 0.f}, {64, 128, 2, 0.90f, 0.86f, 6.f, 0.f},
      {64, 64, 2, 0.457f, 0.44f, 4.5f, 0.f}, {32, 32, 3, 0.132f, 0.117f, 4.2f, 0.f}};
  return sizeof(T) == 2 ? bf : f32;
}

// The tile shape of an M x N x K problem (nseg segments of N columns): the one
// with the least estimated time.  A CU's share is a whole number n of tiles,
// so the estimate is n tiles' k-loops plus the fixed cost of each round; a
// chip that is only part full runs its k-tiles faster (higher clock, less L2
// traffic: 0.75-0.95 of the time at half the CUs).  The choice does not look
// at the gather mode, nor at the epilogue but for the short reductions below.
template <typename T>
inline int pick_tile(int M, int N, int nseg, int K, int epi) {
  const TileShape* ts = tile_shapes<T>();
  const float nk = (float)(K / (128 / (int)sizeof(T)));
  // Store epilogues of up to eight k-tiles, 3/2 to 2 tiles of 128 x 128 per CU:
  // these in two ring slots, so that a CU holds two workgroups and one's loads and
  // stores run under the other's, where one workgroup of a wider tile per CU pays
  // its prologue and its stores in full (11683 x 528 x 384: 10.5 us, 12.3 on 128 x
  // 256; 6077 x 1047 x 320: 13.3 and 15.2; 53 problems of 8 to 20 us: 0.93 of the
  // time, worst 1.03).  With 9 to 14 k-tiles it is 0.94 to 1.06, from 23 on slower.
  // With fewer tiles only where 96 x 256 does not fit one round either.  With GELU
  // or the residual the wide tiles stay (742 x 7309 x 128: 22.2 us, 27.7).
  if (sizeof(T) == 2 && epi == EPI_STORE && nk <= 8.f) {
    auto count = [&](int bm, int bn) { return (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn) * nseg; };
    const int64_t tiles = count(128, 128);
    const bool many = 2 * tiles > 3 * kCus;
    const bool fewer = 3 * tiles > 4 * kCus && nk >= 4.f && count(96, 256) > kCus;
    if (tiles <= 2 * kCus && (many || fewer)) return TS_128D;
  }
  int best = TS_COUNT - 1;
  float tbest = 0.f;
  for (int i = 0; i < TS_COUNT; ++i) {
    const TileShape& t = ts[i];
    if (!t.bm) continue;
    const int64_t tiles = (int64_t)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) * nseg;
    const int64_t n = (tiles + kCus - 1) / kCus;
    const float fill = (float)tiles / (float)(n * kCus);
    const float rounds = (float)((n + t.occ - 1) / t.occ);
    const float longk = n == 1 ? 0.f : nk <= 24.f ? 0.f : nk >= 80.f ? 1.f : (nk - 24.f) / 56.f;
    const float est = nk * (n == 1 ? t.c1 : (float)n * t.cn) * (0.6f + 0.4f * fill) * (1.f + longk * t.g) +
                      t.f * (0.5f + 0.5f * rounds);
    // 256 x 256 unless another shape is better by more than the estimate errs: 2 %
    // per round, up to 8 % (under a long load the clock falls with the LDS reads
    // per flop: 13911 x 7076 x 1600, seven rounds, estimated 8 % better on 224 x
    // 256, took 347 us against 313), and 8 % for less than eight k-tiles, whose
    // rounds do not overlap (15747 x 988 x 64: 15.8 us on 128 x 256 against 14.2).
    const float margin = nk < 8.f ? 0.08f : 0.02f * (n < 4 ? (float)n : 4.f);
    const float bias = i == TS_256 ? 1.f - margin : 1.f;
    if (tbest == 0.f || est * bias < tbest) {
      tbest = est * bias;
      best = i;
    }
  }
  return best;
}

template <typename T, typename OutT, int EPI, int GA, int WGM, int WGN, int AM, int AN, int NST, int OCC>
void launch_ring_cfg(const GemmParams<T, OutT>& p, hipStream_t stream) {
  constexpr int BM = WGM * AM * 16, BN = WGN * AN * 16;
  const int tiles = ((p.M + BM - 1) / BM) * ((p.N + BN - 1) / BN) * p.nseg;
  const size_t dyn = GA == GA_KCH ? (size_t)(p.K / Chunk<T>::VEC) * sizeof(uint16_t) : 0;
  hipLaunchKernelGGL((gemm_ring_kernel<T, OutT, EPI, GA, WGM, WGN, AM, AN, NST, OCC>), dim3(tiles),
                     dim3(64 * WGM * WGN), dyn, stream, p);
}

template <typename T, typename OutT, int EPI, int GA>
hipError_t launch_ring_shape(int shape, const GemmParams<T, OutT>& p, hipStream_t s) {
  if constexpr (sizeof(T) == 2) {
    // (three 160 x 256 slots leave 4 KB for the chunk table; 128 x 256, 16 KB,
    // fits the longest)
    if (GA == GA_KCH && shape == TS_160 && p.K / Chunk<T>::VEC > 2048) shape = TS_128W;
    switch (shape) {
      case TS_256:
        // gathered B; the largest plain problems run gemm.hip
        if constexpr (GA != GA_NONE) launch_ring_cfg<T, OutT, EPI, GA, 2, 4, 8, 4, 2, 1>(p, s);
        else return hipErrorInvalidValue;
        break;
      case TS_224: launch_ring_cfg<T, OutT, EPI, GA, 2, 4, 7, 4, 2, 1>(p, s); break;
      case TS_192: launch_ring_cfg<T, OutT, EPI, GA, 2, 4, 6, 4, 2, 1>(p, s); break;
      case TS_160: launch_ring_cfg<T, OutT, EPI, GA, 2, 4, 5, 4, 3, 1>(p, s); break;
      case TS_128W: launch_ring_cfg<T, OutT, EPI, GA, 2, 4, 4, 4, 3, 1>(p, s); break;
      case TS_96W: launch_ring_cfg<T, OutT, EPI, GA, 2, 4, 3, 4, 3, 1>(p, s); break;
      case TS_128: launch_ring_cfg<T, OutT, EPI, GA, 2, 2, 4, 4, 4, 2>(p, s); break;
      case TS_128D:
        if constexpr (EPI == EPI_STORE) launch_ring_cfg<T, OutT, EPI, GA, 2, 2, 4, 4, 2, 2>(p, s);
        else return hipErrorInvalidValue;
        break;
      case TS_96: launch_ring_cfg<T, OutT, EPI, GA, 2, 2, 3, 4, 5, 2>(p, s); break;
      case TS_64: launch_ring_cfg<T, OutT, EPI, GA, 2, 2, 2, 4, 3, 2>(p, s); break;
      case TS_64S: launch_ring_cfg<T, OutT, EPI, GA, 2, 2, 2, 2, 4, 2>(p, s); break;
      case TS_32: launch_ring_cfg<T, OutT, EPI, GA, 2, 2, 1, 1, 6, 3>(p, s); break;
      default: return hipErrorInvalidValue;
    }
  } else {
    switch (shape) {
      case TS_96: launch_ring_cfg<T, OutT, EPI, GA, 2, 2, 3, 4, 2, 2>(p, s); break;
      case TS_64: launch_ring_cfg<T, OutT, EPI, GA, 2, 2, 2, 4, 3, 2>(p, s); break;
      case TS_64S: launch_ring_cfg<T, OutT, EPI, GA, 2, 2, 2, 2, 4, 2>(p, s); break;
      case TS_32: launch_ring_cfg<T, OutT, EPI, GA, 2, 2, 1, 1, 6, 3>(p, s); break;
      default: return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

// (epi, gather mode) as launch_gemm validated them; one source per (T, OutT)
template <typename T, typename OutT>
hipError_t launch_gemm_ring(int shape, const GemmParams<T, OutT>& p, int epi, int ga, hipStream_t s);

#define DIF_RING_INSTANCE(T, OutT)                                                               \
  template <>                                                                                    \
  hipError_t launch_gemm_ring<T, OutT>(int shape, const GemmParams<T, OutT>& p, int epi, int ga, \
                                       hipStream_t s) {                                          \
    constexpr bool kGather = std::is_same<T, OutT>::value;                                       \
    if (ga == GA_NONE)                                                                           \
      return epi == EPI_STORE  ? launch_ring_shape<T, OutT, EPI_STORE, GA_NONE>(shape, p, s)     \
             : epi == EPI_GELU ? launch_ring_shape<T, OutT, EPI_GELU, GA_NONE>(shape, p, s)      \
                               : launch_ring_shape<T, OutT, EPI_RESIDUAL, GA_NONE>(shape, p, s); \
    if constexpr (kGather) {                                                                     \
      if (ga == GA_KCH) return launch_ring_shape<T, OutT, EPI_RESIDUAL, GA_KCH>(shape, p, s);    \
      return epi == EPI_GELU ? launch_ring_shape<T, OutT, EPI_GELU, GA_ROWS>(shape, p, s)        \
                             : launch_ring_shape<T, OutT, EPI_STORE, GA_ROWS>(shape, p, s);      \
    }                                                                                            \
    return hipErrorInvalidValue;                                                                 \
  }

}  // namespace dif
