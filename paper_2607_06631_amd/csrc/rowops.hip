// HBM-bound row kernels for gfx950: LayerNorm + AdaLN modulation,
// QK RMSNorm + 3D RoPE, plan-time gather, timestep GEMV and
// small elementwise steps.  Rows are read once with 16-byte vector loads,
// kept in registers between the statistics and the apply pass, and written
// once; statistics are fp32 whatever the storage type.
#include <algorithm>
#include <initializer_list>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace dif {

constexpr int R_THREADS = 256;
constexpr int R_WAVES = R_THREADS / kWave;
constexpr int R_MAXC = 16;   // 16-byte chunks per lane per row (D <= 1024 * VEC)

// ---------------------------------------------------------------------------
// LayerNorm (biased variance, eps) + AdaLN modulation or affine.
// The workgroup first folds the per-column vectors into LDS (shift and
// 1 + scale, or weight and bias) while its waves' first rows are on their way;
// each wave then normalises its rows, one at a time: one statistics pass (sum
// and sum of squares of the row shifted by its first element) with the row kept
// packed in registers, then the apply pass.  Reductions are wave-local.
// ---------------------------------------------------------------------------
// The row kernels that stage per-column vectors in LDS run up to 16 waves of 8
// rows per workgroup, so the staging is shared by 128 rows (measured: 4.6 TB/s
// vs 3.3 TB/s with 4 waves on [32760, 5120] bf16).
constexpr int NORM_WAVES = 16;
constexpr int NORM_RPW = 8;

// Rows per wave and waves per workgroup of the row kernels: about one workgroup
// per CU, first by fewer rows per wave, then by fewer waves, never more than
// the given maxima.  With 128 rows per workgroup whatever the row count, 1560
// rows ran on 13 CUs and a wave's rows one after another: LayerNorm of
// [1560, 5120] bf16 took 54 us (11 now), the q / k norm of 2 x [390, 4096]
// 78 us (13).
struct RowSplit {
  int waves, rpw;
};
inline RowSplit row_split(int64_t rows, int max_waves, int max_rpw) {
  const int64_t per = (rows + kCus - 1) / kCus;   // rows per workgroup
  if (per >= (int64_t)max_waves * max_rpw) return {max_waves, max_rpw};
  if (per >= max_waves) return {max_waves, (int)((per + max_waves - 1) / max_waves)};
  int w = 2;
  while (w < per) w *= 2;
  return {w < max_waves ? w : max_waves, 1};
}

// Staging of n per-column values (n a multiple of 4) by the whole workgroup,
// four columns per thread and access: load(c) gives the values of columns
// c .. c + 3, store(c, values) puts them in LDS.  A thread's U loads go out
// together (columns past the end repeat the last four, so there is no branch
// between them): with one turn at a time each was a memory round trip, ten in a
// row for 5120 columns and two waves.
template <int N>
struct ColVecs {
  f32x4 v[N];
};
template <int U, typename Load, typename Store>
__device__ __forceinline__ void stage_columns(int n, Load&& load, Store&& store) {
  const int stride = blockDim.x * 4;
  for (int c0 = threadIdx.x * 4; c0 < n; c0 += U * stride) {
    decltype(load(0)) v[U];
    int c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      c[u] = min(c0 + u * stride, n - 4);
      v[u] = load(c[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) store(c[u], v[u]);
  }
}

// Whether every non-null pointer allows 16-byte accesses.
inline bool aligned16(std::initializer_list<const void*> ps) {
  uintptr_t u = 0;
  for (const void* p : ps) u |= reinterpret_cast<uintptr_t>(p);
  return u % 16 == 0;
}

// 16-byte chunks each lane holds for a row of D elements, rounded up to one
// of the instantiated register budgets (4, 8, 12, 16); 0 if D is too wide.
template <typename T>
inline int chunks_per_lane(int D) {
  const int c = (D / Chunk<T>::VEC + kWave - 1) / kWave;
  return c <= 4 ? 4 : c <= 8 ? 8 : c <= 12 ? 12 : c <= R_MAXC ? R_MAXC : 0;
}
// vec: every per-column vector is there and allows 16-byte loads (D is a
// multiple of 64).
template <typename T, int MAXC>
__global__ __launch_bounds__(64 * NORM_WAVES) void norm_kernel(const T* __restrict__ x, T* __restrict__ y,
                                                         int M, int D, int mode, const float* p0,
                                                         const float* p1, const float* p2,
                                                         const float* p3, float eps, int rpw, int vec) {
  constexpr int VEC = Chunk<T>::VEC;
  extern __shared__ float vec_lds[];  // [2][D]: multiplier, addend
  float* mul = vec_lds;
  float* add = vec_lds + D;
  const int lane = threadIdx.x & 63;
  const int nch = D / VEC;
  const int nwaves = blockDim.x >> 6;
  const int64_t row0 = ((int64_t)blockIdx.x * nwaves + (threadIdx.x >> 6)) * rpw;
  u32x4 raw[MAXC];
  auto load_row = [&](int64_t row) {
    const T* xr = x + row * D;
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
      const int c = lane + kWave * i;
      if (c < nch) raw[i] = *reinterpret_cast<const u32x4*>(xr + c * VEC);
    }
  };
  // (16 chunks per lane leave no registers to hold a row meanwhile)
  constexpr bool AHEAD = MAXC <= 12;
  if (AHEAD && row0 < M) load_row(row0);
  auto ld4 = [](const float* p) { return *reinterpret_cast<const f32x4*>(p); };
  // (three columns' loads at a time beside a row of 12 chunks: four spilled two
  // registers; two are as fast on vectors in the L2, but 0.5 us a launch behind on
  // cold ones with few rows)
  constexpr int U = MAXC == 12 ? 3 : 4;
  if (vec && mode == 0) {
    stage_columns<U>(D, [&](int n) { return ColVecs<4>{ld4(p0 + n), ld4(p1 + n), ld4(p2 + n), ld4(p3 + n)}; },
                     [&](int n, const ColVecs<4>& v) {
                       *reinterpret_cast<f32x4*>(mul + n) = 1.f + v.v[2] + v.v[3];
                       *reinterpret_cast<f32x4*>(add + n) = v.v[0] + v.v[1];
                     });
  } else if (vec) {
    stage_columns<4>(D, [&](int n) { return ColVecs<2>{ld4(p0 + n), ld4(p1 + n)}; },
                     [&](int n, const ColVecs<2>& v) {
                       *reinterpret_cast<f32x4*>(mul + n) = v.v[0];
                       *reinterpret_cast<f32x4*>(add + n) = v.v[1];
                     });
  } else {
    for (int n = threadIdx.x; n < D; n += blockDim.x) {
      if (mode == 0) {
        mul[n] = 1.f + p2[n] + (p3 ? p3[n] : 0.f);
        add[n] = p0[n] + (p1 ? p1[n] : 0.f);
      } else {
        mul[n] = p0[n];
        add[n] = p1[n];
      }
    }
  }
  __syncthreads();
  const float inv_d = 1.f / (float)D;
  for (int rr = 0; rr < rpw; ++rr) {
    const int64_t row = row0 + rr;
    if (row >= M) break;
    if (!AHEAD || rr > 0) load_row(row);
    // one pass over shifted data: sum and sum of squares of (x - x0), where
    // x0 is the row's first element, keep the variance free of cancellation
    const float x0 = to_f32(x[row * D]);
    float s = 0.f, ss = 0.f;
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
      const int c = lane + kWave * i;
      if (c < nch) {
        float v[VEC];
        Chunk<T>::unpack(raw[i], v);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const float d = v[e] - x0;
          s += d;
          ss += d * d;
        }
      }
    }
    const float ms = wave_sum(s) * inv_d;
    const float mean = x0 + ms;
    const float var = fmaxf(wave_sum(ss) * inv_d - ms * ms, 0.f);
    const float rstd = rsqrtf(var + eps);
    T* yr = y + row * D;
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
      const int c = lane + kWave * i;
      if (c < nch) {
        float v[VEC], out[VEC];
        Chunk<T>::unpack(raw[i], v);
        const f32x4* m4 = reinterpret_cast<const f32x4*>(mul + c * VEC);
        const f32x4* a4 = reinterpret_cast<const f32x4*>(add + c * VEC);
#pragma unroll
        for (int q = 0; q < VEC / 4; ++q) {
          const f32x4 mu = m4[q], ad = a4[q];
#pragma unroll
          for (int e = 0; e < 4; ++e) out[4 * q + e] = (v[4 * q + e] - mean) * rstd * mu[e] + ad[e];
        }
        *reinterpret_cast<u32x4*>(yr + c * VEC) = Chunk<T>::pack(out);
      }
      __builtin_amdgcn_sched_barrier(0);  // bound the LDS reads kept in flight
    }
  }
}

template <typename T>
hipError_t launch_norm(const T* x, T* y, int M, int D, int mode, const float* p0, const float* p1,
                       const float* p2, const float* p3, float eps, hipStream_t stream) {
  if (M <= 0) return hipSuccess;
  const RowSplit rs = row_split(M, NORM_WAVES, NORM_RPW);
  const int rows_per_wg = rs.waves * rs.rpw;
  const dim3 grid((M + rows_per_wg - 1) / rows_per_wg), block(64 * rs.waves);
  const size_t lds = 2 * D * sizeof(float);
  const int vec = p0 && p1 && (mode != 0 || (p2 && p3)) && aligned16({p0, p1, p2, p3});
  auto launch = [&](auto c_tag) {
    hipLaunchKernelGGL((norm_kernel<T, decltype(c_tag)::value>), grid, block, lds, stream, x, y, M, D,
                       mode, p0, p1, p2, p3, eps, rs.rpw, vec);
  };
  switch (chunks_per_lane<T>(D)) {
    case 4: launch(std::integral_constant<int, 4>{}); break;
    case 8: launch(std::integral_constant<int, 8>{}); break;
    case 12: launch(std::integral_constant<int, 12>{}); break;
    case 16: launch(std::integral_constant<int, 16>{}); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// QK RMSNorm over the full model width (pruned channels count as zeros, so
// the sum of squares of the kept channels is divided by D) + 3D RoPE.
// Gains are staged in LDS once per workgroup.  Lane l always covers the
// same head-local pairs (64 * VEC is a multiple of head_dim), so its
// rotation factors are fetched once per row.  A wave issues the loads of
// both segments (q and k) of its row before the first reduction waits on
// them, with the rotation-table reads in their shadow.
// ---------------------------------------------------------------------------
constexpr int QK_WAVES = 8;    // 16 KB of loads in flight per wave; registers for both segments
// Rows per wave where there are rows enough for a workgroup per CU.  One
// segment: 4, so 32760 video tokens make 1024 workgroups, several per CU, with
// more rows' loads in flight (5.3 TB/s; 16 rows per wave, one workgroup per CU,
// reached 4.2).  Two segments (q and k, twice the loads per row): 16 (5.4-5.5
// TB/s against 5.3 with 4).  Below that 4 (two segments), then 1, the latter
// with fewer waves per workgroup (row_split).  (Rows of 16 chunks per lane: 1,
// the registers of several spill.)
template <int NSEG, int MAXC>
constexpr int qk_rpw() { return NSEG == 2 ? 16 : MAXC > 12 ? 1 : 4; }
// A rotated pair is (x0 cos - x1 sin, x0 sin + x1 cos), each with one product
// rounded and the other inside a fused multiply-add, written out so that the
// result does not hang on which product the compiler fuses (left to it, instances
// of one width differed with their rows per wave and between builds).  The first
// coordinate rounds x1 sin; the second rounds x0 sin in the instances named here
// and x1 cos in the others, which is what each width has always returned.
template <typename T, int MAXC, int NSEG>
constexpr bool qk_rounds_x0() {
  return MAXC == 16 || (MAXC == 12 && sizeof(T) == 2) || (MAXC == 8 && NSEG == 2);
}
template <typename T, int MAXC, int NSEG, int RPW>
__global__ __launch_bounds__(64 * QK_WAVES) void qk_norm_kernel(T* buf, int64_t ld, int rows, int a,
                                                            int nseg, int off0, int off1,
                                                            const float* g0, const float* g1,
                                                            const int32_t* gidx, float scale0,
                                                            float inv_dim, float eps, RopeDesc rope,
                                                            int vec, int nb1) {
  constexpr int VEC = Chunk<T>::VEC;
  constexpr int NP = VEC / 2;  // pairs per chunk
  extern __shared__ float gain_lds[];  // [nseg][a]
  const int lane = threadIdx.x & 63;
  const int nch = a / VEC;
  const int jb = ((lane * VEC) % rope.head_dim) / 2;  // first head-local pair of this lane
  const int nwaves = blockDim.x >> 6;
  // the first nb1 workgroups take the descriptor's second row set (so its few
  // rows do not end the launch), the others the rows of buf, in place
  const bool second = NSEG == 1 && (int)blockIdx.x < nb1;
  const int64_t row0 = ((int64_t)(blockIdx.x - (second ? 0 : nb1)) * nwaves + (threadIdx.x >> 6)) * RPW;
  const T* src = second ? static_cast<const T*>(rope.src1) : buf;
  const int64_t lds = second ? rope.lds1 : ld;
  const int32_t* sidx = second ? rope.src_idx1 : nullptr;
  if (second) {
    rows = rope.rows1;
    g0 = rope.gain1;
    scale0 = 1.f;
  }
  // both segments' loads of a row together (idx: columns of the second set)
  auto load_row = [&](int64_t row, u32x4 (&to)[NSEG][MAXC], const int32_t* idx) __attribute__((always_inline)) {
#pragma unroll
    for (int sg = 0; sg < NSEG; ++sg) {
      const T* xr = src + row * lds + (sg == 0 ? off0 : off1);
#pragma unroll
      for (int i = 0; i < MAXC; ++i) {
        const int c = lane + kWave * i;
        if (c < nch) {
          const int at = idx ? idx[c * VEC] : c * VEC;
          to[sg][i] = *reinterpret_cast<const u32x4*>(xr + at);
        }
      }
    }
  };
  // a lone row is on its way during the staging; of several, the compiler
  // overlaps one's loads with the others' work (RPW is a constant for that:
  // with a run-time count the wide two-segment launch took 312 us, not 170)
  u32x4 lone[NSEG][MAXC];
  if constexpr (RPW == 1) {
    if (row0 < rows) load_row(row0, lone, sidx);
  }
  auto ld4 = [](const float* p) { return *reinterpret_cast<const f32x4*>(p); };
  if (vec) {   // 16-byte gain loads (a is whole heads, and so are the runs of a gain table)
    stage_columns<4>(
        a,
        [&](int n) {
          const int gn = gidx ? gidx[n] : n;
          ColVecs<NSEG> v;
          v.v[0] = ld4(g0 + gn) * scale0;
          if constexpr (NSEG > 1) v.v[1] = ld4(g1 + gn);
          return v;
        },
        [&](int n, const ColVecs<NSEG>& v) {
          *reinterpret_cast<f32x4*>(gain_lds + n) = v.v[0];
          if constexpr (NSEG > 1) *reinterpret_cast<f32x4*>(gain_lds + a + n) = v.v[1];
        });
  } else {
    for (int n = threadIdx.x; n < a; n += blockDim.x) {
      const int gn = gidx ? gidx[n] : n;
      gain_lds[n] = g0[gn] * scale0;
      if (nseg > 1) gain_lds[a + n] = g1[gn];
    }
  }
  __syncthreads();
  auto work = [&](int64_t row, const u32x4 (&raw)[NSEG][MAXC], T* dst, int64_t ldd) __attribute__((always_inline)) {
    // rotation factors of this lane's pairs (table reads overlap the loads)
    float cs[NP], sn[NP];
    if (rope.table) {
      const int n = (int)(row % rope.L);
      const int pw = n % rope.gw, pr = (n / rope.gw) % rope.gh, pf = n / (rope.gw * rope.gh);
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        const int j = jb + k;
        int idx;
        if (j < rope.jt) {
          idx = pf * rope.jt + j;
        } else if (j < rope.jt + rope.jh) {
          idx = rope.gf * rope.jt + pr * rope.jh + (j - rope.jt);
        } else {
          idx = rope.gf * rope.jt + rope.gh * rope.jh + pw * rope.jw + (j - rope.jt - rope.jh);
        }
        cs[k] = rope.table[2 * idx];
        sn[k] = rope.table[2 * idx + 1];
      }
    }
    float rstd[NSEG];
#pragma unroll
    for (int sg = 0; sg < NSEG; ++sg) {
      float ss = 0.f;
#pragma unroll
      for (int i = 0; i < MAXC; ++i) {
        const int c = lane + kWave * i;
        if (c < nch) {
          float v[VEC];
          Chunk<T>::unpack(raw[sg][i], v);
#pragma unroll
          for (int e = 0; e < VEC; ++e) ss += v[e] * v[e];
        }
      }
      rstd[sg] = rsqrtf(wave_sum(ss) * inv_dim + eps);
    }
#pragma unroll
    for (int sg = 0; sg < NSEG; ++sg) {
      T* xr = dst + row * ldd + (sg == 0 ? off0 : off1);
      const float* gain = gain_lds + sg * a;
#pragma unroll
      for (int i = 0; i < MAXC; ++i) {
        const int c = lane + kWave * i;
        if (c < nch) {
          float out[VEC];
          Chunk<T>::unpack(raw[sg][i], out);
          const f32x4* g4 = reinterpret_cast<const f32x4*>(gain + c * VEC);
#pragma unroll
          for (int q = 0; q < VEC / 4; ++q) {
            const f32x4 gg = g4[q];
#pragma unroll
            for (int e = 0; e < 4; ++e) out[4 * q + e] *= rstd[sg] * gg[e];
          }
          if (rope.table) {
#pragma unroll
            for (int k = 0; k < NP; ++k) {
              const float x0 = out[2 * k], x1 = out[2 * k + 1];
              out[2 * k] = fmaf(x0, cs[k], -(x1 * sn[k]));
              if constexpr (qk_rounds_x0<T, MAXC, NSEG>()) out[2 * k + 1] = fmaf(x1, cs[k], x0 * sn[k]);
              else out[2 * k + 1] = fmaf(x0, sn[k], x1 * cs[k]);
            }
          }
          *reinterpret_cast<u32x4*>(xr + c * VEC) = Chunk<T>::pack(out);
        }
      }
    }
  };
  if constexpr (RPW == 1) {
    if (row0 < rows)
      work(row0, lone, second ? static_cast<T*>(rope.dst1) : buf, second ? rope.ldd1 : ld);
  } else {
    if (NSEG == 1 && second) {
#pragma unroll 1   // (few rows; the loop below sets the kernel's registers)
      for (int rr = 0; rr < RPW; ++rr) {
        u32x4 raw[NSEG][MAXC];
        if (row0 + rr >= rows) break;
        load_row(row0 + rr, raw, sidx);
        work(row0 + rr, raw, static_cast<T*>(rope.dst1), rope.ldd1);
      }
      return;
    }
    for (int rr = 0; rr < RPW; ++rr) {
      u32x4 raw[NSEG][MAXC];
      if (row0 + rr >= rows) break;
      load_row(row0 + rr, raw, nullptr);
      work(row0 + rr, raw, buf, ld);
    }
  }
}

template <typename T>
hipError_t launch_qk_norm(T* buf, int64_t ld, int rows, int a, int nseg, int off0, int off1,
                          const float* g0, const float* g1, float inv_norm_dim, float eps,
                          const RopeDesc* rope, hipStream_t stream, const int32_t* gain_idx,
                          float scale0) {
  if (rows <= 0 || a <= 0) return hipSuccess;
  RopeDesc rd{};
  if (rope) rd = *rope;
  if (rd.head_dim <= 0) rd.head_dim = 64;   // no rotation: any width dividing 64 * VEC
  constexpr int VEC = Chunk<T>::VEC;
  if ((64 * VEC) % rd.head_dim != 0) return hipErrorInvalidValue;
  const int vec = aligned16({g0, g1, rd.gain1});
  if (rd.rows1 > 0 && (nseg != 1 || rd.table || !rd.src1 || !rd.dst1 || !rd.gain1 ||
                       !aligned16({rd.src1, rd.dst1}) || rd.lds1 % VEC || rd.ldd1 % VEC))
    return hipErrorInvalidValue;
  // q and k in one launch while both fit the registers (up to 8 chunks per
  // lane), else one launch per segment
  auto launch = [&](auto c_tag, auto nseg_tag, int off_a, int off_b, const float* ga,
                    const float* gb, float sa) {
    constexpr int C = decltype(c_tag)::value, NS = decltype(nseg_tag)::value;
    const RowSplit rs = row_split(rows, QK_WAVES, qk_rpw<NS, C>());
    auto go = [&](auto rpw_tag) {
      constexpr int RPW = decltype(rpw_tag)::value;
      const int rows_per_wg = rs.waves * RPW;
      const int nb1 = (rd.rows1 + rows_per_wg - 1) / rows_per_wg;
      const dim3 grid((rows + rows_per_wg - 1) / rows_per_wg + nb1);
      hipLaunchKernelGGL((qk_norm_kernel<T, C, NS, RPW>), grid, dim3(64 * rs.waves),
                         NS * a * sizeof(float), stream, buf, ld, rows, a, NS, off_a, off_b, ga, gb,
                         gain_idx, sa, inv_norm_dim, eps, rd, vec, nb1);
    };
    if (rs.rpw == qk_rpw<NS, C>()) {
      go(std::integral_constant<int, qk_rpw<NS, C>()>{});
      return;
    }
    if constexpr (NS == 2) {
      if (rs.rpw >= 4) {
        go(std::integral_constant<int, 4>{});
        return;
      }
    }
    go(std::integral_constant<int, 1>{});
  };
  auto by_chunks = [&](auto c_tag) {
    constexpr int C = decltype(c_tag)::value;
    using One = std::integral_constant<int, 1>;
    using Two = std::integral_constant<int, 2>;
    if (nseg == 1) {
      launch(c_tag, One{}, off0, 0, g0, nullptr, scale0);
      return;
    }
    if constexpr (C <= 8) {
      launch(c_tag, Two{}, off0, off1, g0, g1, scale0);
    } else {
      launch(c_tag, One{}, off0, 0, g0, nullptr, scale0);
      launch(c_tag, One{}, off1, 0, g1, nullptr, 1.f);
    }
  };
  switch (chunks_per_lane<T>(a)) {
    case 4: by_chunks(std::integral_constant<int, 4>{}); break;
    case 8: by_chunks(std::integral_constant<int, 8>{}); break;
    case 12: by_chunks(std::integral_constant<int, 12>{}); break;
    case 16: by_chunks(std::integral_constant<int, 16>{}); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// plan-time gather of kept rows / columns
// ---------------------------------------------------------------------------
// Element by element: whatever the widths, strides and addresses.
template <typename T>
__global__ __launch_bounds__(R_THREADS) void gather_kernel(const T* __restrict__ src, int64_t lds,
                                                           T* __restrict__ dst, int64_t ldd,
                                                           int cols, const int32_t* ridx,
                                                           const int32_t* cidx) {
  const int64_t r = blockIdx.x;
  const int sr = ridx ? ridx[r] : (int)r;
  for (int c = threadIdx.x; c < cols; c += R_THREADS) {
    const int sc = cidx ? cidx[c] : c;
    T v = from_f32<T>(0.f);
    if (sr >= 0 && sc >= 0) v = src[(int64_t)sr * lds + sc];
    dst[r * ldd + c] = v;
  }
}

// One vector of kept entries (biases, gains): dst[r] = src[ridx[r]].
template <typename T>
__global__ __launch_bounds__(R_THREADS) void gather_vec_kernel(const T* __restrict__ src,
                                                               T* __restrict__ dst, int rows,
                                                               const int32_t* __restrict__ ridx) {
  const int r = blockIdx.x * R_THREADS + threadIdx.x;
  if (r >= rows) return;
  const int sr = ridx[r];
  dst[r] = sr >= 0 ? src[sr] : from_f32<T>(0.f);
}

// HBM-bound: a lane writes the same 16-byte vector of G_ROWS destination rows.
// Its column indices are read once; where they are consecutive and start on a
// vector (kept heads, kept chunks of 8 channels) each row is one 16-byte load,
// all G_ROWS in flight together, else V element loads.  (One element per lane
// and turn moved 1.1 TB/s: Wo of 32 kept heads, [5120, 4096] bf16, 77 us; 16 us now,
// and 4.3-4.6 TB/s over the rows of Wq and the chunks of W2.)
// src_vec: the source's rows start on 16-byte boundaries.
constexpr int G_ROWS = 8, G_THREADS = 128;
template <typename T, bool COLS>
__global__ __launch_bounds__(G_THREADS) void gather16_kernel(const T* __restrict__ src, int64_t lds,
                                                             T* __restrict__ dst, int64_t ldd,
                                                             int rows, int nvec,
                                                             const int32_t* __restrict__ ridx,
                                                             const int32_t* __restrict__ cidx,
                                                             int src_vec) {
  constexpr int V = 16 / sizeof(T);
  typedef T TV __attribute__((ext_vector_type(V)));
  const int q = blockIdx.x * G_THREADS + threadIdx.x;
  if (q >= nvec) return;
  const int r0 = blockIdx.y * G_ROWS, nr = min(G_ROWS, rows - r0);
  int c[V];
  bool run = src_vec;
#pragma unroll
  for (int e = 0; e < V; ++e) {
    c[e] = COLS ? cidx[q * V + e] : q * V + e;
    if (COLS) run = run && c[e] == c[0] + e;
  }
  if (COLS) run = run && c[0] >= 0 && c[0] % V == 0;
  int sr[G_ROWS];
#pragma unroll
  for (int k = 0; k < G_ROWS; ++k) sr[k] = r0 + min(k, nr - 1);
  if (ridx) {
#pragma unroll
    for (int k = 0; k < G_ROWS; ++k) sr[k] = ridx[sr[k]];
  }
  // (no branch around a load: dropped entries read entry 0 and are then zeroed,
  // so all loads go out before the first is waited for)
  u32x4 v[G_ROWS];
  if (run) {
#pragma unroll
    for (int k = 0; k < G_ROWS; ++k)
      v[k] = *reinterpret_cast<const u32x4*>(src + (int64_t)max(sr[k], 0) * lds + c[0]);
  } else {
    T x[G_ROWS][V];
#pragma unroll
    for (int k = 0; k < G_ROWS; ++k)
#pragma unroll
      for (int e = 0; e < V; ++e) x[k][e] = src[(int64_t)max(sr[k], 0) * lds + max(c[e], 0)];
#pragma unroll
    for (int k = 0; k < G_ROWS; ++k) {
      TV y;
#pragma unroll
      for (int e = 0; e < V; ++e) y[e] = c[e] >= 0 ? x[k][e] : from_f32<T>(0.f);
      v[k] = __builtin_bit_cast(u32x4, y);
    }
  }
#pragma unroll
  for (int k = 0; k < G_ROWS; ++k)
    if (sr[k] < 0) v[k] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
  for (int k = 0; k < G_ROWS; ++k)
    if (k < nr) *reinterpret_cast<u32x4*>(dst + (int64_t)(r0 + k) * ldd + (int64_t)q * V) = v[k];
}

template <typename T>
hipError_t launch_gather(const T* src, int64_t lds, T* dst, int64_t ldd, int rows, int cols,
                         const int32_t* ridx, const int32_t* cidx, hipStream_t stream) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  constexpr int V = 16 / sizeof(T);
  if (cols == 1 && lds == 1 && ldd == 1 && ridx && !cidx) {
    hipLaunchKernelGGL((gather_vec_kernel<T>), dim3((rows + R_THREADS - 1) / R_THREADS), dim3(R_THREADS),
                       0, stream, src, dst, rows, ridx);
    return hipGetLastError();
  }
  // whole destination vectors (the plan's matrices always; a caller's reordered
  // weights may start or end anywhere)
  const unsigned gy = (unsigned)((rows + G_ROWS - 1) / G_ROWS);
  if (cols % V == 0 && ldd % V == 0 && reinterpret_cast<uintptr_t>(dst) % 16 == 0 && gy <= 65535) {
    const int nvec = cols / V;
    const dim3 grid((unsigned)((nvec + G_THREADS - 1) / G_THREADS), gy);
    const int src_vec = lds % V == 0 && reinterpret_cast<uintptr_t>(src) % 16 == 0;
    if (cidx)
      hipLaunchKernelGGL((gather16_kernel<T, true>), grid, dim3(G_THREADS), 0, stream, src, lds, dst, ldd,
                         rows, nvec, ridx, cidx, src_vec);
    else
      hipLaunchKernelGGL((gather16_kernel<T, false>), grid, dim3(G_THREADS), 0, stream, src, lds, dst, ldd,
                         rows, nvec, ridx, cidx, src_vec);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((gather_kernel<T>), dim3(rows), dim3(R_THREADS), 0, stream, src, lds, dst, ldd,
                     cols, ridx, cidx);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Kept heads of the cached V^T, 16 bytes per lane:
//   dst[b, r, :] = src[b, idx[r], :]        (r < rows, n per row)
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(R_THREADS) void gather_rows16_kernel(const T* __restrict__ src,
                                                                  int64_t src_bs, T* __restrict__ dst,
                                                                  int64_t dst_bs, int64_t ld, int rows,
                                                                  const int32_t* __restrict__ idx) {
  constexpr int V = 16 / sizeof(T);
  const int64_t nvec = ld / V;
  const int64_t i = (int64_t)blockIdx.x * R_THREADS + threadIdx.x;
  if (i >= (int64_t)rows * nvec) return;
  const int64_t r = i / nvec, q = i - r * nvec;
  const int64_t b = blockIdx.y;
  *reinterpret_cast<u32x4*>(dst + b * dst_bs + r * ld + q * V) =
      *reinterpret_cast<const u32x4*>(src + b * src_bs + (int64_t)idx[r] * ld + q * V);
}

template <typename T>
hipError_t launch_gather_rows16(const T* src, int64_t src_bs, T* dst, int64_t dst_bs, int64_t ld,
                                int rows, int batches, const int32_t* idx, hipStream_t stream) {
  constexpr int V = 16 / sizeof(T);
  if (rows <= 0 || batches <= 0 || ld <= 0) return hipSuccess;
  if (ld % V || src_bs % V || dst_bs % V || reinterpret_cast<uintptr_t>(src) % 16 ||
      reinterpret_cast<uintptr_t>(dst) % 16)
    return hipErrorInvalidValue;
  const int64_t total = (int64_t)rows * (ld / V);
  hipLaunchKernelGGL((gather_rows16_kernel<T>),
                     dim3((unsigned)((total + R_THREADS - 1) / R_THREADS), (unsigned)batches),
                     dim3(R_THREADS), 0, stream, src, src_bs, dst, dst_bs, ld, rows, idx);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// FFN channel norms: sqrt(|W1[j, :]|^2 + b1[j]^2 + |W2[:, j]|^2), in double
// (one-time preprocessing; a thread per channel, W2 reads coalesced over j)
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(R_THREADS) void ffn_norms_kernel(const T* __restrict__ w1,
                                                              const float* __restrict__ b1,
                                                              const T* __restrict__ w2, int D, int F,
                                                              double* __restrict__ out) {
  const int j = blockIdx.x * R_THREADS + threadIdx.x;
  if (j >= F) return;
  double acc = (double)b1[j] * (double)b1[j];
  for (int d = 0; d < D; ++d) {
    const double v = (double)to_f32(w1[(int64_t)j * D + d]);
    const double u = (double)to_f32(w2[(int64_t)d * F + j]);
    acc += v * v + u * u;
  }
  out[j] = sqrt(acc);
}

template <typename T>
hipError_t launch_ffn_norms(const T* w1, const float* b1, const T* w2, int D, int F, double* out,
                            hipStream_t stream) {
  if (F <= 0) return hipSuccess;
  hipLaunchKernelGGL((ffn_norms_kernel<T>), dim3((F + R_THREADS - 1) / R_THREADS), dim3(R_THREADS), 0,
                     stream, w1, b1, w2, D, F, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// timestep embedding pieces
// ---------------------------------------------------------------------------
// HBM-bound (W is read once).  A wave takes R rows together, so a lane's slice
// of x, twice W's bytes, is read once for them.  R = 4 where that leaves four
// waves per SIMD ([30720, 5120] bf16: 57 us against 60 with one row), else 1 (of
// 5120 rows 4 would leave one wave per SIMD: 20 us against 11).
template <typename T, int GEMV_R>
__global__ __launch_bounds__(R_THREADS) void gemv_kernel(const T* __restrict__ W,
                                                         const float* __restrict__ x,
                                                         const float* __restrict__ bias,
                                                         float* __restrict__ out, int N, int K) {
  constexpr int VEC = Chunk<T>::VEC;
  const int n0 = (blockIdx.x * R_WAVES + (threadIdx.x >> 6)) * GEMV_R;
  const int lane = threadIdx.x & 63;
  if (n0 >= N) return;
  const T* wr[GEMV_R];
  float acc[GEMV_R];
#pragma unroll
  for (int r = 0; r < GEMV_R; ++r) {
    wr[r] = W + (int64_t)min(n0 + r, N - 1) * K;
    acc[r] = 0.f;
  }
#pragma unroll 4
  for (int k = lane * VEC; k < K; k += kWave * VEC) {
    u32x4 raw[GEMV_R];
#pragma unroll
    for (int r = 0; r < GEMV_R; ++r) raw[r] = *reinterpret_cast<const u32x4*>(wr[r] + k);
    float xv[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) xv[e] = x[k + e];
#pragma unroll
    for (int r = 0; r < GEMV_R; ++r) {
      float w[VEC];
      Chunk<T>::unpack(raw[r], w);
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[r] += w[e] * xv[e];
    }
  }
#pragma unroll
  for (int r = 0; r < GEMV_R; ++r) {
    acc[r] = wave_sum(acc[r]);
    if (lane == 0 && n0 + r < N) out[n0 + r] = acc[r] + (bias ? bias[n0 + r] : 0.f);
  }
}

template <typename T>
hipError_t launch_gemv(const T* W, const float* x, const float* bias, float* out, int N, int K,
                       hipStream_t stream) {
  if (N <= 0) return hipSuccess;
  auto launch = [&](auto r_tag) {
    constexpr int R = decltype(r_tag)::value, rows = R_WAVES * R;
    hipLaunchKernelGGL((gemv_kernel<T, R>), dim3((N + rows - 1) / rows), dim3(R_THREADS), 0, stream, W, x,
                       bias, out, N, K);
  };
  if (N >= 16384) launch(std::integral_constant<int, 4>{});
  else launch(std::integral_constant<int, 1>{});
  return hipGetLastError();
}

// [cos(t w_j), sin(t w_j)], w_j = 10000^(-j/half), in double precision:
// t w_j reaches ~1e3 rad, where a float argument already loses 1e-4.
__global__ void sinusoid_kernel(float t, int half, float* out) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= half) return;
  const double arg = (double)t * pow(10000.0, -(double)j / (double)half);
  out[j] = (float)cos(arg);
  out[half + j] = (float)sin(arg);
}

hipError_t launch_sinusoid(float t, int dim, float* out, hipStream_t stream) {
  const int half = dim / 2;
  hipLaunchKernelGGL(sinusoid_kernel, dim3((half + 255) / 256), dim3(256), 0, stream, t, half, out);
  return hipGetLastError();
}

__global__ void silu_kernel(const float* x, float* y, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = x[i] / (1.f + expf(-x[i]));
}

hipError_t launch_silu(const float* x, float* y, int n, hipStream_t stream) {
  hipLaunchKernelGGL(silu_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, x, y, n);
  return hipGetLastError();
}

__global__ void euler_kernel(float* z, const float* v, float dsig, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    z[i] = fmaf(dsig, v[i], z[i]);
}

hipError_t launch_euler(float* z, const float* v, float dsig, int64_t n, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 65536);
  hipLaunchKernelGGL(euler_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, z, v, dsig, n);
  return hipGetLastError();
}

// z = (1 - st) * (z - sf * v) + st * eps   (eps unused when st == 0)
__global__ void renoise_kernel(float* z, const float* v, float sf, float st, const float* eps,
                               int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float x = fmaf(-sf, v[i], z[i]);
    z[i] = eps ? fmaf(st, eps[i], (1.f - st) * x) : x;
  }
}

hipError_t launch_renoise(float* z, const float* v, float sigma_from, float sigma_to,
                          const float* eps, int64_t n, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 65536);
  hipLaunchKernelGGL(renoise_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, z, v, sigma_from,
                     sigma_to, eps, n);
  return hipGetLastError();
}

template <typename T>
__global__ void cast_kernel(const float* src, T* dst, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = from_f32<T>(src[i]);
}

template <typename T>
hipError_t launch_cast(const float* src, T* dst, int64_t n, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 65536);
  hipLaunchKernelGGL((cast_kernel<T>), dim3((unsigned)blocks), dim3(256), 0, stream, src, dst, n);
  return hipGetLastError();
}

#define INST(T)                                                                                \
  template hipError_t launch_norm<T>(const T*, T*, int, int, int, const float*, const float*,  \
                                     const float*, const float*, float, hipStream_t);          \
  template hipError_t launch_qk_norm<T>(T*, int64_t, int, int, int, int, int, const float*,    \
                                        const float*, float, float, const RopeDesc*,           \
                                        hipStream_t, const int32_t*, float);                   \
  template hipError_t launch_gather<T>(const T*, int64_t, T*, int64_t, int, int,               \
                                       const int32_t*, const int32_t*, hipStream_t);           \
  template hipError_t launch_gather_rows16<T>(const T*, int64_t, T*, int64_t, int64_t, int, int,\
                                              const int32_t*, hipStream_t);                    \
  template hipError_t launch_gemv<T>(const T*, const float*, const float*, float*, int, int,   \
                                     hipStream_t);                                             \
  template hipError_t launch_cast<T>(const float*, T*, int64_t, hipStream_t);                  \
  template hipError_t launch_ffn_norms<T>(const T*, const float*, const T*, int, int, double*,  \
                                          hipStream_t);
INST(float)
INST(bf16)
#undef INST

}  // namespace dif
