// What the two GEMM kernels (gemm.hip: large problems, gemm_ring.h: the
// others) share: launch parameters, operand-gather modes, vector accesses.
#pragma once
#include "common.h"
#include "kernels.h"

namespace dif {

// Fragment k of a k-step in the order its MFMAs first use them (MFMA i
// multiplies A row block i / TN by B column block i % TN): the value is a
// row block index (< TM) or TM + a column block index.  For 4 x 2 blocks:
// A0 B0 B1 A1 A2 A3.
// (a table built at compile time: indexing it with an unrolled loop's
// counter gives constants, so the fragment arrays stay in registers)
template <int TM, int TN>
struct FirstUse {
  int v[TM + TN];
};
template <int TM, int TN>
__host__ __device__ constexpr FirstUse<TM, TN> first_use_table() {
  FirstUse<TM, TN> t{};
  bool seen[TM + TN] = {};
  int n = 0;
  for (int i = 0; i < TM * TN; ++i) {
    const int a = i / TN, b = TM + i % TN;
    if (!seen[a]) {
      seen[a] = true;
      t.v[n++] = a;
    }
    if (!seen[b]) {
      seen[b] = true;
      t.v[n++] = b;
    }
  }
  return t;
}

constexpr int G_BKC = 8;    // 16-byte chunks per k-tile row (128 bytes)

enum { GA_NONE = 0, GA_ROWS = 1, GA_KCH = 2 };
constexpr uint32_t kMasked = 0x80000000u;  // buffer offset beyond any descriptor range

// Up to three B matrices ("segments", e.g. the q, k and v weights) share A
// and one launch; segment s writes output columns [s*N, (s+1)*N).
constexpr int kMaxSeg = 3;

template <typename T, typename OutT>
struct GemmParams {
  const T* A;
  const T* Bs[kMaxSeg];
  OutT* C;
  int64_t lda, ldb, ldc;
  int M, N, K;
  const float* biases[kMaxSeg];
  int nseg;
  const float* gate0;
  const float* gate1;
  const int32_t* rows;   // GA_ROWS
  const int32_t* kch;    // GA_KCH
  int b_rows;            // GA_ROWS: rows of the union B matrix
  int vec4;              // C rows allow aligned 4-element accesses
  // transposed output: columns from output column vt_col0 on go to
  // vt[(b * vt_dims + col - vt_col0) * ldvt + j] for row m = b * vt_L + j
  OutT* vt;
  int64_t ldvt;
  int vt_col0, vt_dims, vt_L;
  int vt_vec4;           // vt rows allow aligned 4-element stores and vt_L % 4 == 0
  int vt_pad;            // columns vt_L .. ldvt are zeroed
};

// four consecutive output elements: 8-byte (bf16) or 16-byte (f32) accesses
__device__ __forceinline__ void store4(bf16* p, const float* v) {
  bf16x4 x;
#pragma unroll
  for (int e = 0; e < 4; ++e) x[e] = (bf16)v[e];
  *reinterpret_cast<bf16x4*>(p) = x;
}
__device__ __forceinline__ void store4(float* p, const float* v) {
  f32x4 x;
#pragma unroll
  for (int e = 0; e < 4; ++e) x[e] = v[e];
  *reinterpret_cast<f32x4*>(p) = x;
}

// Four consecutive rows m .. m+3 (m a multiple of 4, m < M) of transposed
// column `dim`.  The lane that stores a sample's last token zeroes the padding.
template <typename T, typename OutT>
__device__ __forceinline__ void store_vt4(const GemmParams<T, OutT>& p, int m, int dim, const float* v) {
  auto pad = [&](OutT* row) {
    if (p.vt_pad)
      for (int64_t j = p.vt_L; j < p.ldvt; ++j) row[j] = from_f32<OutT>(0.f);
  };
  const int bb = m / p.vt_L, jt = m - bb * p.vt_L;
  if (p.vt_vec4 && m + 4 <= p.M) {   // same sample, aligned
    OutT* row = p.vt + ((int64_t)bb * p.vt_dims + dim) * p.ldvt;
    store4(row + jt, v);
    if (jt + 4 == p.vt_L) pad(row);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int me = m + e;
      if (me >= p.M) break;
      const int be = me / p.vt_L, je = me - be * p.vt_L;
      OutT* row = p.vt + ((int64_t)be * p.vt_dims + dim) * p.ldvt;
      row[je] = from_f32<OutT>(v[e]);
      if (je + 1 == p.vt_L) pad(row);
    }
  }
}

// Logical tile of this workgroup: XCD-contiguous ranges of tiles, then groups
// of GM row tiles that walk the N tiles of all segments together (operand
// reuse in L2).
__device__ __forceinline__ void tile_of(int block, int nbm, int nbv, int& mt, int& nt) {
  constexpr int GM = 8;
  const int bid = xcd_remap(block, nbm * nbv);
  const int group = bid / (GM * nbv);
  const int first_m = group * GM;
  const int gsize = min(nbm - first_m, GM);
  const int in_group = bid - group * GM * nbv;
  mt = first_m + in_group % gsize;
  nt = in_group / gsize;
}

}  // namespace dif
