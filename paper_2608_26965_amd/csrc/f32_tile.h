// The fp32 softmax over keys on the fp32 matrix instructions
// (v_mfma_f32_16x16x4_f32: fp32 products and sums), shared by the block-sparse
// attention and the compensation.
//
// One wavefront takes 16 queries against tiles of 16 keys. As in the bf16
// kernels the products are formed transposed: S^T = K Q^T (keys on the MFMA
// rows, queries on the columns) leaves lane l with query l % 16 and the logits
// of keys 4 (l / 16) + r, r = 0 .. 3, which is the P^T operand of
// O^T = V^T P^T as it stands. The order of a contraction's indices is free as
// long as both operands share it, so the operands are read 16 bytes a lane:
// step (j, e) of S^T contracts dims 16 j + 4 g + e over the lane groups
// g = l / 16, step r of O^T the keys 4 g + r.
//
// What bounds it: at the sizes fp32 is used for, the latency of one pass over
// a query's keys. So a workgroup takes 16 queries only, its wavefronts share
// the keys (step by step of kTps tiles, a softmax state each, merged through
// LDS at the end), and the operands go from L2 straight to registers: no
// barrier until the merge. One thread per query with K and V through LDS took
// 278 + 63 us (attention + compensation) for 2 heads of 1,000 queries x 12 of
// 47 clusters of 64 keys at d = 64 and 118 + 36 us for 1,024 tokens x 4 of 16
// clusters, one head; now 23 + 13 us and 13 + 13 us.
#pragma once

#include <type_traits>

#include "common.h"

namespace ca {

// 16 bytes at 4-byte alignment: dense fp32 inputs need no more than their own
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ f32x4 load4u(const float* p) {
  const f32x4u v = *reinterpret_cast<const f32x4u*>(p);
  return f32x4{v.x, v.y, v.z, v.w};
}

template <int DP>
struct F32Tile {
  static constexpr int NJ = DP / 16;              // 16-wide tiles of the head dimension
  static constexpr int TPS = DP == 128 ? 2 : 4;   // key tiles per step (registers)
  static constexpr int NW = DP == 128 ? 4 : 8;    // wavefronts of a workgroup, at most
  static constexpr int QP = 17;                   // queries per LDS row, padded
};

// Waves per SIMD of the kernels (their second launch bound): 256 registers.
constexpr int kF32Waves = 2;

// Calls f with two std::integral_constant<int>, the number of wavefronts of a
// workgroup and the number of parts that its tiles are cut into, for ntile tiles of 16 keys and a launch of wgs workgroups: where
// there is more than one workgroup a CU (256 of them), as many as get tiles,
// since others only keep registers from the next workgroup; else all, which
// then share the prologue and the output rows. 8 heads of 16,384 queries at
// d = 64: attention on one tile 228 us with 8 wavefronts, 62 with one;
// compensation with 8 tiles 424 and 157 (two). One head of 1,024 queries (64
// workgroups), compensation with one tile: 20 us with 8 wavefronts, 23 with
// one. Large launches with more tiles than four wavefronts' first steps take
// four wavefronts, two parts each: two workgroups fit a CU, and one's loads and
// merge run beside the other's products (40 heads of 6,553 tokens at d = 64:
// attention on 79 tiles 1.84 -> 1.60 ms, compensation with 26 tiles 1.04 -> 0.83; one
// head of 4,160 queries, 260 workgroups, both calls 70 -> 62 us). Which part has
// which tiles does not depend on the number of wavefronts, so neither do the
// results.
template <int DP, typename F>
void f32_wavefronts(int ntile, int64_t wgs, F&& f) {
  constexpr int TPS = F32Tile<DP>::TPS, NW = F32Tile<DP>::NW;
  if (wgs > 256 && ntile <= TPS)
    f(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{});
  else if (wgs > 256 && ntile <= 2 * TPS)
    f(std::integral_constant<int, 2>{}, std::integral_constant<int, 2>{});
  else if (NW == 4 || (wgs > 256 && ntile <= 4 * TPS))
    f(std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{});
  else if (wgs > 256)
    f(std::integral_constant<int, 4>{}, std::integral_constant<int, NW>{});
  else
    f(std::integral_constant<int, NW>{}, std::integral_constant<int, NW>{});
}

template <int DP>
struct F32State {
  f32x4 o[F32Tile<DP>::NJ];  // O^T: dims 16 t + 4 g + r of query l % 16
  float m, l;                // reference of the query; this lane's part of the sum
};

// The Q^T operand of 16 rows (this lane's row; zeros past d)
template <int DP>
__device__ __forceinline__ void f32_load_rows(const float* row, int d, int g,
                                              f32x4 (&f)[F32Tile<DP>::NJ]) {
#pragma unroll
  for (int j = 0; j < F32Tile<DP>::NJ; ++j) {
    const int t = 16 * j + 4 * g;
    f[j] = t < d ? load4u(row + t) : f32x4{0.f, 0.f, 0.f, 0.f};
  }
}

// Online softmax of one wavefront over tiles w * TPS + u + i * NP * TPS of
// src (part w of NP), for which
//   src.rows(T, kf)   the K operand of tile T (lane: key l % 16)
//   src.vals(T, vf)   the V^T operand (lane: dim l % 16, keys 4 g .. 4 g + 3)
//   src.logits(T, s)  scales the products and masks keys (-inf)
//   src.mask_vals(T, vf)  clears values of masked keys that may not be finite
//                     (late, so that the products above do not wait for them)
// take any T; tiles at or past src.ntile are all masked.
template <int DP, int NP, typename Src>
__device__ __forceinline__ void f32_online(const Src& src, const f32x4 (&qf)[F32Tile<DP>::NJ],
                                           int w, F32State<DP>& st) {
  constexpr int NJ = F32Tile<DP>::NJ, TPS = F32Tile<DP>::TPS;
  st.m = -INFINITY;
  st.l = 0.f;
#pragma unroll
  for (int j = 0; j < NJ; ++j) st.o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int t0 = w * TPS; t0 < src.ntile; t0 += NP * TPS) {
    f32x4 kf[TPS][NJ], vf[TPS][NJ], s[TPS];
#pragma unroll
    for (int u = 0; u < TPS; ++u) src.rows(t0 + u, kf[u]);
#pragma unroll
    for (int u = 0; u < TPS; ++u) src.vals(t0 + u, vf[u]);
    // four partial sums a logit: the chains of rounded sums are a
    // quarter as long, and their error smaller (outputs 1.1e-6 from
    // 64 bits with one chain, 5.4e-7 with four, 6.1e-7 with the former kernel)
    f32x4 p[TPS][4];
#pragma unroll
    for (int u = 0; u < TPS; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) p[u][e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int u = 0; u < TPS; ++u)
          p[u][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[u][j][e], qf[j][e], p[u][e], 0, 0, 0);
#pragma unroll
    for (int u = 0; u < TPS; ++u) s[u] = (p[u][0] + p[u][1]) + (p[u][2] + p[u][3]);
    float mx = st.m;
#pragma unroll
    for (int u = 0; u < TPS; ++u) {
      src.logits(t0 + u, s[u]);
#pragma unroll
      for (int r = 0; r < 4; ++r) mx = fmaxf(mx, s[u][r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mu = mx == -INFINITY ? 0.f : mx;  // nothing but masked keys so far
    if (__builtin_amdgcn_ballot_w64(mx > st.m)) {
      const float al = expf(st.m - mu);
      st.l *= al;
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) st.o[j][r] *= al;
      st.m = mx;
    }
#pragma unroll
    for (int u = 0; u < TPS; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[u][r] = expf(s[u][r] - mu);
        st.l += s[u][r];
      }
#pragma unroll
    for (int u = 0; u < TPS; ++u) src.mask_vals(t0 + u, vf[u]);
#pragma unroll
    for (int u = 0; u < TPS; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          st.o[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[u][j][r], s[u][r], st.o[j], 0, 0, 0);
  }
  st.l += __shfl_xor(st.l, 16, 64);
  st.l += __shfl_xor(st.l, 32, 64);
}

// LDS of the merge of the parts' states
template <int DP, int NP>
struct F32Merge {
  float o[NP][DP][F32Tile<DP>::QP];
  float f[NP][16];               // weight of part w for a query
  float m[NP][16], l[NP][16];
  float mx[16], sum[16];         // reference and sum of a query over all parts
};

// Part w's state, for the merge
template <int DP, int NP>
__device__ __forceinline__ void f32_store(F32Merge<DP, NP>& M, const F32State<DP>& st, int w, int lane) {
  constexpr int NJ = F32Tile<DP>::NJ;
  const int q = lane & 15, g = lane >> 4;
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) M.o[w][16 * j + 4 * g + r][q] = st.o[j][r];
  if (g == 0) {
    M.m[w][q] = st.m;
    M.l[w][q] = st.l;
  }
}

// The online softmax of all parts by NW wavefronts, stored for the merge
template <int DP, int NW, int NP, typename Src>
__device__ __forceinline__ void f32_parts(const Src& src, const f32x4 (&qf)[F32Tile<DP>::NJ],
                                          F32Merge<DP, NP>& M, int w, int lane) {
#pragma unroll 1
  for (int p = w; p < NP; p += NW) {
    F32State<DP> st;
    f32_online<DP, NP>(src, qf, p, st);
    f32_store<DP, NP>(M, st, p, lane);
  }
}

// Merges the parts' states: afterwards query q's sum of exponentials is
// sum[q] against the reference mx[q] (sum 0: no key), and its output before
// the division is sum_w f[w][q] o[w][t][q] (f32_merged).
template <int DP, int NP>
__device__ __forceinline__ void f32_merge(F32Merge<DP, NP>& M, int w, int lane) {
  const int q = lane & 15, g = lane >> 4;
  __syncthreads();
  if (w == 0 && g == 0) {
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < NP; ++i) mx = fmaxf(mx, M.m[i][q]);
    const float mu = mx == -INFINITY ? 0.f : mx;
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const float f = expf(M.m[i][q] - mu);
      M.f[i][q] = f;
      sum += f * M.l[i][q];
    }
    M.mx[q] = mu;
    M.sum[q] = sum;
  }
  __syncthreads();
}

template <int DP, int NP>
__device__ __forceinline__ float f32_merged(const F32Merge<DP, NP>& M, int q, int t) {
  float x = 0.f;
#pragma unroll
  for (int i = 0; i < NP; ++i) x += M.f[i][q] * M.o[i][t][q];
  return x;
}

}  // namespace ca
