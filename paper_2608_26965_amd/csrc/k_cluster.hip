// Clustering (paper: Method, Clustering): split spaces (Transforms), the
// diagonalized recursive split, and the permuted copies plus centroids.
//
// Pipeline per head, both sides batched in every launch:
//   moments      X^T X and column sums (fp32 partials, fp64 reduction)
//   eigh         Householder tridiagonal reduction, Sturm bisection and
//                inverse iteration on d x d matrices, one workgroup each
//   transforms   metric roots, the key-side covariance in the query metric,
//                the normalised query representation and its covariance
//   project      Y = X T (queries additionally scaled by 1/|q S_k|)
//   split        levels with nodes larger than the tail size: multi-block
//                exact select (256 linear bins, then within one) + stable
//                partition;
//                remaining levels: one workgroup per node, in LDS
//   gather       permuted Q/K/V, centroids of the original vectors, counts
//
// The split is exact integer work on order-preserving images of the fp32
// coordinates; the only floating-point decision, the highest-variance
// coordinate of a node's subsample, is taken in fp64 with a fixed operation
// order and no contraction, so it is reproducible bit for bit.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "attn_tile.h"
#include "common.h"

namespace ca {

namespace {

// ---------------------------------------------------------------------------
// Parameters of the two sides (0 = queries, 1 = keys)
// ---------------------------------------------------------------------------

struct Side {
  const void* x;    // input tensor (strides lx)
  Lay lx;
  float* y;         // split coordinates [BH][n][d]
  float* ycol;      // the first kColCopy of them, [BH][kColCopy][n] (or NULL)
  int32_t* perm;    // [BH][n]
  int32_t* cid;     // [BH][n] (may be null)
  int32_t* count;   // [BH][nc]
  float* cent;      // [BH][nc][d]
  void* xp;         // permuted copy [BH][npad][d]
  int n, c, nc, npad, levels, big, tail;
};

struct Ctx {
  Side s[2];
  const void* v;    // values (may be null)
  float* cent_v;
  void* vp;         // value tiles [BH][nkc][d][ck]
  Lay lv;           // strides of the values
  int BH, H, d, dtype, xf, nmax, nblk, mom_rows, proj_rows;
  float* mats;      // [BH][kMats][d][d]
  float* vecs;      // [BH][kVecs][d]
  float* inv_q;     // [BH][nq]
  float* mom_part;  // [2][BH][nblk][d*d + d]
  float* qn_part;   // [BH][nblk][d*d + d]
  bf16* wops;       // [BH][3][2][d][d] transposed hi/lo bf16 operands
  int32_t* idx0;
  int32_t* idx1;
  uint32_t* keys;
  int32_t* node_state;
  uint32_t* hist;
  uint32_t* ghist;
  uint32_t* cand;
  int32_t* chunk_cnt;
  int max_nodes, hist_slots, ghist_slots;
  int split;        // ca_split
  float* dirs;      // [2 levels][2][BH][max_nodes][d] split directions (basic splitting)
};

// Matrix slots
enum { M_A0 = 0, M_CK = 1, M_E0 = 2, M_EK = 3, M_C3 = 4, M_TK = 5, M_TQ = 6 };
// Operand slots (MFMA A operands W^T, split in bf16 hi + lo)
enum { O_FK = 0, O_TK = 1, O_TQ = 2 };
// Vector slots
enum { V_MUQ = 0, V_MUK = 1, V_MUR = 2 };

__device__ __forceinline__ float* mat(const Ctx& C, int bh, int slot) {
  return C.mats + ((size_t)bh * kMats + slot) * C.d * C.d;
}
__device__ __forceinline__ bf16* wop(const Ctx& C, int bh, int slot) {
  return C.wops + ((size_t)bh * 3 + slot) * 2 * C.d * C.d;
}
__device__ __forceinline__ float* vec(const Ctx& C, int bh, int slot) {
  return C.vecs + ((size_t)bh * kVecs + slot) * C.d;
}

__device__ __forceinline__ float load_x(const void* x, int bh, int i, const Lay& L, int t,
                                        int dtype) {
  return load_elem(x, row_off(bh, i, L) + t, dtype);
}

// ---------------------------------------------------------------------------
// Second moments: part[pid][blk] = (sum_rows x x^T, sum_rows x) over a row block
// ---------------------------------------------------------------------------

constexpr int kStage = 32;  // rows staged in LDS at a time
constexpr int kDP = kMaxD + 4;

// Accumulates sum_r a_r b_r^T for the rows staged in A/B into per-thread 4x4
// blocks (up to 4 blocks per thread: d <= 128).
__device__ __forceinline__ void acc_outer(float (*A)[kDP], float (*B)[kDP], int rows, int d4,
                                          float acc[4][16]) {
  const int nb = d4 * d4;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int blk = threadIdx.x + 256 * q;
    if (blk >= nb) break;
    const int bi = blk / d4, bj = blk % d4;
#pragma unroll 8
    for (int r = 0; r < rows; ++r) {
      const float4 a = *(const float4*)&A[r][4 * bi];
      const float4 b = *(const float4*)&B[r][4 * bj];
      const float av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[q][4 * i + j] = __builtin_fmaf(av[i], bv[j], acc[q][4 * i + j]);
    }
  }
}

__device__ __forceinline__ void write_outer(float* out, int d, int d4, float acc[4][16]) {
  const int nb = d4 * d4;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int blk = threadIdx.x + 256 * q;
    if (blk >= nb) break;
    const int bi = blk / d4, bj = blk % d4;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int r = 4 * bi + i, c = 4 * bj + j;
        if (r < d && c < d) out[r * d + c] = acc[q][4 * i + j];
      }
  }
}

__global__ __launch_bounds__(256) void moments_partial_kernel(Ctx C) {
  __shared__ __attribute__((aligned(16))) float X[kStage][kDP];
  const int pid = blockIdx.y, side = pid / C.BH, bh = pid % C.BH, blk = blockIdx.x;
  const Side& S = C.s[side];
  const int d = C.d, d4 = (d + 3) / 4;
  const int r0 = blk * C.mom_rows, r1 = min(S.n, r0 + C.mom_rows);
  float acc[4][16];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[q][e] = 0.f;
  float csum = 0.f;
  for (int rs = r0; rs < r1; rs += kStage) {
    const int rows = min(kStage, r1 - rs);
    __syncthreads();
    for (int e = threadIdx.x; e < kStage * 4 * d4; e += 256) {
      const int r = e / (4 * d4), t = e % (4 * d4);
      X[r][t] = (r < rows && t < d)
                    ? load_x(S.x, bh, rs + r, S.lx, t, C.dtype)
                    : 0.f;
    }
    __syncthreads();
    acc_outer(X, X, rows, d4, acc);
    if (threadIdx.x < d)
#pragma unroll 8
      for (int r = 0; r < rows; ++r) csum += X[r][threadIdx.x];
  }
  float* out = C.mom_part + ((size_t)pid * C.nblk + blk) * (d * d + d);
  write_outer(out, d, d4, acc);
  if (threadIdx.x < d) out[d * d + threadIdx.x] = csum;
}

// The finishing kernels sum nb partials p[0], p[stride], ... in fp64 as eight
// interleaved sums added pairwise (a fixed order, so deterministic), by one
// thread an element (U = 1, its loads eight at a time) or by eight (U = 8, one
// sum each, exchanged through LDS). One thread an element is all load latency
// where the elements are few: the moments of 8 heads (64 partials) took 9.5 us
// against 7.1, of one fp32 head 8.9 against 5.0; eight are too little work a
// workgroup where the elements are many: 67 us against 30 on 40 heads at
// d = 128. The line between (2^18 elements over all heads and both sides) is
// their middle.
template <int U>
__device__ __forceinline__ double sum_partials(const float* p, size_t stride, int nb,
                                               double (*sh)[256 / U], bool in) {
  if constexpr (U == 1) {
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (!in) return 0.0;
    int b = 0;
    for (; b + 8 <= nb; b += 8) {
#pragma unroll
      for (int u = 0; u < 8; ++u) acc[u] += (double)p[(size_t)(b + u) * stride];
    }
    for (; b < nb; ++b) acc[b & 7] += (double)p[(size_t)b * stride];
    return ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
  } else {
    static_assert(U == 8, "eight interleaved sums");
    const int u = threadIdx.x / (256 / U), e = threadIdx.x % (256 / U);
    double acc = 0.0;
    if (in) {
#pragma unroll 8
      for (int b = u; b < nb; b += 8) acc += (double)p[(size_t)b * stride];
    }
    sh[u][e] = acc;
    __syncthreads();
    return ((sh[0][e] + sh[1][e]) + (sh[2][e] + sh[3][e])) +
           ((sh[4][e] + sh[5][e]) + (sh[6][e] + sh[7][e]));
  }
}

// Reduces the moment partials and writes the matrices the eigensolver starts
// from:
//   queries: metric -> Q^T Q / n;  pca -> centred covariance of Q
//   keys:    centred covariance of K (both modes)
// plus the means. Grid: (element blocks of 256 / U, BH, side).
template <int U>
__global__ __launch_bounds__(256) void moments_finish_kernel(Ctx C) {
  __shared__ double sh[3][U][256 / U];
  const int side = blockIdx.z, bh = blockIdx.y, d = C.d, dd = d * d;
  const int e = blockIdx.x * (256 / U) + threadIdx.x % (256 / U);
  const int pid = side * C.BH + bh;
  const size_t stride = (size_t)dd + d;
  const float* part = C.mom_part + (size_t)pid * C.nblk * stride;
  const bool centred = side == 1 || C.xf == CA_XF_PCA;
  const bool in = e < dd + d, cov = e < dd && centred;
  const int i = e / d, j = e % d;
  const double n = (double)C.s[side].n;
  double v = sum_partials<U>(part + e, stride, C.nblk, sh[0], in) / n;
  const double mi = sum_partials<U>(part + dd + i, stride, C.nblk, sh[1], cov) / n;
  const double mj = sum_partials<U>(part + dd + j, stride, C.nblk, sh[2], cov) / n;
  if (!in || threadIdx.x >= 256 / U) return;
  if (e >= dd) {
    vec(C, bh, side == 0 ? V_MUQ : V_MUK)[e - dd] = (float)v;
    return;
  }
  if (centred) v -= mi * mj;
  mat(C, bh, side == 0 ? M_A0 : M_CK)[e] = (float)v;
}

// ---------------------------------------------------------------------------
// Symmetric eigenproblems of the transforms (the algorithm is described at
// eigh_kernel). Output: eigenvalues in descending order and the matching
// eigenvectors as columns.
// ---------------------------------------------------------------------------

// One eigenproblem: A = B, A = B - m m^T, or A = S^T B S (- u u^T with
// u = S^T m); the eigenvectors are oriented so that o . U[:, j] >= 0 with
// o = u (when u is formed) or a given vector, and the split projection
// T = F U (or U) is written in fp32 and, for bf16 inputs, as the transposed
// hi/lo bf16 MFMA operand.
struct EighJob {
  int b, s, m;     // matrix B, factor S (-1: none), vector m (-1: none)
  int rank1;       // subtract u u^T
  int orient;      // orientation vector slot, used when u is not formed
  int t_f;         // factor F of the projection T = F U (-1: T = U)
  int t_out, wop_out;
};
struct EighJobs {
  EighJob j[2];
};

// Symmetric eigensolver, one workgroup of kEighM * DM threads per d x d
// problem (d <= DM):
//  1. Householder reduction to a tridiagonal matrix T = Q^T A Q (A fp32 in
//     LDS; column norms and reflector scales in fp64). Every wavefront builds
//     reflector k from column k itself, so the pass over the trailing block,
//     which applies reflector k-1 (the symmetric rank-two update) and forms
//     p = A v_k in the same sweep, needs one barrier a step.
//  2. Off-diagonal entries below 2^-24 of the norm are set to zero, so T
//     splits into unreduced blocks (distinct eigenvalues, eigenvectors with
//     disjoint supports). Eigenvalues by bisection on Sturm counts in fp64:
//     sign changes of the leading minors (division free, rescaled every
//     eight steps), kEighM points per eigenvalue and round.
//  3. Eigenvectors of T by two steps of inverse iteration (an LDL^T
//     factorisation of T - lambda I in fp64) from pseudo-random starts;
//     eigenvalues closer than 1e-8 of the norm form clusters whose vectors
//     are re-orthogonalised (modified Gram-Schmidt) after each step.
//  4. Back-transformation by the reflectors: V = Q Z.
// (Golub and Van Loan, Matrix Computations: the Householder tridiagonal
// reduction, Sturm sequence bisection and inverse iteration.)
constexpr int kEighM = 4;
template <int DM>
constexpr int eigh_threads() {
  return kEighM * DM;
}
// Row stride of the LDS matrices (float4-aligned rows)
__host__ __device__ constexpr int eigh_stride(int dm) { return dm + 4; }
__host__ __device__ constexpr size_t eigh_lds_bytes(int dm) {
  return 2 * (size_t)dm * eigh_stride(dm) * sizeof(float);
}
// Bisection rounds: (kEighM + 1)^-17 of the width 2 is 1.5e-12 of the norm,
// far inside the cluster tolerance, so two inverse-iteration steps converge.
constexpr int kBisectRounds = 17;
constexpr double kDeflate = 0x1p-24;  // relative size of a negligible off-diagonal
constexpr double kClusterTol = 1e-8;  // relative gap below which vectors are re-orthogonalised
constexpr double kPivMin = 0x1p-50;   // smallest pivot magnitude of the LDL^T factorisation
constexpr double kStore = 0x1p-64;    // scale of the intermediate vectors kept in fp32

__device__ __forceinline__ void wave_lds_order() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Cross-lane sums through DPP (no LDS round trip). dpp_add: x + x of lane
// (CTRL); lanes outside the row mask add 0.
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROWS, 0xF, false));
}
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ double dpp_add(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xF, false);
  return x + __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// Sum over the 4 lanes of a quad (every lane of the quad gets it)
template <typename F>
__device__ __forceinline__ F quad_sum(F x) {
  x = dpp_add<0xB1>(x);  // quad_perm [1, 0, 3, 2]
  return dpp_add<0x4E>(x);  // quad_perm [2, 3, 0, 1]
}
// Sum over the wavefront, returned to every lane (a uniform value)
__device__ __forceinline__ float wave_sum(float x) {
  x = quad_sum(x);
  x = dpp_add<0x141>(x);        // row_half_mirror: 8 lanes
  x = dpp_add<0x140>(x);        // row_mirror: 16 lanes
  x = dpp_add<0x142, 0xA>(x);   // row_bcast15 into rows 1, 3
  x = dpp_add<0x143, 0xC>(x);   // row_bcast31 into rows 2, 3: lane 63 holds the sum
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}
__device__ __forceinline__ double wave_sum(double x) {
  x = quad_sum(x);
  x = dpp_add<0x141>(x);
  x = dpp_add<0x140>(x);
  x = dpp_add<0x142, 0xA>(x);
  x = dpp_add<0x143, 0xC>(x);
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)b, 63), hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// Largest value of the wavefront (NaN only if all are), returned to every lane
template <int CTRL>
__device__ __forceinline__ float dpp_max(float x) {
  return fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(
                      __float_as_int(x), __float_as_int(x), CTRL, 0xF, 0xF, false)));
}
__device__ __forceinline__ float wave_max(float x) {
  x = dpp_max<0xB1>(x);   // quad_perm [1, 0, 3, 2]
  x = dpp_max<0x4E>(x);   // quad_perm [2, 3, 0, 1]
  x = dpp_max<0x141>(x);  // row_half_mirror
  x = dpp_max<0x140>(x);  // row_mirror
  x = fmaxf(fmaxf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 0)),
                  __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 16))),
            fmaxf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 32)),
                  __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 48))));
  return x;
}
// Inclusive sum over the lanes up to this one
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ int dpp_shift_add(int x) {
  return x + __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ int wave_scan(int x) {
  x = dpp_shift_add<0x111>(x);       // row_shr:1
  x = dpp_shift_add<0x112>(x);       // row_shr:2
  x = dpp_shift_add<0x114>(x);       // row_shr:4
  x = dpp_shift_add<0x118>(x);       // row_shr:8
  x = dpp_shift_add<0x142, 0xA>(x);  // row_bcast15 into rows 1, 3
  x = dpp_shift_add<0x143, 0xC>(x);  // row_bcast31 into rows 2, 3
  return x;
}
__device__ __forceinline__ float read_lane(float x, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}
// 1 / x in fp64: the hardware reciprocal and two Newton steps
__device__ __forceinline__ double recip64(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}

// Number of eigenvalues below x of the block [s, t) of the scaled
// tridiagonal matrix, tq[i] = (diagonal i, squared off-diagonal i - 1): the
// sign changes of the sequence 1, p_s, ..., p_{t-1} of leading minors of
// T - x I (a zero minor counts as positive).
__device__ __forceinline__ int sturm_below(const double2* tq, int s, int t, double x) {
  // The minors' sign bits are shifted into a word and the changes counted
  // eight at a time: four instructions a step, and with one wavefront a SIMD
  // the instructions are what a step costs (comparing and adding per step took
  // 75,000 cycles for the 17 rounds at d = 64, now 55,000). A minor that is
  // exactly zero is +0, so it counts as positive: the next one then has the
  // opposite sign of the one before, and the pair adds exactly one change.
  // The next eight entries are read while the current eight are used; the
  // last, partial eight run on past the block (tq holds nine more finite
  // entries) with their changes not counted.
  auto sign_in = [](uint32_t bits, double p) {
    return __builtin_amdgcn_alignbit(bits, (uint32_t)((uint64_t)__double_as_longlong(p) >> 32), 31);
  };
  double p2 = 1.0, p1 = tq[s].x - x;
  uint32_t bits = sign_in(0u, p1);  // (the sequence starts with 1: positive)
  int cnt = (int)bits;
  double2 q[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) q[u] = tq[s + 1 + u];
  int i0 = s + 1;
  for (; i0 + 8 <= t; i0 += 8) {
    double2 nq[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) nq[u] = tq[i0 + 8 + u];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const double p = (q[u].x - x) * p1 - q[u].y * p2;
      bits = sign_in(bits, p);
      p2 = p1;
      p1 = p;
    }
    cnt += (int)__popc((bits ^ (bits >> 1)) & 0xFFu);
    int ex;
    (void)frexp(fmax(fabs(p1), fabs(p2)), &ex);
    p1 = ldexp(p1, -ex);
    p2 = ldexp(p2, -ex);
#pragma unroll
    for (int u = 0; u < 8; ++u) q[u] = nq[u];
  }
#pragma unroll
  for (int u = 0; u < 7; ++u) {
    const double p = (q[u].x - x) * p1 - q[u].y * p2;
    bits = sign_in(bits, p);
    p2 = p1;
    p1 = p;
  }
  const int over = 7 - max(t - i0, 0);  // steps past the block
  cnt += (int)__popc(((bits ^ (bits >> 1)) & 0x7Fu) >> over);
  return cnt;
}

// Separately rounded fp32 operations: a product is never fused into the sum
// that follows it, and the quotient and square root are the correctly rounded
// ones (the default contraction would otherwise turn a + x * y into an FMA,
// and the HIP __f*_rn intrinsics are plain operators here).
__device__ __forceinline__ float add_rn(float a, float b) {
#pragma clang fp contract(off)
  return a + b;
}
__device__ __forceinline__ float sub_rn(float a, float b) {
#pragma clang fp contract(off)
  return a - b;
}
__device__ __forceinline__ float mul_rn(float a, float b) {
#pragma clang fp contract(off)
  return a * b;
}

// Pseudo-random start of inverse iteration: +-[0.5, 1.5)
__device__ __forceinline__ float start_value(int g, int i) {
  uint32_t h = (uint32_t)(g * 0x9E3779B1u) ^ (uint32_t)(i * 0x85EBCA77u + 0x165667B1u);
  h ^= h >> 15;
  h *= 0x2C1B3C6Du;
  h ^= h >> 12;
  h *= 0x297A2D39u;
  h ^= h >> 15;
  const float u = 0.5f + (float)(h & 0xFFFFu) * (1.f / 65536.f);
  return (h & 0x10000u) ? -u : u;
}

// 4x4 register blocks of a d x d product (d <= 128, NT threads: at most two
// blocks per thread): acc = op(X) op(Y), op(Z) = Z or Z^T, with X, Y in LDS
// at row stride ld (a multiple of 4, 16-byte aligned rows) and zeros up to a
// multiple of 4; the sum runs over 4 indices per float4 load.
struct MMAcc {
  float v[2][16];
};

template <int NT>
__device__ __forceinline__ void lds_mm(const float* X, bool tX, const float* Y, bool tY, int ld,
                                       int d, MMAcc& acc) {
  const int d4 = (d + 3) >> 2, nb = d4 * d4;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
#pragma unroll
    for (int e = 0; e < 16; ++e) acc.v[u][e] = 0.f;
    const int blk = threadIdx.x + NT * u;
    if (blk >= nb) continue;
    const int i0 = 4 * (blk / d4), j0 = 4 * (blk % d4);
    for (int t = 0; t < d; t += 4) {
      float x[4][4], y[4][4];  // x[a][s] = op(X)[i0 + a][t + s], y[s][b] = op(Y)[t + s][j0 + b]
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float4 xv = *reinterpret_cast<const float4*>(tX ? &X[(t + k) * ld + i0] : &X[(i0 + k) * ld + t]);
        const float4 yv = *reinterpret_cast<const float4*>(tY ? &Y[(j0 + k) * ld + t] : &Y[(t + k) * ld + j0]);
        const float xs[4] = {xv.x, xv.y, xv.z, xv.w}, ys[4] = {yv.x, yv.y, yv.z, yv.w};
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          if (tX) x[m][k] = xs[m]; else x[k][m] = xs[m];
          if (tY) y[m][k] = ys[m]; else y[k][m] = ys[m];
        }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int b = 0; b < 4; ++b)
            acc.v[u][4 * a + b] = __builtin_fmaf(x[a][s], y[s][b], acc.v[u][4 * a + b]);
    }
  }
}

// Writes acc to an LDS matrix (stride ld); entries outside d x d stay zero.
template <int NT>
__device__ __forceinline__ void lds_mm_store(const MMAcc& acc, float* Z, int ld, int d) {
  const int d4 = (d + 3) >> 2, nb = d4 * d4;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int blk = threadIdx.x + NT * u;
    if (blk >= nb) continue;
    const int i0 = 4 * (blk / d4), j0 = 4 * (blk % d4);
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b)
        Z[(i0 + a) * ld + j0 + b] = i0 + a < d && j0 + b < d ? acc.v[u][4 * a + b] : 0.f;
  }
}

// Rows wv, wv + NW, ... (RI of them) of a d x d matrix, CPL columns a lane,
// zero outside it.
template <int RI, int CPL, int NW>
__device__ __forceinline__ void load_square(const float* __restrict__ g, int d, int wv, int lane,
                                            float (&r)[RI * CPL]) {
#pragma unroll
  for (int ii = 0; ii < RI; ++ii)
#pragma unroll
    for (int cc = 0; cc < CPL; ++cc) {
      const int i = wv + NW * ii, j = lane + 64 * cc;
      const bool in = i < d && j < d;
      const float x = g[in ? i * d + j : 0];
      r[ii * CPL + cc] = in ? x : 0.f;
    }
}

template <int DM>
__global__ __launch_bounds__(eigh_threads<DM>()) void eigh_kernel(Ctx C, EighJobs J) {
  constexpr int NT = eigh_threads<DM>();
  static_assert((DM / 4) * (DM / 4) <= 2 * NT, "two 4x4 product blocks per thread");
  constexpr int EP = eigh_stride(DM);
  constexpr int NW = NT / 64;
  constexpr int CPL = DM / 64;           // rows (or columns) per lane in a wavefront sweep
  constexpr int NQ = DM / (4 * kEighM);  // float4 column groups per thread in a row pass
  constexpr int RW = DM / kEighM;        // rows per thread in the back-transformation
  constexpr int RI = DM / NW;            // matrix rows per wavefront in a load or store
  static_assert(CPL >= 1 && NQ >= 1 && RW % 4 == 0, "matrix size");
  extern __shared__ __attribute__((aligned(16))) float esh[];
  float* A = esh;             // [DM][EP]; row k keeps reflector k once reduced
  float* Vt = esh + DM * EP;  // [DM][EP]: S during the prologue, then Z[g][r] (vector g)
  __shared__ __attribute__((aligned(16))) float vvs[2][NW][DM];  // reflectors, one copy per wave
  __shared__ __attribute__((aligned(16))) float pbuf[2][DM];     // p = A v of the last two steps
  __shared__ float kpart[2][NW];
  __shared__ __attribute__((aligned(16))) float4 colb[2][DM];  // the next step's column (in its group of 4)
  __shared__ float last2[2][2];
  __shared__ float trid[2][DM];  // diagonal, off-diagonal of T
  __shared__ double2 tq[DM + 9]; // scaled (diagonal i, squared off-diagonal i - 1), zeros past d
  __shared__ double es[DM], lam64[DM];
  __shared__ int bs[DM], be[DM], inv[DM];
  __shared__ double sh_tn;
  __shared__ uint64_t sh_link[CPL];
  __shared__ __attribute__((aligned(16))) float ovec[DM];
  __shared__ float uvec[DM], mvec[DM], lam[DM], sgn[DM];
  const int bh = blockIdx.x, d = C.d, tid = threadIdx.x;
  const EighJob& jb = J.j[blockIdx.y];
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // ---- prologue: the matrix to diagonalize
  {
    const float* Bg = mat(C, bh, jb.b);
    const float* Sg = jb.s >= 0 ? mat(C, bh, jb.s) : nullptr;
    // every load is issued before the first is used
    float lb[RI * CPL], ls[RI * CPL];
    load_square<RI, CPL, NW>(Bg, d, wv, lane, lb);
    if (Sg) load_square<RI, CPL, NW>(Sg, d, wv, lane, ls);
    if (tid < DM) {
      ovec[tid] = 0.f;
      mvec[tid] = jb.m >= 0 && tid < d ? vec(C, bh, jb.m)[tid] : 0.f;
    }
    if (tid < 9) tq[DM + tid] = make_double2(0.0, 0.0);
#pragma unroll
    for (int ii = 0; ii < RI; ++ii)
#pragma unroll
      for (int cc = 0; cc < CPL; ++cc) {
        const int at = (wv + NW * ii) * EP + lane + 64 * cc;
        A[at] = lb[ii * CPL + cc];
        Vt[at] = Sg ? ls[ii * CPL + cc] : 0.f;  // S while it is needed
      }
    __syncthreads();
    if (jb.m >= 0) {
      // u = S^T m (or m)
      if (tid < d) {
        float u;
        if (Sg) {
          float u4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
          for (int t = 0; t < d; t += 4)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              u4[e] = __builtin_fmaf(Vt[(t + e) * EP + tid], mvec[t + e], u4[e]);
          u = (u4[0] + u4[1]) + (u4[2] + u4[3]);
        } else {
          u = mvec[tid];
        }
        uvec[tid] = u;
        ovec[tid] = u;
      }
    } else if (tid < d) {
      ovec[tid] = vec(C, bh, jb.orient)[tid];
    }
    if (Sg) {
      // A = S^T (B S)
      MMAcc acc;
      lds_mm<NT>(A, false, Vt, false, EP, d, acc);  // T1 = B S
      __syncthreads();
      lds_mm_store<NT>(acc, A, EP, d);
      __syncthreads();
      lds_mm<NT>(Vt, true, A, false, EP, d, acc);   // S^T T1
      __syncthreads();
      lds_mm_store<NT>(acc, A, EP, d);
    }
    __syncthreads();
    if (jb.rank1)
      for (int i = wv; i < d; i += NW)
#pragma unroll
        for (int cc = 0; cc < CPL; ++cc) {
          const int j = lane + 64 * cc;
          if (j < d) A[i * EP + j] -= uvec[i] * uvec[j];
        }
    __syncthreads();
  }
  // ---- 1. Householder reduction. Step k: reflector H_k = I - v v^T (|v|^2 = 2,
  // support k+1..d-1) from column k after the update by H_{k-1}; the row pass
  // applies H_{k-1} to the block [k+1, d)^2 and accumulates p = A v; with
  // w = p - (v^T p / 2) v, H A H = A - v w^T - w v^T.
  //
  // The matrix is held in registers: the 16 lanes of a DPP row share 4 rows
  // (rs, rs + DM/4, rs + DM/2, rs + 3 DM/4; rs = 4 * wave + lane / 16, so the
  // live rows of a step are spread over all wavefronts) and split their float4
  // column groups (c16, c16 + 16, ...). LDS passes only the vectors (v, p, the
  // next column), so a step is one chain: column -> norm (fp64) -> v -> p.
  // Entries of v outside the live block are zero, so the pass needs no masks:
  // dead entries take part with zeros (or change without being read again), and
  // a block of rows that is dead as a whole is left out.
  // What bounds it: that chain with one wavefront a SIMD, where every
  // instruction counts (about 8 cycles each; 1,800 cycles a step at d = 64). With
  // the matrix in LDS, masks per entry and two more waits a step it was 2,400.
  // The whole kernel took 152 us for 16 problems at d = 64 and 423 us for 80 at
  // d = 128; now 118 and 344 us (with the second inverse-iteration step reusing
  // the first one's factorisation, and every global read issued ahead of its
  // use).
  const int nref = d > 2 ? d - 2 : 0;
  {
    constexpr int RPT = 4;               // rows per lane
    constexpr int NG = DM / 64;          // column groups per lane
    const int c16 = lane & 15, rs = 4 * wv + (lane >> 4);
    float ar[NG][RPT][4];
#pragma unroll
    for (int q = 0; q < NG; ++q)
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        const float4 a = *reinterpret_cast<const float4*>(
            &A[(rs + r * (DM / RPT)) * EP + 4 * (c16 + 16 * q)]);
        ar[q][r][0] = a.x; ar[q][r][1] = a.y; ar[q][r][2] = a.z; ar[q][r][3] = a.w;
      }
    // before the first step: no reflector yet, and column 0 as it is
    if (tid < DM) {
      colb[1][tid] = *reinterpret_cast<const float4*>(&A[tid * EP]);
      pbuf[1][tid] = 0.f;
    }
#pragma unroll
    for (int h = 0; h < CPL; ++h) vvs[1][wv][lane + 64 * h] = 0.f;
    if (tid < NW) kpart[1][tid] = 0.f;
    __syncthreads();  // A is read: its rows take the reflectors from here
    float vr[RPT] = {0.f, 0.f, 0.f, 0.f}, pr[RPT] = {0.f, 0.f, 0.f, 0.f};  // v and p at own rows
    auto step = [&](auto r0_tag, int k) __attribute__((always_inline)) {
#pragma clang fp contract(off)
      constexpr int R0 = decltype(r0_tag)::value;  // row blocks below R0 are done with
      const int cur = k & 1, prv = cur ^ 1;
      float* vcur = vvs[cur][wv];
      const float* vprv = vvs[prv][wv];
      const float* pprv = pbuf[prv];
      float Kp = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) Kp += kpart[prv][w];
      Kp *= 0.5f;
      const float* colk = reinterpret_cast<const float*>(colb[prv]) + (k & 3);  // column k
      const float vk = vprv[k], akk = colk[4 * k];
      const float wk = __builtin_fmaf(-Kp, vk, pprv[k]);
      // column k below the diagonal (every wavefront, one or two rows a lane)
      float x[CPL];
      double s2 = 0.0;
#pragma unroll
      for (int h = 0; h < CPL; ++h) {
        const int i = lane + 64 * h;
        const float vi = vprv[i], wi = __builtin_fmaf(-Kp, vi, pprv[i]);
        const float xi = colk[4 * i] - __builtin_fmaf(wk, vi, vk * wi);
        x[h] = i > k && i < d ? xi : 0.f;
        s2 = fma((double)x[h], (double)x[h], s2);  // the product is exact
      }
      s2 = wave_sum(s2);
      // the block after H_{k-1}, and its column k + 1 for the next step
      const int kn = k + 1;
#pragma unroll
      for (int q = 0; q < NG; ++q) {
        const int j0 = 4 * (c16 + 16 * q);
        const float4 vp = *reinterpret_cast<const float4*>(&vprv[j0]);
        const float4 pp = *reinterpret_cast<const float4*>(&pprv[j0]);
        const float vpv[4] = {vp.x, vp.y, vp.z, vp.w};
        const float wpv[4] = {__builtin_fmaf(-Kp, vp.x, pp.x), __builtin_fmaf(-Kp, vp.y, pp.y),
                              __builtin_fmaf(-Kp, vp.z, pp.z), __builtin_fmaf(-Kp, vp.w, pp.w)};
#pragma unroll
        for (int r = R0; r < RPT; ++r) {
          const float wr = __builtin_fmaf(-Kp, vr[r], pr[r]);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            ar[q][r][e] = ar[q][r][e] - __builtin_fmaf(vr[r], wpv[e], wr * vpv[e]);
        }
        if ((kn >> 2) == c16 + 16 * q)
#pragma unroll
          for (int r = R0; r < RPT; ++r)
            colb[cur][rs + r * (DM / RPT)] =
                make_float4(ar[q][r][0], ar[q][r][1], ar[q][r][2], ar[q][r][3]);
      }
      const int i0 = k + 1;
      float x0 = x[0];
#pragma unroll
      for (int h = 1; h < CPL; ++h) x0 = (i0 >> 6) == h ? x[h] : x0;
      x0 = read_lane(x0, i0 & 63);
      // sigma = |x|, alpha = -sign(x0) sigma, scale 1 / sqrt(sigma (sigma + |x0|)):
      // hardware reciprocal square roots with one Newton step each
      double rs2 = __builtin_amdgcn_rsq(s2);
      rs2 = rs2 * fma(-0.5 * s2 * rs2, rs2, 1.5);
      const double sig = s2 > 0.0 ? s2 * rs2 : 0.0;
      const double alpha = x0 >= 0.f ? -sig : sig;
      const double hq = sig * (sig + fabs((double)x0));
      double scl = __builtin_amdgcn_rsq(hq);
      scl = s2 > 0.0 ? scl * fma(-0.5 * hq * scl, scl, 1.5) : 0.0;
#pragma unroll
      for (int h = 0; h < CPL; ++h) {
        const int i = lane + 64 * h;
        const float vi = (float)(((double)x[h] - (i == i0 ? alpha : 0.0)) * scl);
        x[h] = i > k && i < d ? vi : 0.f;
        vcur[i] = x[h];
      }
      // one wavefront's LDS operations run in order: its reads of v need no wait
      asm volatile("" ::: "memory");
      // p = A v over the rows
      float acc[RPT];
#pragma unroll
      for (int r = R0; r < RPT; ++r) {
        vr[r] = vcur[rs + r * (DM / RPT)];
        acc[r] = 0.f;
      }
#pragma unroll
      for (int q = 0; q < NG; ++q) {
        const float4 vn = *reinterpret_cast<const float4*>(&vcur[4 * (c16 + 16 * q)]);
        const float vnv[4] = {vn.x, vn.y, vn.z, vn.w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int r = R0; r < RPT; ++r) acc[r] = acc[r] + ar[q][r][e] * vnv[e];
      }
      // row sums over the 16 lanes of the DPP row (every lane gets them)
#pragma unroll
      for (int r = R0; r < RPT; ++r) acc[r] = quad_sum(acc[r]);
#pragma unroll
      for (int r = R0; r < RPT; ++r) acc[r] = dpp_add<0x141>(acc[r]);  // row_half_mirror
#pragma unroll
      for (int r = R0; r < RPT; ++r) acc[r] = dpp_add<0x140>(acc[r]);  // row_mirror
      float vp_part = 0.f;
#pragma unroll
      for (int r = R0; r < RPT; ++r) {
        const int row = rs + r * (DM / RPT);
        pr[r] = row > k && row < d ? acc[r] : 0.f;
        vp_part = vp_part + vr[r] * pr[r];
      }
      if (c16 == 0)
#pragma unroll
        for (int r = R0; r < RPT; ++r) pbuf[cur][rs + r * (DM / RPT)] = pr[r];
      vp_part = dpp_add<0x142, 0xA>(vp_part);  // row_bcast15 into rows 1, 3
      vp_part = dpp_add<0x143, 0xC>(vp_part);  // row_bcast31 into rows 2, 3: lane 63 holds the sum
      if (lane == 63) kpart[cur][wv] = vp_part;
      if (wv == 0) {  // the reflector and T's entries, kept for the later stages
#pragma unroll
        for (int h = 0; h < CPL; ++h) A[k * EP + lane + 64 * h] = x[h];
        if (lane == 0) {
          trid[0][k] = __builtin_fmaf(-wk, vk + vk, akk);
          trid[1][k] = (float)alpha;
        }
      }
      __syncthreads();
    };
    // rows rs + r DM/4 of block r are all at or above the diagonal once k
    // reaches (r + 1) DM/4 - 1
    auto upto = [&](auto r0_tag, int k0) __attribute__((always_inline)) {
      constexpr int R0 = decltype(r0_tag)::value;
      int k = k0;
      for (; k < min(nref, (R0 + 1) * (DM / RPT) - 1); ++k) step(r0_tag, k);
      return k;
    };
    int kh = upto(std::integral_constant<int, 0>{}, 0);
    kh = upto(std::integral_constant<int, 1>{}, kh);
    kh = upto(std::integral_constant<int, 2>{}, kh);
    for (; kh < nref; ++kh) step(std::integral_constant<int, 3>{}, kh);
    // the last 2 x 2 block after the last reflector
    if (d >= 2) {
#pragma unroll
      for (int q = 0; q < NG; ++q)
#pragma unroll
        for (int r = 0; r < RPT; ++r)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int row = rs + r * (DM / RPT), j = 4 * (c16 + 16 * q) + e;
            if (row >= d - 2 && row < d && j >= d - 2 && j < d)
              last2[row - (d - 2)][j - (d - 2)] = ar[q][r][e];
          }
    }
    __syncthreads();
    if (tid == 0) {
      if (d == 1) {
        trid[0][0] = ar[0][0][0];
      } else if (d >= 2) {
        const int i = d - 2, j = d - 1;
        float vi = 0.f, wi = 0.f, vj = 0.f, wj = 0.f;
        if (nref > 0) {
          const int l = (nref - 1) & 1;
          float Kp = 0.f;
          for (int w = 0; w < NW; ++w) Kp += kpart[l][w];
          Kp *= 0.5f;
          vi = vvs[l][0][i];
          vj = vvs[l][0][j];
          wi = pbuf[l][i] - Kp * vi;
          wj = pbuf[l][j] - Kp * vj;
        }
        trid[0][i] = last2[0][0] - 2.f * vi * wi;
        trid[0][j] = last2[1][1] - 2.f * vj * wj;
        trid[1][i] = last2[1][0] - (vj * wi + wj * vi);
      }
    }
    __syncthreads();
  }
  // ---- 2. scaling, deflation, blocks (wavefront 0), then bisection
  if (wv == 0) {
    double tn = 0.0;
    double dv[CPL], ev[CPL];
#pragma unroll
    for (int h = 0; h < CPL; ++h) {
      const int i = lane + 64 * h;
      dv[h] = i < d ? (double)trid[0][i] : 0.0;
      ev[h] = i + 1 < d ? (double)trid[1][i] : 0.0;
      const double el = i >= 1 && i < d ? fabs((double)trid[1][i - 1]) : 0.0;
      tn = fmax(tn, fabs(dv[h]) + fabs(ev[h]) + el);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) tn = fmax(tn, __shfl_xor(tn, o, 64));
    const double inv_tn = tn > 0.0 ? 1.0 / tn : 0.0;
    uint64_t brk[CPL];
#pragma unroll
    for (int h = 0; h < CPL; ++h) {
      const int i = lane + 64 * h;
      double e = ev[h] * inv_tn;
      if (fabs(e) <= kDeflate) e = 0.0;
      es[i] = e;
      // a block ends after i when i is the last index or T decouples there
      brk[h] = __ballot(i < d && (i == d - 1 || e == 0.0));
    }
    wave_lds_order();
#pragma unroll
    for (int h = 0; h < CPL; ++h) {
      const int i = lane + 64 * h;
      const double em = i >= 1 ? es[i - 1] : 0.0;
      tq[i] = make_double2(dv[h] * inv_tn, em * em);
      // start: one past the last break before i; end: one past the first break at or after i
      int st = 0, en = d;
#pragma unroll
      for (int g = CPL - 1; g >= 0; --g) {
        if (g > h) continue;
        const uint64_t m = g == h ? (lane == 0 ? 0ull : (brk[g] & ((~0ull) >> (64 - lane)))) : brk[g];
        if (m && st == 0) st = 64 * g + 63 - __builtin_clzll(m) + 1;
      }
#pragma unroll
      for (int g = 0; g < CPL; ++g) {
        if (g < h) continue;
        const uint64_t m = g == h ? (brk[g] & ((~0ull) << lane)) : brk[g];
        if (m && en == d) en = 64 * g + __builtin_ctzll(m) + 1;
      }
      bs[i] = i < d ? st : 0;
      be[i] = i < d ? en : 1;
    }
    if (lane == 0) sh_tn = tn;
  }
  __syncthreads();
  const double tn = sh_tn;
  {
    const int g = tid / kEighM, q = tid % kEighM;
    const bool live = g < d && tn > 0.0;
    const int s = live ? bs[g] : 0, t = live ? be[g] : 1, j = g - s;
    double lo = -1.0 - 0x1p-40, hi = 1.0 + 0x1p-40;
    for (int round = 0; round < kBisectRounds; ++round) {
      const double step = (hi - lo) / (double)(kEighM + 1);
      const int c = live ? sturm_below(tq, s, t, lo + step * (double)(q + 1)) : 0;
      // counts of the quad's four points (quad_perm broadcasts)
      const int below = (__builtin_amdgcn_update_dpp(0, c, 0x00, 0xF, 0xF, false) <= j) +
                        (__builtin_amdgcn_update_dpp(0, c, 0x55, 0xF, 0xF, false) <= j) +
                        (__builtin_amdgcn_update_dpp(0, c, 0xAA, 0xF, 0xF, false) <= j) +
                        (__builtin_amdgcn_update_dpp(0, c, 0xFF, 0xF, 0xF, false) <= j);
      const double nlo = below > 0 ? lo + step * (double)below : lo;
      const double nhi = below < kEighM ? lo + step * (double)(below + 1) : hi;
      lo = nlo;
      hi = nhi;
    }
    if (q == 0) lam64[g] = live ? 0.5 * (lo + hi) : 0.0;
  }
  __syncthreads();
  // ---- 3. eigenvectors of T: clusters (wavefront 0), start vectors (all)
  if (wv == 0) {
#pragma unroll
    for (int h = 0; h < CPL; ++h) {
      const int g = lane + 64 * h;
      const bool link = g >= 1 && g < d && bs[g] == bs[g - 1] &&
                        lam64[g] - lam64[g - 1] < kClusterTol;
      const uint64_t m = __ballot(link);
      if (lane == 0) sh_link[h] = m;
    }
  }
  for (int idx = tid; idx < DM * DM; idx += NT) {
    const int g = idx / DM, i = idx % DM;
    const bool in = g < d && i >= bs[g] && i < be[g];
    Vt[g * EP + i] = in ? (tn > 0.0 ? start_value(g, i) : (i == g ? 1.f : 0.f)) : 0.f;
  }
  __syncthreads();
  if (tn > 0.0) {
    // vector g on the kEighM lanes of a quad, SEG consecutive entries each.
    // No per-entry masks: the off-diagonal entry at each end of g's block is
    // zero, so both recurrences restart there, and the start vector is zero
    // outside the block, so those entries stay exactly zero.
    constexpr int SEG = DM / kEighM;
    const int g = tid / kEighM, part = tid % kEighM;
    const bool live = g < d;
    const double sigma = live ? lam64[g] : 0.0;
    float* z = Vt + (size_t)(live ? g : 0) * EP + SEG * part;
    const double2* tqs = tq + SEG * part;
    const double* ess = es + SEG * part;
    double r[SEG];     // 1 / pivot of this lane's entries, kept for the second step
    double lin = 0.0;  // the L entry that leads into this lane's segment
    for (int it = 0; it < 2; ++it) {
      // forward: T - sigma I = L D L^T (first step only), y = L^{-1} b (kept
      // in z, scaled); the quad's lanes take their segments in turn, passing
      // (l, y) on
      double lprev = 0.0, yprev = 0.0;
#pragma unroll
      for (int h = 0; h < kEighM; ++h) {
        if (h > 0) {
          const int src = (lane & ~(kEighM - 1)) + h - 1;
          lprev = __shfl(lprev, src, 64);
          yprev = __shfl(yprev, src, 64);
        }
        if (live && part == h) {
          if (it == 0) {
            lin = lprev;
#pragma unroll
            for (int u = 0; u < SEG; ++u) {
              if ((u & 7) == 0) asm volatile("" ::: "memory");
              const double a = tqs[u].x - sigma;
              const double em = u > 0 ? ess[u - 1] : (h > 0 ? es[SEG * h - 1] : 0.0);
              double dl = fma(-lprev, em, a);
              const double y = fma(-lprev, yprev, (double)z[u]);
              dl = fabs(dl) < kPivMin ? (dl < 0.0 ? -kPivMin : kPivMin) : dl;
              r[u] = recip64(dl);
              lprev = ess[u] * r[u];
              yprev = y;
              z[u] = (float)(y * kStore);
            }
          } else {
            lprev = lin;
#pragma unroll
            for (int u = 0; u < SEG; ++u) {
              if ((u & 7) == 0) asm volatile("" ::: "memory");
              const double y = fma(-lprev, yprev, (double)z[u]);
              lprev = ess[u] * r[u];
              yprev = y;
              z[u] = (float)(y * kStore);
            }
          }
        }
      }
      // backward: x = D^{-1} y - L^T x, kept in z (scaled); max |x|
      double xn = 0.0, mx = 0.0;
#pragma unroll
      for (int h = kEighM - 1; h >= 0; --h) {
        if (h < kEighM - 1) xn = __shfl(xn, (lane & ~(kEighM - 1)) + h + 1, 64);
        if (live && part == h) {
#pragma unroll
          for (int u = SEG - 1; u >= 0; --u) {
            if ((u & 7) == 7) asm volatile("" ::: "memory");
            const double xv = r[u] * fma(-ess[u], xn, (double)z[u] * (1.0 / kStore));
            xn = xv;
            mx = fmax(mx, fabs(xv));
            z[u] = (float)(xv * kStore);
          }
        }
      }
      mx = fmax(mx, __shfl_xor(mx, 1, 64));
      mx = fmax(mx, __shfl_xor(mx, 2, 64));
      // normalise
      const double sc = mx > 0.0 ? 1.0 / (mx * kStore) : 0.0;
      double ss = 0.0;
      if (live)
#pragma unroll
        for (int u = 0; u < SEG; ++u) {
          const double v = (double)z[u] * sc;
          ss += v * v;
        }
      ss = quad_sum(ss);
      const double nrm = ss > 0.0 ? sc / sqrt(ss) : 0.0;
      if (live)
#pragma unroll
        for (int u = 0; u < SEG; ++u) z[u] = (float)((double)z[u] * nrm);
      __syncthreads();
      // clusters: modified Gram-Schmidt in slot order (wavefront 0)
      if (wv == 0) {
        for (int h = 0; h < CPL; ++h) {
          uint64_t m = sh_link[h];
          while (m) {
            const int gj = 64 * h + __builtin_ctzll(m);
            m &= m - 1;
            int g0 = gj;
            while (g0 > 0 && ((sh_link[g0 >> 6] >> (g0 & 63)) & 1)) --g0;
            float zj[CPL];
#pragma unroll
            for (int c = 0; c < CPL; ++c) zj[c] = Vt[gj * EP + lane + 64 * c];
            for (int gi = g0; gi < gj; ++gi) {
              float dot = 0.f;
#pragma unroll
              for (int c = 0; c < CPL; ++c) dot += Vt[gi * EP + lane + 64 * c] * zj[c];
              dot = wave_sum(dot);
#pragma unroll
              for (int c = 0; c < CPL; ++c) zj[c] -= dot * Vt[gi * EP + lane + 64 * c];
            }
            float nn = 0.f;
#pragma unroll
            for (int c = 0; c < CPL; ++c) nn += zj[c] * zj[c];
            nn = wave_sum(nn);
            const float rn = nn > 0.f ? 1.f / sqrtf(nn) : 0.f;
#pragma unroll
            for (int c = 0; c < CPL; ++c) Vt[gj * EP + lane + 64 * c] = zj[c] * rn;
            wave_lds_order();
          }
        }
      }
      __syncthreads();
    }
  }
  // ---- 4. back-transformation: vector g (rows split over kEighM threads)
  const bool fv = jb.t_f >= 0;
  float lf[RI * CPL];  // F of the epilogue, read meanwhile
  if (fv) load_square<RI, CPL, NW>(mat(C, bh, jb.t_f), d, wv, lane, lf);
  {
    const int g = tid / kEighM, c = tid % kEighM;
    float zr[RW];
#pragma unroll
    for (int u = 0; u < RW; u += 4) {
      const float4 v4 = *reinterpret_cast<const float4*>(&Vt[g * EP + c * RW + u]);
      zr[u] = v4.x;
      zr[u + 1] = v4.y;
      zr[u + 2] = v4.z;
      zr[u + 3] = v4.w;
    }
    float nv[RW];  // the next reflector, read one step ahead
    auto fetch = [&](int k) {
#pragma unroll
      for (int u = 0; u < RW; u += 4) {
        const float4 v4 = *reinterpret_cast<const float4*>(&A[k * EP + c * RW + u]);
        nv[u] = v4.x;
        nv[u + 1] = v4.y;
        nv[u + 2] = v4.z;
        nv[u + 3] = v4.w;
      }
    };
    if (nref > 0) fetch(nref - 1);
    for (int k = nref - 1; k >= 0; --k) {
      float vr[RW];
      float dp[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < RW; ++u) vr[u] = nv[u];
      fetch(k > 0 ? k - 1 : 0);
#pragma unroll
      for (int u = 0; u < RW; ++u) dp[u & 3] = __builtin_fmaf(vr[u], zr[u], dp[u & 3]);
      const float dot = quad_sum((dp[0] + dp[1]) + (dp[2] + dp[3]));
#pragma unroll
      for (int u = 0; u < RW; ++u) zr[u] = __builtin_fmaf(-dot, vr[u], zr[u]);
    }
#pragma unroll
    for (int u = 0; u < RW; u += 4)
      *reinterpret_cast<float4*>(&Vt[g * EP + c * RW + u]) =
          make_float4(zr[u], zr[u + 1], zr[u + 2], zr[u + 3]);
  }
  __syncthreads();
  float* Ac = A;
  const float* Vc = Vt;
  // ---- epilogue: eigenvalues, ranks (descending, ties by index), orientation
  if (tid < d) {
    lam[tid] = (float)(lam64[tid] * tn);
    float o4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int t = 0; t < d; t += 4) {
      const float4 ov = *reinterpret_cast<const float4*>(&ovec[t]);
      const float4 vv = *reinterpret_cast<const float4*>(&Vc[tid * EP + t]);
      o4[0] = __builtin_fmaf(ov.x, vv.x, o4[0]);
      o4[1] = __builtin_fmaf(ov.y, vv.y, o4[1]);
      o4[2] = __builtin_fmaf(ov.z, vv.z, o4[2]);
      o4[3] = __builtin_fmaf(ov.w, vv.w, o4[3]);
    }
    const float o = (o4[0] + o4[1]) + (o4[2] + o4[3]);
    sgn[tid] = o < 0.f ? -1.f : 1.f;
    inv[tid] = tid;  // (the ranks below leave entries out where eigenvalues are NaN)
  }
  __syncthreads();
  if (tid < d) {
    const float li = lam[tid];
    int r = 0;
#pragma unroll 8
    for (int j = 0; j < d; ++j) {
      const float lj = lam[j];
      r += (lj > li) || (lj == li && j < tid);
    }
    inv[r] = tid;
  }
  __syncthreads();
  float* T = mat(C, bh, jb.t_out);
  bf16* W = jb.wop_out >= 0 ? wop(C, bh, jb.wop_out) : nullptr;
  // Eigenvector g becomes column rnk[g] of U: U[r][c] = sgn[g] Vc[g][r], g = inv[c].
  // The projection T[r][c] = sgn[g] P[r][g] with P = F V (t_f) or V, and its
  // bf16 operand pair W[c][r] (hi) and W[d * d + c * d + r] (lo).
  const float* P = Vc;  // P[r][g] at Vc[g * EP + r] (V), or at Ac[r * EP + g] (F V)
  if (fv) {
    // P = F V: F goes into the A region
#pragma unroll
    for (int ii = 0; ii < RI; ++ii)
#pragma unroll
      for (int cc = 0; cc < CPL; ++cc)
        Ac[(wv + NW * ii) * EP + lane + 64 * cc] = lf[ii * CPL + cc];
    __syncthreads();
    MMAcc acc;
    lds_mm<NT>(Ac, false, Vc, true, EP, d, acc);
    __syncthreads();
    lds_mm_store<NT>(acc, Ac, EP, d);
    __syncthreads();
    P = Ac;
  }
#pragma unroll 4
  for (int r = wv; r < d; r += NW)
#pragma unroll
    for (int cc = 0; cc < CPL; ++cc) {
      const int c = lane + 64 * cc;
      if (c < d) {
        const int g = inv[c];
        T[r * d + c] = sgn[g] * (fv ? P[r * EP + g] : P[g * EP + r]);
      }
    }
  if (W)
#pragma unroll 4
    for (int c = wv; c < d; c += NW) {
      const int g = inv[c];
#pragma unroll
      for (int cc = 0; cc < CPL; ++cc) {
        const int r = lane + 64 * cc;
        if (r < d) {
          const float v = sgn[g] * (fv ? P[r * EP + g] : P[g * EP + r]);
          const bf16 hi = (bf16)v;
          W[c * d + r] = hi;
          W[d * d + c * d + r] = (bf16)(v - (float)hi);
        }
      }
    }
}

// ---------------------------------------------------------------------------
// Metric roots: a factor F with F F^T = M. Any such factor gives the same
// split coordinates after the principal-axis step (F = E sqrt(L) R for an
// orthogonal R, which the principal axes absorb), so the root of each metric
// is taken as its Cholesky factor, in fp64; pivots below a relative threshold
// are treated as zero (positive semi-definite metrics; this equals clamping
// the eigenvalues at zero up to rounding).
// ---------------------------------------------------------------------------

// What bounds it: the chain of d elimination steps, one workgroup per matrix.
// The matrix lives in registers, 4 x 4 entries a thread spread cyclically over
// a DM/4 x DM/4 thread grid, so a step only passes the next column and the
// reciprocal of its pivot through LDS: one round trip and one barrier. With
// the matrix in LDS (read, updated and written there at every step, and the
// pivot divided in every thread) the 16 problems of an 8-head layer at d = 64
// took 47.6 us and the 80 problems of a 40-head layer at d = 128 193.8 us; now
// 21.3 and 54.9 us. The operations on each entry and their order
// are the same, so the factors are the same bits.
template <int DM>
constexpr int chol_threads() {
  return (DM / 4) * (DM / 4);
}

template <int DM>
__global__ __launch_bounds__(chol_threads<DM>()) void cholesky_kernel(Ctx C, int in0, int out0,
                                                                      int in1, int out1,
                                                                      int pack1) {
  constexpr int G = DM / 4, FP = DM + 1;
  __shared__ double col[2][DM];  // the step's column (unscaled), by parity
  __shared__ double rcp[2];      // 1 / its pivot, 0 for a pivot at or below tol
  __shared__ double piv[DM], ipiv[DM];
  __shared__ double sh_tol;
  extern __shared__ __attribute__((aligned(16))) float chf[];  // [DM][FP] the factor (pack only)
  const int bh = blockIdx.x, job = blockIdx.y, d = C.d, tid = threadIdx.x;
  const int tr = tid / G, tc = tid % G;
  const float* M = mat(C, bh, job == 0 ? in0 : in1);
  float* F = mat(C, bh, job == 0 ? out0 : out1);
  const int pack = job == 1 ? pack1 : -1;
  double A[4][4];  // entry (tr + G a, tc + G b)
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int i = tr + G * a, k = tc + G * b;
      A[a][b] = i < d && k < d ? (double)M[i * d + k] : 0.0;
    }
  if (tid < 64) {
    double mx = 0.0;
#pragma unroll
    for (int i = tid; i < DM; i += 64) mx = fmax(mx, i < d ? (double)M[i * d + i] : 0.0);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
    if (tid == 0) sh_tol = mx * 1e-12;
  }
  __syncthreads();
  const double tol = sh_tol;
  if (tc == 0) {
#pragma unroll
    for (int a = 0; a < 4; ++a) col[0][tr + G * a] = A[a][0];
    if (tr == 0) rcp[0] = A[0][0] > tol ? 1.0 / A[0][0] : 0.0;
  }
  __syncthreads();
  // Elimination on unscaled columns (the order of an L D L^T factorisation):
  // step j subtracts a_ij a_kj / a_jj from the trailing lower triangle (rows
  // i > j, columns j < k <= i) and leaves column j as it is. A pivot at or
  // below tol contributes nothing and gives a zero column. Entries above the
  // diagonal hold values that nothing reads.
#pragma unroll
  for (int jb = 0; jb < 4; ++jb) {
    for (int jj = 0; jj < G; ++jj) {
      const int j = jb * G + jj;
      if (j >= d) break;
      const int cur = j & 1;
      const double inv = rcp[cur];
      double l[4], ak[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        l[a] = a >= jb ? col[cur][tr + G * a] * inv : 0.0;
        // columns up to j are final
        ak[a] = a > jb || (a == jb && tc > jj) ? col[cur][tc + G * a] : 0.0;
      }
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
          if (a >= b && b >= jb) A[a][b] = fma(-l[a], ak[b], A[a][b]);
      // column j + 1 and the reciprocal of its pivot, for the next step
      const bool wrap = jj == G - 1;
      const int jn = j + 1;
      if (jn < d && tc == (wrap ? 0 : jj + 1)) {
        double nx[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          nx[a] = wrap && jb < 3 ? A[a][jb < 3 ? jb + 1 : jb] : A[a][jb];
          if (a >= jb) col[cur ^ 1][tr + G * a] = nx[a];
        }
        if (tr == tc) {
          const double dj = wrap && jb < 3 ? nx[jb < 3 ? jb + 1 : jb] : nx[jb];
          rcp[cur ^ 1] = dj > tol ? 1.0 / dj : 0.0;
        }
      }
      __syncthreads();
    }
  }
  // Scale: l_jj = sqrt(a_jj), l_ij = a_ij / l_jj.
  if (tr == tc)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const double dj = A[a][a];
      const double p = dj > tol ? sqrt(dj) : 0.0;
      piv[tr + G * a] = p;
      ipiv[tr + G * a] = p > 0.0 ? 1.0 / p : 0.0;
    }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int i = tr + G * a, k = tc + G * b;
      const float f = k > i ? 0.f : (float)(k == i ? piv[k] : A[a][b] * ipiv[k]);
      if (i < d && k < d) F[i * d + k] = f;
      if (pack >= 0) chf[i * FP + k] = f;
    }
  if (pack >= 0) {
    // transposed hi/lo bf16 operand of the factor (the MFMA query pass)
    __syncthreads();
    bf16* out = wop(C, bh, pack);
    for (int e = tid; e < d * d; e += chol_threads<DM>()) {
      const int i = e / d, k = e % d;  // out row i (output dim), column k (input dim)
      const float w = chf[k * FP + i];
      const bf16 hi = (bf16)w;
      out[e] = hi;
      out[d * d + e] = (bf16)(w - (float)hi);
    }
  }
}

// Metric mode, queries: rho = q S_k, inv = 1/|rho| (0 if rho = 0), r = rho*inv;
// partial sums of r r^T and r per row block; inv is kept for the projection.
__global__ __launch_bounds__(256) void qnorm_partial_kernel(Ctx C) {
  extern __shared__ __attribute__((aligned(16))) float qsh[];
  float* Sk = qsh;                                        // [d][kDP]
  float (*X)[kDP] = (float(*)[kDP])(qsh + kMaxD * kDP);   // [kStage][kDP]
  float (*R)[kDP] = (float(*)[kDP])(qsh + (kMaxD + kStage) * kDP);
  __shared__ float invs[kStage];
  const int bh = blockIdx.y, blk = blockIdx.x, d = C.d, d4 = (d + 3) / 4;
  const Side& S = C.s[0];
  const float* Skg = mat(C, bh, M_EK);
  for (int e = threadIdx.x; e < d * 4 * d4; e += 256) {
    const int t = e / (4 * d4), j = e % (4 * d4);
    Sk[t * kDP + j] = j < d ? Skg[t * d + j] : 0.f;
  }
  const int r0 = blk * C.mom_rows, r1 = min(S.n, r0 + C.mom_rows);
  float acc[4][16];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[q][e] = 0.f;
  float csum = 0.f;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int rs = r0; rs < r1; rs += kStage) {
    const int rows = min(kStage, r1 - rs);
    __syncthreads();
    for (int e = threadIdx.x; e < kStage * 4 * d4; e += 256) {
      const int r = e / (4 * d4), t = e % (4 * d4);
      X[r][t] = (r < rows && t < d) ? load_x(S.x, bh, rs + r, S.lx, t, C.dtype)
                                    : 0.f;
    }
    __syncthreads();
    // rho for the staged rows
    for (int e = threadIdx.x; e < kStage * d4; e += 256) {
      const int r = e / d4, j4 = e % d4;
      float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
#pragma unroll 8
      for (int t = 0; t < d; ++t) {
        const float xv = X[r][t];
        const float4 s4 = *(const float4*)&Sk[t * kDP + 4 * j4];
        a0 = __builtin_fmaf(xv, s4.x, a0);
        a1 = __builtin_fmaf(xv, s4.y, a1);
        a2 = __builtin_fmaf(xv, s4.z, a2);
        a3 = __builtin_fmaf(xv, s4.w, a3);
      }
      *(float4*)&R[r][4 * j4] = make_float4(a0, a1, a2, a3);
    }
    __syncthreads();
    // one wave per row: 1/|rho|
    float ss[kStage / 4];  // rows w, w + 4, ...: their reductions overlap
#pragma unroll
    for (int q = 0; q < kStage / 4; ++q) {
      const int r = w + 4 * q;
      ss[q] = 0.f;
      for (int t = lane; t < d; t += 64) ss[q] = __builtin_fmaf(R[r][t], R[r][t], ss[q]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
      for (int q = 0; q < kStage / 4; ++q) ss[q] += __shfl_xor(ss[q], o, 64);
#pragma unroll
    for (int q = 0; q < kStage / 4; ++q)
      if (lane == q) {
        const int r = w + 4 * q;
        const float inv = ss[q] > 0.f ? 1.f / sqrtf(ss[q]) : 0.f;
        invs[r] = inv;
        if (r < rows) C.inv_q[(size_t)bh * S.n + rs + r] = inv;
      }
    __syncthreads();
    for (int e = threadIdx.x; e < kStage * 4 * d4; e += 256) {
      const int r = e / (4 * d4), t = e % (4 * d4);
      R[r][t] = r < rows ? R[r][t] * invs[r] : 0.f;
    }
    __syncthreads();
    acc_outer(R, R, rows, d4, acc);
    if (threadIdx.x < d)
#pragma unroll 8
      for (int r = 0; r < rows; ++r) csum += R[r][threadIdx.x];
  }
  float* out = C.qn_part + ((size_t)bh * C.nblk + blk) * (d * d + d);
  write_outer(out, d, d4, acc);
  if (threadIdx.x < d) out[d * d + threadIdx.x] = csum;
}

// Means of the query-representation partials: M_C3 <- sum/n of the d x d part, V_MUR <- sum/n of the vector
// part. The partials hold either r r^T and r (then cov(r) = M_C3 - mu mu^T),
// or inv^2 x x^T and inv x (then cov(r) = S_k^T M_C3 S_k - u u^T with
// u = S_k^T V_MUR); the eigensolver's prologue forms cov(r).
__global__ __launch_bounds__(256) void qnorm_finish_kernel(Ctx C) {
  const int bh = blockIdx.y, d = C.d;
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= d * d + d) return;
  const size_t stride = (size_t)d * d + d;
  const float* part = C.qn_part + (size_t)bh * C.nblk * stride;
  const double v = sum_partials<1>(part + e, stride, C.nblk, nullptr, true) / (double)C.s[0].n;
  if (e < d * d)
    mat(C, bh, M_C3)[e] = (float)v;
  else
    vec(C, bh, V_MUR)[e - d * d] = (float)v;
}

// ---------------------------------------------------------------------------
// Projection Y = X T (fp32), or Y = X for the raw-coordinate mode.
// ---------------------------------------------------------------------------

constexpr int kProjRows = 256;  // rows per projection block (at most)

// Pseudo-random split coordinate in [0, 1) of the random-cluster control:
// output number c (counting from 0) of splitmix64 (S. Vigna's generator,
// started at state 0), top 24 bits, so the value is exact in fp32.
__device__ __forceinline__ float random_coord(int bh, int side, int i, int j) {
  const uint64_t c = ((((uint64_t)bh * 2 + (uint64_t)side) << 22 | (uint64_t)i) << 7) | (uint64_t)j;
  uint64_t z = (c + 1ull) * 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  z ^= z >> 31;
  return (float)(uint32_t)(z >> 40) * 0x1p-24f;
}

__global__ __launch_bounds__(256) void project_kernel(Ctx C) {
  extern __shared__ __attribute__((aligned(16))) float psh[];
  float* T = psh;                                        // [d][kDP]
  float (*X)[kDP] = (float(*)[kDP])(psh + kMaxD * kDP);  // [kStage][kDP]
  const int pid = blockIdx.y, side = pid / C.BH, bh = pid % C.BH;
  const Side& S = C.s[side];
  const int d = C.d, d4 = (d + 3) / 4;
  const int r0 = blockIdx.x * C.proj_rows, r1 = min(S.n, r0 + C.proj_rows);
  if (r0 >= r1) return;
  float* Y = S.y + (size_t)bh * S.n * d;
  if (C.xf == CA_XF_NONE) {
    for (int e = threadIdx.x; e < (r1 - r0) * d; e += 256) {
      const int r = r0 + e / d, t = e % d;
      Y[(size_t)r * d + t] = load_x(S.x, bh, r, S.lx, t, C.dtype);
    }
    return;
  }
  if (C.xf == CA_XF_RANDOM) {
    for (int e = threadIdx.x; e < (r1 - r0) * d; e += 256) {
      const int r = r0 + e / d, t = e % d;
      Y[(size_t)r * d + t] = random_coord(bh, side, r, t);
    }
    return;
  }
  const float* Tg = mat(C, bh, side == 0 ? M_TQ : M_TK);
  for (int e = threadIdx.x; e < d * 4 * d4; e += 256) {
    const int t = e / (4 * d4), j = e % (4 * d4);
    T[t * kDP + j] = j < d ? Tg[t * d + j] : 0.f;
  }
  const bool scale = side == 0 && C.xf == CA_XF_METRIC;
  for (int rs = r0; rs < r1; rs += kStage) {
    const int rows = min(kStage, r1 - rs);
    __syncthreads();
    for (int e = threadIdx.x; e < kStage * 4 * d4; e += 256) {
      const int r = e / (4 * d4), t = e % (4 * d4);
      X[r][t] = (r < rows && t < d) ? load_x(S.x, bh, rs + r, S.lx, t, C.dtype)
                                    : 0.f;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < rows * d4; e += 256) {
      const int r = e / d4, j4 = e % d4;
      float a[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
      for (int t = 0; t < d; ++t) {
        const float xv = X[r][t];
        const float4 t4 = *(const float4*)&T[t * kDP + 4 * j4];
        a[0] = __builtin_fmaf(xv, t4.x, a[0]);
        a[1] = __builtin_fmaf(xv, t4.y, a[1]);
        a[2] = __builtin_fmaf(xv, t4.z, a[2]);
        a[3] = __builtin_fmaf(xv, t4.w, a[3]);
      }
      const float sc = scale ? C.inv_q[(size_t)bh * S.n + rs + r] : 1.f;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (4 * j4 + j < d) Y[(size_t)(rs + r) * d + 4 * j4 + j] = a[j] * sc;
    }
  }
}

// ---------------------------------------------------------------------------
// MFMA versions of the dense passes (bf16 inputs, d in {64, 128}).
//
// A 32-token tile of X is held as MFMA operands: lane l owns token l % 32 and
// features 16 ks + 8 (l / 32) + [0, 8) for k-step ks, loaded with 16-byte
// reads straight from the rows. With X as the B operand and W^T as the A
// operand, (X W)^T comes out with one token per lane (column = token), so
// per-token scalings stay in the lane. For the second moments X^T X the tile
// is first transposed on the matrix core by multiplying with an identity
// operand (exact for bf16 data), which leaves one feature per lane.
// ---------------------------------------------------------------------------

template <int D>
__device__ __forceinline__ void load_xtile(const bf16* __restrict__ x, int bh, int tok0, int lim,
                                           const Lay& L, int l32, int h,
                                           bf16x8 (&xop)[D / 16]) {
  const int tok = tok0 + l32;
  if (tok < lim) {
    const bf16* row = x + row_off(bh, tok, L);
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) xop[ks] = *(const bf16x8*)(row + 16 * ks + 8 * h);
  } else {
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
      for (int u = 0; u < 8; ++u) xop[ks][u] = (bf16)0.f;
  }
}

// Identity operands: B[k][n] = 1 iff k == n for the two 16-row halves of a
// 32-wide feature tile.
__device__ __forceinline__ void ident_ops(int l32, int h, bf16x8 (&id)[2]) {
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int u = 0; u < 8; ++u) id[s][u] = (bf16)((l32 == 16 * s + 8 * h + u) ? 1.f : 0.f);
}

// xT[ft]: lane l holds feature 32 ft + l % 32 of tokens 8 (r/4) + 4 h + r % 4.
template <int D>
__device__ __forceinline__ void transpose_tile(const bf16x8 (&xop)[D / 16], const bf16x8 (&id)[2],
                                               f32x16 (&xT)[D / 32]) {
#pragma unroll
  for (int ft = 0; ft < D / 32; ++ft) {
#pragma unroll
    for (int r = 0; r < 16; ++r) xT[ft][r] = 0.f;
    xT[ft] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xop[2 * ft], id[0], xT[ft], 0, 0, 0);
    xT[ft] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xop[2 * ft + 1], id[1], xT[ft], 0, 0, 0);
  }
}

__device__ __forceinline__ bf16x8 pack_half(const f32x16& v, int s) {
  float t[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) t[j] = v[8 * s + j];
  return pack8(t);
}

// Stages the hi/lo W^T operands of one head into LDS (row = output dim,
// 2D-byte rows, chunk-swizzled).
template <int D>
__device__ __forceinline__ void stage_wops(const bf16* __restrict__ src, char* lds) {
  constexpr int ROWB = 2 * D, NCH = ROWB / 16;
  for (int c = threadIdx.x; c < 2 * D * NCH; c += 256) {
    const int m = c / (D * NCH), rem = c % (D * NCH);
    const int r = rem / NCH, lc = rem % NCH;
    *(uint4*)(lds + m * D * ROWB + swz_off<ROWB>(r, lc)) =
        *(const uint4*)(src + (size_t)m * D * D + r * D + lc * 8);
  }
}

// acc[ot] = (X W)^T tile ot (output dims 32 ot.., tokens = lanes) with W = hi + lo.
template <int D>
__device__ __forceinline__ void project_tile(const char* wl, const bf16x8 (&xop)[D / 16], int l32,
                                             int h, f32x16 (&acc)[D / 32]) {
  constexpr int ROWB = 2 * D;
#pragma unroll
  for (int ot = 0; ot < D / 32; ++ot) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[ot][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
      const int off = swz_off<ROWB>(32 * ot + l32, 2 * ks + h);
      const bf16x8 ahi = *(const bf16x8*)(wl + off);
      const bf16x8 alo = *(const bf16x8*)(wl + D * ROWB + off);
      acc[ot] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ahi, xop[ks], acc[ot], 0, 0, 0);
      acc[ot] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(alo, xop[ks], acc[ot], 0, 0, 0);
    }
  }
}

// Output tile ot of (X W)^T alone (dims 32 ot.., tokens = lanes).
template <int D>
__device__ __forceinline__ void project_tile1(const char* wl, const bf16x8 (&xop)[D / 16], int l32,
                                              int h, int ot, f32x16& acc) {
  constexpr int ROWB = 2 * D;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) {
    const int off = swz_off<ROWB>(32 * ot + l32, 2 * ks + h);
    const bf16x8 ahi = *(const bf16x8*)(wl + off);
    const bf16x8 alo = *(const bf16x8*)(wl + D * ROWB + off);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ahi, xop[ks], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(alo, xop[ks], acc, 0, 0, 0);
  }
}

// Adds the symmetric Gram tiles (it <= jt) of one wave into red[d][d] (and
// the mirror), waves in a fixed order.
template <int D>
__device__ __forceinline__ void reduce_gram(float* red, const f32x16* g, int w, int l32, int h) {
  constexpr int FT = D / 32;
  for (int wv = 0; wv < 4; ++wv) {
    if (w == wv) {
      int t = 0;
#pragma unroll
      for (int it = 0; it < FT; ++it)
#pragma unroll
        for (int jt = it; jt < FT; ++jt, ++t)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int i = 32 * it + 8 * (r >> 2) + 4 * h + (r & 3), j = 32 * jt + l32;
            const float v = g[t][r];
            red[i * D + j] = wv == 0 ? v : red[i * D + j] + v;
            if (it != jt) red[j * D + i] = wv == 0 ? v : red[j * D + i] + v;
          }
    }
    __syncthreads();
  }
}

template <int D>
__global__ __launch_bounds__(256) void moments_mfma_kernel(Ctx C) {
  constexpr int FT = D / 32, KS = D / 16, NT = FT * (FT + 1) / 2;
  __shared__ float red[D * D];
  __shared__ float csr[4][D];
  const int pid = blockIdx.y, side = pid / C.BH, bh = pid % C.BH, blk = blockIdx.x;
  const Side& S = C.s[side];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = lane >> 5, l32 = lane & 31;
  const int r0 = blk * C.mom_rows, r1 = min(S.n, r0 + C.mom_rows);
  bf16x8 id[2];
  ident_ops(l32, h, id);
  f32x16 g[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) g[t][r] = 0.f;
  float cs[FT];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) cs[ft] = 0.f;
  for (int tok0 = r0 + 32 * w; tok0 < r1; tok0 += 128) {
    bf16x8 xop[KS];
    load_xtile<D>((const bf16*)S.x, bh, tok0, r1, S.lx, l32, h, xop);
    f32x16 xT[FT];
    transpose_tile<D>(xop, id, xT);
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
      for (int r = 0; r < 16; ++r) cs[ft] += xT[ft][r];
    int t = 0;
#pragma unroll
    for (int it = 0; it < FT; ++it)
#pragma unroll
      for (int jt = it; jt < FT; ++jt, ++t)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
          g[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pack_half(xT[it], s2),
                                                          pack_half(xT[jt], s2), g[t], 0, 0, 0);
  }
  reduce_gram<D>(red, g, w, l32, h);
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
    const float v = cs[ft] + __shfl_xor(cs[ft], 32, 64);
    if (h == 0) csr[w][32 * ft + l32] = v;
  }
  __syncthreads();
  float* out = C.mom_part + ((size_t)pid * C.nblk + blk) * (D * D + D);
  for (int e = tid; e < D * D; e += 256) out[e] = red[e];
  for (int f = tid; f < D; f += 256) out[D * D + f] = ((csr[0][f] + csr[1][f]) + csr[2][f]) + csr[3][f];
}

// Metric mode, queries: rho = q S_k (MFMA, lane = token), inv = 1/|rho| (0 if
// rho = 0) kept for the projection, and per row block the partial sums of
// inv^2 x x^T and inv x (r r^T = S_k^T (inv^2 x x^T) S_k is formed after the
// reduction).
template <int D>
__global__ __launch_bounds__(256) void qnorm_mfma_kernel(Ctx C) {
  constexpr int FT = D / 32, KS = D / 16, NT = FT * (FT + 1) / 2;
  __shared__ __attribute__((aligned(16))) char wl[2 * D * 2 * D];
  __shared__ float red[D * D];
  __shared__ float csr[4][D];
  __shared__ float sinv[4][32];
  const int bh = blockIdx.y, blk = blockIdx.x;
  const Side& S = C.s[0];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = lane >> 5, l32 = lane & 31;
  stage_wops<D>(wop(C, bh, O_FK), wl);
  __syncthreads();
  const int r0 = blk * C.mom_rows, r1 = min(S.n, r0 + C.mom_rows);
  bf16x8 id[2];
  ident_ops(l32, h, id);
  f32x16 g[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) g[t][r] = 0.f;
  float cs[FT];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) cs[ft] = 0.f;
  for (int tok0 = r0 + 32 * w; tok0 < r1; tok0 += 128) {
    bf16x8 xop[KS];
    load_xtile<D>((const bf16*)S.x, bh, tok0, r1, S.lx, l32, h, xop);
    f32x16 acc[FT];
    project_tile<D>(wl, xop, l32, h, acc);
    float nrm = 0.f;
#pragma unroll
    for (int ot = 0; ot < FT; ++ot)
#pragma unroll
      for (int r = 0; r < 16; ++r) nrm = __builtin_fmaf(acc[ot][r], acc[ot][r], nrm);
    nrm += __shfl_xor(nrm, 32, 64);
    const float inv = nrm > 0.f ? 1.f / sqrtf(nrm) : 0.f;
    if (h == 0) {
      sinv[w][l32] = inv;
      if (tok0 + l32 < r1) C.inv_q[(size_t)bh * S.n + tok0 + l32] = inv;
    }
    __builtin_amdgcn_wave_barrier();
    f32x16 xT[FT];
    transpose_tile<D>(xop, id, xT);
    float wt[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) wt[r] = sinv[w][8 * (r >> 2) + 4 * h + (r & 3)];
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
      for (int r = 0; r < 16; ++r) cs[ft] = __builtin_fmaf(wt[r], xT[ft][r], cs[ft]);
    int t = 0;
#pragma unroll
    for (int it = 0; it < FT; ++it)
#pragma unroll
      for (int jt = it; jt < FT; ++jt, ++t)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          float bw[8], bl[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const float v = wt[8 * s2 + j] * wt[8 * s2 + j] * xT[jt][8 * s2 + j];
            bw[j] = v;
          }
          const bf16x8 bhi = pack8(bw);
#pragma unroll
          for (int j = 0; j < 8; ++j) bl[j] = bw[j] - (float)bhi[j];
          const bf16x8 a = pack_half(xT[it], s2);
          g[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bhi, g[t], 0, 0, 0);
          g[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pack8(bl), g[t], 0, 0, 0);
        }
    __builtin_amdgcn_wave_barrier();
  }
  reduce_gram<D>(red, g, w, l32, h);
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
    const float v = cs[ft] + __shfl_xor(cs[ft], 32, 64);
    if (h == 0) csr[w][32 * ft + l32] = v;
  }
  __syncthreads();
  float* out = C.qn_part + ((size_t)bh * C.nblk + blk) * (D * D + D);
  for (int e = tid; e < D * D; e += 256) out[e] = red[e];
  for (int f = tid; f < D; f += 256) out[D * D + f] = ((csr[0][f] + csr[1][f]) + csr[2][f]) + csr[3][f];
}

// Y = X T (keys) or inv * (X W_Q) (metric queries), lane = token, fp32 rows.
template <int D>
__global__ __launch_bounds__(256, 2) void project_mfma_kernel(Ctx C) {
  constexpr int FT = D / 32, KS = D / 16;
  __shared__ __attribute__((aligned(16))) char wl[2 * D * 2 * D];
  const int pid = blockIdx.y, side = pid / C.BH, bh = pid % C.BH;
  const Side& S = C.s[side];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = lane >> 5, l32 = lane & 31;
  const int r0 = blockIdx.x * C.proj_rows, r1 = min(S.n, r0 + C.proj_rows);
  if (r0 >= r1) return;
  stage_wops<D>(wop(C, bh, side == 0 ? O_TQ : O_TK), wl);
  __syncthreads();
  const bool scale = side == 0 && C.xf == CA_XF_METRIC;
  float* Y = S.y + (size_t)bh * S.n * D;
  for (int tok0 = r0 + 32 * w; tok0 < r1; tok0 += 128) {
    bf16x8 xop[KS];
    load_xtile<D>((const bf16*)S.x, bh, tok0, r1, S.lx, l32, h, xop);
    const int tok = tok0 + l32;
    const float sc = scale && tok < r1 ? C.inv_q[(size_t)bh * S.n + tok] : 1.f;
    float* yrow = Y + (size_t)tok * D;
    // one 32-column output tile at a time: a single accumulator stays live
    // (not unrolled, so the operand reads of later tiles are not hoisted)
#pragma unroll 1
    for (int ot = 0; ot < FT; ++ot) {
      f32x16 acc;
      project_tile1<D>(wl, xop, l32, h, ot, acc);
      if (tok < r1) {
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const int col = 32 * ot + 8 * g4 + 4 * h;
          *(float4*)(yrow + col) = make_float4(acc[4 * g4] * sc, acc[4 * g4 + 1] * sc,
                                               acc[4 * g4 + 2] * sc, acc[4 * g4 + 3] * sc);
        }
        // the same values of coordinates 0 .. 15, coordinate-major: each
        // store is 32 consecutive tokens of one coordinate per half-wave
        if (ot == 0 && S.ycol) {
          static_assert(kColCopy == 16, "coordinates of g4 = 0, 1 of the first tile");
#pragma unroll
          for (int g4 = 0; g4 < 2; ++g4)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              S.ycol[((size_t)bh * kColCopy + 8 * g4 + 4 * h + e) * S.n + tok] =
                  acc[4 * g4 + e] * sc;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Recursive split
// ---------------------------------------------------------------------------

// Position of subsample row j of m in a node of `size` tokens (at most 2^22):
// floor((2j + 1) size / (2m)).
__device__ __forceinline__ int sample_pos(int j, int size, int m) {
  const uint32_t x = (uint32_t)(2 * j + 1) * (uint32_t)size;
  return (int)((m & (m - 1)) == 0 ? x >> (__builtin_ctz(m) + 1) : x / (uint32_t)(2 * m));
}

// Highest-variance coordinate of the node's subsample, computed by one
// wavefront: lane t owns coordinates t and t + 64. fp64, two passes over the
// rows in order, mean = sum/m, variance = sum((y - mean)^2)/m, no contraction;
// ties go to the lowest coordinate. The sample rows are located first (lane j
// holds the row of sample j and j + 64), then read in batches of B independent
// loads, once for each pass; at most B samples are read once.
template <int B>
__device__ int choose_coordinate(const float* __restrict__ Y, int d, const int32_t* idx,
                                 bool identity, int start, int size, int lane,
                                 double* mean_out = nullptr, double* var_out = nullptr) {
#pragma clang fp contract(off)
  const int m = size < d ? size : d;
  int row[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int j = lane + 64 * h;
    int r = 0;
    if (j < m) {
      const int p = start + sample_pos(j, size, m);
      r = identity ? p : idx[p];
    }
    row[h] = r;
  }
  double best = -1.0, bmean = 0.0;
  int bt = 0x7fffffff;
  for (int half = 0; half * 64 < d; ++half) {
    const int t = lane + 64 * half;
    const bool tv = t < d;
    const float* Yt = Y + (tv ? t : 0);
    double acc = 0.0;
    float v[B];
    auto load = [&](int j0) {
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int j = j0 + u;
        const int r = __builtin_amdgcn_readlane(j < 64 ? row[0] : row[1], j & 63);
        v[u] = Yt[(size_t)r * d];
      }
    };
    for (int j0 = 0; j0 < m; j0 += B) {
      load(j0);
#pragma unroll
      for (int u = 0; u < B; ++u)
        if (j0 + u < m) acc = acc + (double)v[u];
    }
    const double mean = acc / (double)m;
    double acc2 = 0.0;
    for (int j0 = 0; j0 < m; j0 += B) {
      if (m > B) load(j0);  // (a single batch is still in registers)
#pragma unroll
      for (int u = 0; u < B; ++u)
        if (j0 + u < m) {
          const double dv = (double)v[u] - mean;
          const double sq = dv * dv;
          acc2 = acc2 + sq;
        }
    }
    const double var = acc2 / (double)m;
    if (tv && (var > best || (var == best && t < bt))) {
      best = var;
      bmean = mean;
      bt = t;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double ob = __shfl_xor(best, o, 64);
    const double om = __shfl_xor(bmean, o, 64);
    const int ot = __shfl_xor(bt, o, 64);
    if (ob > best || (ob == best && ot < bt)) {
      best = ob;
      bmean = om;
      bt = ot;
    }
  }
  if (mean_out) *mean_out = bmean;
  if (var_out) *var_out = best;
  return bt < d ? bt : 0;  // no variance is a number (values that are not, or overflow): any serves
}

// The same choice by several wavefronts and mostly in fp32. The fp64 sums above
// run in one fixed order, 2 m dependent additions a coordinate; but they decide
// only where two coordinates' variances come close. So each of P wavefronts
// sums d = v - s and d^2 (s: the value of subsample row 0) over every P-th
// sample row in fp32, and with S and Q the sums over all rows,
// Q/m - (S/m)^2 is within (3m + 16) 2^-24 Q/m of the exact variance whatever
// the order (each d carries one rounding, a sum of m terms at most m, and
// S^2 <= m Q; the fp64 variance's own error is below 2^-40 of it). A coordinate
// whose lower bound is above every other's upper bound is the choice; where
// none is (close calls, ties, constant or non-finite samples), the fp64 sums
// decide. Mean and variance also give the range of the select's bins.
//
// What bounds it: the latency of the sample rows. One wavefront with the fp64
// sums took 12,000 to 17,500 cycles a node at d = 64 and 56,000 at d = 128, most
// of them in dependent fp64 operations; now 4,200 to 8,900 and 14,000.
struct Moments {
  float s0, S, Q;  // the shift, the sum and the sum of squares of v - s0
};

// Wavefront part `part` of P: coordinates lane + 64 h over sample rows part,
// part + P, ...; off[h]: byte offset of sample row lane + 64 h.
// U rows are in flight at a time.
template <int H, int U>
__device__ __forceinline__ void sample_moments(const float* __restrict__ Y, int d, int m,
                                               const uint32_t (&off)[2], int part, int P,
                                               int lane, Moments (&mo)[H]) {
  const char* base = reinterpret_cast<const char*>(Y);
  uint32_t lo[H];
  float S[H][2], Q[H][2];
  const uint32_t o0 = (uint32_t)__builtin_amdgcn_readlane((int)off[0], 0);
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int t = lane + 64 * h;
    lo[h] = 4u * (uint32_t)(t < d ? t : 0);
    mo[h].s0 = *reinterpret_cast<const float*>(base + (o0 + lo[h]));
    S[h][0] = S[h][1] = Q[h][0] = Q[h][1] = 0.f;
  }
  for (int j0 = part; j0 < m; j0 += U * P) {
    float v[U][H];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = min(j0 + u * P, m - 1);
      const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)(j < 64 ? off[0] : off[1]), j & 63);
#pragma unroll
      for (int h = 0; h < H; ++h) v[u][h] = *reinterpret_cast<const float*>(base + (o + lo[h]));
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const float dv = j0 + u * P < m ? v[u][h] - mo[h].s0 : 0.f;
        S[h][u & 1] += dv;
        Q[h][u & 1] = __builtin_fmaf(dv, dv, Q[h][u & 1]);
      }
  }
#pragma unroll
  for (int h = 0; h < H; ++h) {
    mo[h].S = S[h][0] + S[h][1];
    mo[h].Q = Q[h][0] + Q[h][1];
  }
}

// The choice from the moments over all sample rows (one wavefront): the
// coordinate, or -1 where the bounds leave it open; its mean and variance.
template <int H>
__device__ __forceinline__ int choose_by_bounds(const Moments (&mo)[H], int d, int m, int lane,
                                                float* mean, float* var_out) {
  const float inv = 1.f / (float)m, eps = (float)(3 * m + 16) * 0x1p-24f;
  float lo[H], hi[H], var[H], best = -INFINITY;
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const float a = mo[h].S * inv, q = mo[h].Q * inv;
    var[h] = q - a * a;
    const float e = eps * q + 0x1p-110f;  // the second term: squares that underflow
    lo[h] = lane + 64 * h < d ? var[h] - e : -INFINITY;
    hi[h] = var[h] + e;
    best = fmaxf(best, lo[h]);
  }
  best = wave_max(best);
  uint64_t open[H];
  int n = 0;
#pragma unroll
  for (int h = 0; h < H; ++h) {
    open[h] = __ballot(lane + 64 * h < d && !(hi[h] < best));  // NaN stays open
    n += __popcll(open[h]);
  }
  if (n != 1) return -1;
  int t = 0;
  float a = 0.f, v = 0.f;
#pragma unroll
  for (int h = 0; h < H; ++h)
    if (open[h]) {
      const int l = __builtin_ctzll(open[h]);
      t = 64 * h + l;
      a = read_lane(mo[h].s0 + mo[h].S * inv, l);
      v = read_lane(var[h], l);
    }
  *mean = a;
  *var_out = v;
  return t;
}

// The choice where the bounds leave it open (one wavefront): coordinate 0 where
// all sample rows are equal (every variance is exactly zero), else the fp64 sums.
// Squares of differences that underflow also sum to zero, so the rows are
// compared. (The sums, and radix passes over equal keys, made the clustering of
// 40 heads of 75,600 equal tokens at d = 128 take 9.2 ms; now 7.4.)
template <int H, int B>
__device__ __forceinline__ int choose_open(const float* __restrict__ Y, int d,
                                           const int32_t* idx, bool identity, int start, int size,
                                           int m, const Moments (&mo)[H], int lane, float* mean,
                                           float* var) {
  bool flat = true;
#pragma unroll
  for (int h = 0; h < H; ++h) flat = flat && (mo[h].Q == 0.f || lane + 64 * h >= d);
  if (__ballot(!flat) == 0ull) {
    uint32_t off[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int p = start + sample_pos(min(lane + 64 * h, m - 1), size, m);
      off[h] = 4u * (uint32_t)d * (uint32_t)(identity ? p : idx[p]);
    }
    const char* base = reinterpret_cast<const char*>(Y);
    for (int j0 = 0; j0 < m && flat; j0 += 16) {
      float v[16][H];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int j = min(j0 + u, m - 1);
        const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)(j < 64 ? off[0] : off[1]), j & 63);
#pragma unroll
        for (int h = 0; h < H; ++h) {
          const int t = lane + 64 * h;
          v[u][h] = *reinterpret_cast<const float*>(base + (o + 4u * (uint32_t)(t < d ? t : 0)));
        }
      }
#pragma unroll
      for (int u = 0; u < 16; ++u)
#pragma unroll
        for (int h = 0; h < H; ++h) flat = flat && (v[u][h] == mo[h].s0 || lane + 64 * h >= d);
      flat = __ballot(!flat) == 0ull;
    }
    if (flat) {
      *mean = read_lane(mo[0].s0, 0);
      *var = 0.f;
      return 0;
    }
  }
  double dmean, dvar;
  const int js = choose_coordinate<B>(Y, d, idx, identity, start, size, lane, &dmean, &dvar);
  *mean = (float)dmean;
  *var = (float)dvar;
  return js;
}

// Origin and scale of nb linear bins over mean +- 4 sd (scale 0, one bin,
// where there is no spread). Any range serves: bins only narrow the exact
// select down, so hardware reciprocal square roots do.
__device__ __forceinline__ void bin_range(float mean, float var, int nb, float* lo, float* scale) {
  const float rs = __builtin_amdgcn_rsqf(var);  // 1 / sd
  float l = mean - 4.f * (var * rs), s = 0.125f * (float)nb * rs;
  if (!(var > 0.f) || !isfinite(l) || !isfinite(s)) l = s = 0.f;
  *lo = l;
  *scale = s;
}

// Rows of a sample of m that the bins of a multi-block level are laid by (at
// most 64, spread over the sample): the row of lane `lane`.
__device__ __forceinline__ int bin_row(int lane, int m) {
  return m > 64 ? lane * m / 64 : min(lane, m - 1);
}

// Bins of a multi-block level (one wavefront). The threshold is the key of rank
// mL of size; the keys x of those rows (one a lane) bound its place by 2 sqrt(64)
// ranks (four standard deviations) to each side, whatever the distribution. The
// bins lie between two values found by halving, from mean +- 4 sd: with at most
// that many sample keys less and, unless runs of equal keys forbid it, not many
// fewer. Mean -+ sd mostly serves at once; where outliers stretch the deviation or
// the keys lie in clumps, halving goes on. Samples too small for such a bound (m
// below 17) keep mean +- 4 sd.
// Normal keys: about one in 250 is listed, one in 80 with 256 bins over mean +- 4
// sd. Clustering with those and with these: 8 heads of 1,048,576 tokens 11.7 and
// 10.5 ms, of 65,521 tokens 825 and 824 us, the latter's tokens as they are
// (transform none) with one far sample row 1,396 and 1,047.
__device__ __forceinline__ void threshold_bins(float x, int m, int mL, int size, float mean,
                                               float sd, int lane, float* lo, float* scale) {
  const int mm = min(m, 64);
  float a0 = mean - 4.f * sd, b1 = mean + 4.f * sd;
  const float at = (float)mL / (float)size * (float)mm, w = 2.f * sqrtf((float)mm);
  const int c0 = (int)floorf(at - w), c1 = (int)ceilf(at + w), slack = (int)(0.5f * w);
  if (c0 >= 0 && c1 <= mm) {
    float p0 = b1, t0 = mean - sd, p1 = a0, t1 = mean + sd;
    const bool in = lane < mm;
    for (int it = 0; it < 16; ++it) {
      // a0 has at most c0 of the keys below it and p0 more, b1 at least c1 and p1 fewer
      const int n0 = (int)__popcll(__ballot(in && x < t0)), n1 = (int)__popcll(__ballot(in && x < t1));
      const bool done0 = n0 <= c0 && n0 >= c0 - slack, done1 = n1 >= c1 && n1 <= c1 + slack;
      if (n0 <= c0) a0 = t0; else p0 = t0;
      if (n1 >= c1) b1 = t1; else p1 = t1;
      if (done0 && done1) break;
      if (!done0) t0 = 0.5f * (a0 + p0);
      if (!done1) t1 = 0.5f * (b1 + p1);
    }
  }
  float s = (float)kBins / (b1 - a0);
  if (!(sd > 0.f) || !isfinite(a0) || !(s > 0.f) || !isfinite(s)) a0 = s = 0.f;  // one bin
  *lo = a0;
  *scale = s;
}

// Multi-block levels. A node's split threshold is its m_L-th smallest key,
// found exactly in three passes over chunks of its keys:
//   keys:    every chunk block gathers its keys and counts them into kBins
//            linear bins between two keys that the node's sample puts around
//            the threshold (threshold_bins; the clamped linear map is monotone,
//            so each bin is a contiguous key range); the chunk's histogram goes
//            to its own slot.
//   bins:    every chunk block sums the node's histograms, finds the bin that
//            holds the wanted rank, and lists its chunk's keys of that bin
//            (typically one in 250) behind those of the chunks before it.
//   scatter: every chunk block selects exactly among the listed keys, counts
//            those of the chunks before it, and partitions its chunk stably.
// Kernel boundaries order the passes, but for nodes with more than kListed
// listed keys (runs of equal keys at the threshold, or more than about a million
// keys): there the last chunk block of the bins pass to arrive selects for the
// node, since every chunk reading so long a list would cost chunks times keys (16
// heads of 262,144 tokens, 40% of them zero: ca_cluster 11.4 ms so, 6.3 ms with
// the last block; 10% zero: 7.1 and 5.7 ms; 6.4 and 5.8 ms with 4,096 bins).
// Otherwise no pass leaves a node to one workgroup: the histograms are small
// (kBins) and the select is repeated in every block. With 4,096 bins over mean
// +- 4 sd and one workgroup a node for the select (which read all keys of the
// node again), the keys/select/scatter passes of a level took 12.7/19.7/14.8 us on
// average at 8 heads of 65,521 tokens, 48/40/46 us at 40 heads of 75,600, and
// 64/46/52 us at 16 heads of 262,144; now keys/bins/scatter take 11.4/10.1/16.3,
// 43.8/17.4/51.5 and 61.8/20.2/60.7 us (rocprofv3 kernel trace).
//
// Node state (int32): 0 j* (-1: leaf), 1 threshold key (selected) or number of
// listed keys, 2 rank of the threshold among the keys equal to it (selected) or
// among the listed ones, 3 left size, 4 start, 5 size, 6 bin origin (float),
// 7 number of chunks, 8 bin scale (float), 9 rank of the threshold, 10 selected
// with its keys (nodes of one chunk) or in the bins pass, 11 bin of the
// threshold, 12 chunk blocks that have listed their keys.
// Chunk state (int32): 0 keys below the bin and 1 listed keys in the chunks
// before it, 2 and 3 smallest and largest listed key of the chunk; of a node
// selected in the bins pass: 0 keys below and 1 equal to the threshold in the
// chunks before it.
__device__ __forceinline__ int32_t* node_ptr(const Ctx& C, int pid, int node) {
  return C.node_state + ((size_t)pid * C.max_nodes + node) * kNodeInts;
}

__device__ __forceinline__ float key_value(uint32_t key) {
  return __uint_as_float((key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key);
}

// Bin of a key: floor((v - lo) * scale) clamped to [0, nb); infinities and
// NaNs go to the end bin their key order puts them in.
__device__ __forceinline__ int lin_bin(uint32_t key, float lo, float scale, int nb = kBins) {
  if (key >= 0xFF800000u) return nb - 1;  // +inf, positive NaNs
  if (key <= 0x007FFFFFu) return 0;       // -inf, negative NaNs
  float t = (key_value(key) - lo) * scale;
  t = fminf(fmaxf(t, 0.f), (float)(nb - 1));
  return (int)t;
}

constexpr int kPer = kChunk / 256;  // positions per thread in a 256-thread chunk block

// Nodes of more than kGroupedFrom chunks also sum their chunks' histograms by
// groups of kGroup, so that a block of the bins pass reads the groups and the
// chunks of its own group instead of every chunk, whose number grows with the
// square of the node. The bins passes of 4,194,304 tokens (one head, up to 1,024
// chunks) took 1,364 us without, 1,179 with; of 8 heads of 2,097,152 1,989 and
// 1,702.
__device__ __forceinline__ uint32_t* group_hist(const Ctx& C, int cpn, int pid, int node) {
  return C.ghist +
         ((size_t)pid * C.ghist_slots + (size_t)node * ((cpn + kGroup - 1) / kGroup)) * kBins;
}
// Cleared by the kernel that chooses the node's coordinate (its threads all).
__device__ __forceinline__ void clear_group_hist(const Ctx& C, int cpn, int pid, int node) {
  if (cpn <= kGroupedFrom) return;
  uint4* h = reinterpret_cast<uint4*>(group_hist(C, cpn, pid, node));
  const int n = (cpn + kGroup - 1) / kGroup * (kBins / 4);
  for (int i = threadIdx.x; i < n; i += blockDim.x) h[i] = make_uint4(0u, 0u, 0u, 0u);
}

struct LevelArgs {
  int level;
  int first;  // input permutation is the identity
  int cpn;    // chunk slots per node at this level
  const int32_t* idx_in;
  int32_t* idx_out;
};

constexpr int kChooseWaves = 4;

template <int H>
__global__ __launch_bounds__(64 * kChooseWaves) void split_choose_kernel(Ctx C, LevelArgs L) {
  __shared__ float2 part[kChooseWaves][64 * H];
  const int pid = blockIdx.y, side = pid / C.BH, bh = pid % C.BH, node = blockIdx.x;
  const Side& S = C.s[side];
  if (L.level >= S.big) return;
  int start, size;
  node_range(S.n, S.c, L.level, node, &start, &size);
  int32_t* ns = node_ptr(C, pid, node);
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int d = C.d;
  if (size <= S.c) {
    if (threadIdx.x == 0) ns[0] = -1;
    return;
  }
  clear_group_hist(C, L.cpn, pid, node);
  const int32_t* idx = L.idx_in + (size_t)pid * C.nmax;
  const float* Y = S.y + (size_t)bh * S.n * d;
  const int m = size < d ? size : d;
  uint32_t off[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int p = start + sample_pos(min(lane + 64 * h, m - 1), size, m);
    off[h] = 4u * (uint32_t)d * (uint32_t)(L.first ? p : idx[p]);
  }
  Moments mo[H];
  sample_moments<H, 32>(Y, d, m, off, w, kChooseWaves, lane, mo);
#pragma unroll
  for (int h = 0; h < H; ++h) part[w][lane + 64 * h] = make_float2(mo[h].S, mo[h].Q);
  __syncthreads();
  if (w != 0) return;
#pragma unroll
  for (int i = 1; i < kChooseWaves; ++i)
#pragma unroll
    for (int h = 0; h < H; ++h) {
      mo[h].S += part[i][lane + 64 * h].x;
      mo[h].Q += part[i][lane + 64 * h].y;
    }
  float mean, var;
  int js = choose_by_bounds<H>(mo, d, m, lane, &mean, &var);
  if (js < 0) js = choose_open<H, 32>(Y, d, idx, L.first, start, size, m, mo, lane, &mean, &var);
  const int mL = left_size(size, S.c);
  float lo, scale;
  {
    uint32_t o = off[0];
    if (H == 2 && m > 64) {
      const int j = bin_row(lane, m);
      const uint32_t o0 = __shfl(off[0], j & 63, 64), o1 = __shfl(off[1], j & 63, 64);
      o = j < 64 ? o0 : o1;
    }
    const float x = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(Y) +
                                                    (o + 4u * (uint32_t)js));
    const float sd = var * __builtin_amdgcn_rsqf(var);  // NaN where there is no spread
    threshold_bins(x, m, mL, size, mean, sd, lane, &lo, &scale);
  }
  if (lane == 0) {
    ns[0] = js;
    ns[10] = 0;
    ns[12] = 0;
    ns[1] = 0;
    ns[2] = 0;
    ns[3] = mL;
    ns[4] = start;
    ns[5] = size;
    ns[6] = __float_as_int(lo);
    ns[7] = (size + kChunk - 1) / kChunk;
    ns[8] = __float_as_int(scale);
    ns[9] = mL - 1;
  }
}

// ---------------------------------------------------------------------------
// Basic splitting (Method: recursive splitting, basic; a variation of
// principal direction divisive partitioning): the direction of each node at
// one level, by power iteration on its strided subsample. Every reduction
// runs in a fixed order with separately rounded products and sums (no fused
// multiply-add), so the directions, and the splits made on them, are
// reproducible bit for bit.
// ---------------------------------------------------------------------------

__device__ __forceinline__ float div_rn(float a, float b) { return a / b; }
__device__ __forceinline__ float sqrt_rn(float a) { return __builtin_sqrtf(a); }

constexpr int kBasicThreads = 128;
constexpr int kBasicIters = 8;

__device__ __forceinline__ float* dir_ptr(const Ctx& C, int level, int pid, int node) {
  return C.dirs + ((((size_t)(level & 1) * 2 * C.BH) + pid) * C.max_nodes + node) * C.d;
}

// Output number c (counting from 0) of splitmix64 started at state 0
// (S. Vigna's generator).
__device__ __forceinline__ uint64_t splitmix64_at(uint64_t c) {
  uint64_t z = (c + 1ull) * 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

// Approximately standard normal: the sum of 12 uniforms minus 6 (Irwin-Hall),
// uniform u the top 24 bits of output 16 c + u, summed as integers.
__device__ __forceinline__ float irwin_hall(uint64_t c) {
  long long sum = 0;
#pragma unroll
  for (int u = 0; u < 12; ++u) sum += (long long)(splitmix64_at(c * 16ull + (uint64_t)u) >> 40);
  return (float)((double)sum * 0x1p-24 - 6.0);
}

// One block per node of the level. Dynamic LDS: the subsample, m x (d + 1).
// D is the feature count when it is a compile-time constant (64, 128), so the
// in-order chains unroll and their LDS reads are issued ahead; D = 0 reads d
// from the problem. Norms are computed by every thread from the same LDS
// values (identical results), which saves a barrier per iteration.
template <int D>
__global__ __launch_bounds__(kBasicThreads) void basic_choose_kernel(Ctx C, LevelArgs L) {
  extern __shared__ __attribute__((aligned(16))) float bsub[];
  __shared__ float mu[kMaxD], v[kMaxD], t[kMaxD], w[kMaxD];
  const int pid = blockIdx.y, side = pid / C.BH, bh = pid % C.BH, node = blockIdx.x;
  const Side& S = C.s[side];
  if (L.level >= S.big) return;
  int start, size;
  node_range(S.n, S.c, L.level, node, &start, &size);
  int32_t* ns = node_ptr(C, pid, node);
  const int tid = threadIdx.x, d = D ? D : C.d, DP = d + 1;
  if (size <= S.c) {
    if (tid == 0) ns[0] = -1;
    return;
  }
  clear_group_hist(C, L.cpn, pid, node);
  const int m = d < size ? d : size;
  const int32_t* idx = L.idx_in + (size_t)pid * C.nmax;
  const float* Y = S.y + (size_t)bh * S.n * d;
  if (D != 0 && D % 4 == 0) {
    // float4 reads of the sample rows
    const int d4 = d / 4;
    for (int e = tid; e < m * d4; e += kBasicThreads) {
      const int j = e / d4, k4 = e % d4;
      const int p = (int)(((long long)(2 * j + 1) * size) / (2 * m));
      const int row = L.first ? start + p : idx[start + p];
      const float4 x = *(const float4*)(Y + (size_t)row * d + 4 * k4);
      float* dst = bsub + j * DP + 4 * k4;
      dst[0] = x.x;
      dst[1] = x.y;
      dst[2] = x.z;
      dst[3] = x.w;
    }
  } else {
    for (int e = tid; e < m * d; e += kBasicThreads) {
      const int j = e / d, k = e % d;
      const int p = (int)(((long long)(2 * j + 1) * size) / (2 * m));
      const int row = L.first ? start + p : idx[start + p];
      bsub[j * DP + k] = Y[(size_t)row * d + k];
    }
  }
  // warm start noise of this node
  if (tid < d) {
    const uint64_t base = ((((uint64_t)(2 * bh + side) << 5 | (uint64_t)L.level) << 20 |
                            (uint64_t)node) << 7);
    t[tid] = irwin_hall(base | (uint64_t)tid);
  }
  __syncthreads();
  if (tid < d) {
    float a = 0.f;
    for (int j = 0; j < m; ++j) a = add_rn(a, bsub[j * DP + tid]);
    mu[tid] = div_rn(a, (float)m);
  }
  __syncthreads();
  for (int e = tid; e < m * d; e += kBasicThreads) {
    const int j = e / d, k = e % d;
    bsub[j * DP + k] = sub_rn(bsub[j * DP + k], mu[k]);
  }
  // the parent's direction one level up, mixed with the noise
  const float* vp = L.level > 0 ? dir_ptr(C, L.level - 1, pid, node >> 1) : nullptr;
  if (tid < d) {
    float vk = t[tid];
    if (vp) {
      float nv = 0.f, nr = 0.f;
#pragma unroll 16
      for (int k = 0; k < d; ++k) {
        const float pk = vp[k];
        nv = add_rn(nv, mul_rn(pk, pk));
        nr = add_rn(nr, mul_rn(t[k], t[k]));
      }
      const float sc = div_rn(sqrt_rn(nv), sqrt_rn(nr));
      vk = mul_rn(add_rn(vp[tid], mul_rn(vk, sc)), 0.5f);
    }
    v[tid] = vk;
  }
  for (int it = 0; it < kBasicIters; ++it) {
    __syncthreads();
    if (tid < m) {
      float a = 0.f;
#pragma unroll 16
      for (int k = 0; k < d; ++k) a = add_rn(a, mul_rn(bsub[tid * DP + k], v[k]));
      t[tid] = a;
    }
    __syncthreads();
    if (tid < d) {
      float a = 0.f;
#pragma unroll 16
      for (int j = 0; j < m; ++j) a = add_rn(a, mul_rn(t[j], bsub[j * DP + tid]));
      w[tid] = a;
    }
    __syncthreads();
    if (tid < d) {
      float nn = 0.f;
#pragma unroll 16
      for (int k = 0; k < d; ++k) nn = add_rn(nn, mul_rn(w[k], w[k]));
      if (nn > 0.f) v[tid] = div_rn(w[tid], sqrt_rn(nn));
    }
  }
  __syncthreads();
  float* vo = dir_ptr(C, L.level, pid, node);
  if (tid < d) vo[tid] = v[tid];
  // spread of the subsample's projections, for the linear bins of the select
  if (tid < m) {
    float a = 0.f;
#pragma unroll 16
    for (int k = 0; k < d; ++k) a = add_rn(a, mul_rn(bsub[tid * DP + k], v[k]));
    t[tid] = a;
  }
  __syncthreads();
  if (tid >= 64) return;
  double mp = 0.0, vv = 0.0;
  for (int k = 0; k < d; ++k) mp += (double)mu[k] * (double)v[k];
  for (int j = 0; j < m; ++j) vv += (double)t[j] * (double)t[j];
  const int mL = left_size(size, S.c);
  float lo, scale;
  threshold_bins((float)(mp + (double)t[bin_row(tid, m)]), m, mL, size, (float)mp,
                 (float)sqrt(vv / m), tid, &lo, &scale);
  if (tid == 0) {
    ns[0] = 0;
    ns[1] = 0;
    ns[2] = 0;
    ns[3] = mL;
    ns[10] = 0;
    ns[12] = 0;
    ns[4] = start;
    ns[5] = size;
    ns[6] = __float_as_int(lo);
    ns[7] = (size + kChunk - 1) / kChunk;
    ns[8] = __float_as_int(scale);
    ns[9] = mL - 1;
  }
}

// d = 64: one wavefront per node. Lane j holds sample row j and lane k holds
// coordinate k of every sample row (the sample column), both read straight
// from HBM, so each in-order chain runs on registers and 16-byte broadcast
// reads of one LDS vector (v, t or w). Same operations, in the same order, as
// basic_choose_kernel.
__global__ __launch_bounds__(64) void basic_choose64_kernel(Ctx C, LevelArgs L) {
  constexpr int D = 64;
  __shared__ __attribute__((aligned(16))) float mu[D], v[D], t[D], w[D];
  const int pid = blockIdx.y, side = pid / C.BH, bh = pid % C.BH, node = blockIdx.x;
  const Side& S = C.s[side];
  if (L.level >= S.big) return;
  int start, size;
  node_range(S.n, S.c, L.level, node, &start, &size);
  int32_t* ns = node_ptr(C, pid, node);
  const int lane = threadIdx.x;
  if (size <= S.c) {
    if (lane == 0) ns[0] = -1;
    return;
  }
  clear_group_hist(C, L.cpn, pid, node);
  const int m = D < size ? D : size;
  const int32_t* idx = L.idx_in + (size_t)pid * C.nmax;
  const float* Y = S.y + (size_t)bh * S.n * D;
  int myrow = L.first ? start : idx[start];
  if (lane < m) {
    const int p = (int)(((long long)(2 * lane + 1) * size) / (2 * m));
    myrow = L.first ? start + p : idx[start + p];
  }
  float row[D], col[D];
  {
    const float4* src = (const float4*)(Y + (size_t)myrow * D);
#pragma unroll
    for (int k4 = 0; k4 < D / 4; ++k4) {
      const float4 x = src[k4];
      row[4 * k4] = x.x;
      row[4 * k4 + 1] = x.y;
      row[4 * k4 + 2] = x.z;
      row[4 * k4 + 3] = x.w;
    }
  }
  // Entries past the m sample rows are held at exactly zero, so every chain
  // can run over all D terms without branches: a sum that starts at +0 never
  // becomes -0 in round-to-nearest, so adding a zero product leaves it as is.
  uint32_t keep[D / 32];
#pragma unroll
  for (int h = 0; h < D / 32; ++h)
    keep[h] = m >= 32 * (h + 1) ? 0xFFFFFFFFu : (m <= 32 * h ? 0u : (1u << (m - 32 * h)) - 1u);
  auto kept = [&](float x, int j) {
    return __uint_as_float(__float_as_uint(x) & (0u - ((keep[j >> 5] >> (j & 31)) & 1u)));
  };
#pragma unroll
  for (int j = 0; j < D; ++j) {
    const int rj = __builtin_amdgcn_readlane(myrow, j);
    col[j] = kept(Y[(size_t)rj * D + lane], j);
  }
  float a = 0.f;
#pragma unroll
  for (int j = 0; j < D; ++j) a = add_rn(a, col[j]);
  const float muk = div_rn(a, (float)m);
  mu[lane] = muk;
#pragma unroll
  for (int j = 0; j < D; ++j) col[j] = kept(sub_rn(col[j], muk), j);
  const uint64_t base = ((((uint64_t)(2 * bh + side) << 5 | (uint64_t)L.level) << 20 |
                          (uint64_t)node) << 7);
  const float noise = irwin_hall(base | (uint64_t)lane);
  t[lane] = noise;
  __syncthreads();
#pragma unroll
  for (int k4 = 0; k4 < D / 4; ++k4) {
    const float4 u = *(const float4*)(mu + 4 * k4);
    row[4 * k4] = sub_rn(row[4 * k4], u.x);
    row[4 * k4 + 1] = sub_rn(row[4 * k4 + 1], u.y);
    row[4 * k4 + 2] = sub_rn(row[4 * k4 + 2], u.z);
    row[4 * k4 + 3] = sub_rn(row[4 * k4 + 3], u.w);
  }
  // warm start: the parent's direction one level up, mixed with the noise
  float vk = noise;
  if (L.level > 0) {
    const float* vp = dir_ptr(C, L.level - 1, pid, node >> 1);
    float nv = 0.f, nr = 0.f;
#pragma unroll
    for (int k4 = 0; k4 < D / 4; ++k4) {
      const float4 pv = *(const float4*)(vp + 4 * k4);
      const float4 r4 = *(const float4*)(t + 4 * k4);
      nv = add_rn(nv, mul_rn(pv.x, pv.x));
      nr = add_rn(nr, mul_rn(r4.x, r4.x));
      nv = add_rn(nv, mul_rn(pv.y, pv.y));
      nr = add_rn(nr, mul_rn(r4.y, r4.y));
      nv = add_rn(nv, mul_rn(pv.z, pv.z));
      nr = add_rn(nr, mul_rn(r4.z, r4.z));
      nv = add_rn(nv, mul_rn(pv.w, pv.w));
      nr = add_rn(nr, mul_rn(r4.w, r4.w));
    }
    const float sc = div_rn(sqrt_rn(nv), sqrt_rn(nr));
    vk = mul_rn(add_rn(vp[lane], mul_rn(noise, sc)), 0.5f);
  }
  __syncthreads();
  v[lane] = vk;
  for (int it = 0; it < kBasicIters; ++it) {
    __syncthreads();
    float ta = 0.f;
#pragma unroll
    for (int k4 = 0; k4 < D / 4; ++k4) {
      const float4 q = *(const float4*)(v + 4 * k4);
      ta = add_rn(ta, mul_rn(row[4 * k4], q.x));
      ta = add_rn(ta, mul_rn(row[4 * k4 + 1], q.y));
      ta = add_rn(ta, mul_rn(row[4 * k4 + 2], q.z));
      ta = add_rn(ta, mul_rn(row[4 * k4 + 3], q.w));
    }
    t[lane] = lane < m ? ta : 0.f;
    __syncthreads();
    float wa = 0.f;
#pragma unroll
    for (int j4 = 0; j4 < D / 4; ++j4) {
      const float4 q = *(const float4*)(t + 4 * j4);
      wa = add_rn(wa, mul_rn(q.x, col[4 * j4]));
      wa = add_rn(wa, mul_rn(q.y, col[4 * j4 + 1]));
      wa = add_rn(wa, mul_rn(q.z, col[4 * j4 + 2]));
      wa = add_rn(wa, mul_rn(q.w, col[4 * j4 + 3]));
    }
    w[lane] = wa;
    __syncthreads();
    float nn = 0.f;
#pragma unroll
    for (int k4 = 0; k4 < D / 4; ++k4) {
      const float4 q = *(const float4*)(w + 4 * k4);
      nn = add_rn(nn, mul_rn(q.x, q.x));
      nn = add_rn(nn, mul_rn(q.y, q.y));
      nn = add_rn(nn, mul_rn(q.z, q.z));
      nn = add_rn(nn, mul_rn(q.w, q.w));
    }
    if (nn > 0.f) v[lane] = div_rn(wa, sqrt_rn(nn));
  }
  __syncthreads();
  dir_ptr(C, L.level, pid, node)[lane] = v[lane];
  // spread of the subsample's projections, for the linear bins of the select
  float ta = 0.f;
#pragma unroll
  for (int k4 = 0; k4 < D / 4; ++k4) {
    const float4 q = *(const float4*)(v + 4 * k4);
    ta = add_rn(ta, mul_rn(row[4 * k4], q.x));
    ta = add_rn(ta, mul_rn(row[4 * k4 + 1], q.y));
    ta = add_rn(ta, mul_rn(row[4 * k4 + 2], q.z));
    ta = add_rn(ta, mul_rn(row[4 * k4 + 3], q.w));
  }
  t[lane] = ta;
  __syncthreads();
  double mp = 0.0, vv = 0.0;
  for (int k = 0; k < D; ++k) mp += (double)mu[k] * (double)v[k];
  for (int j = 0; j < m; ++j) vv += (double)t[j] * (double)t[j];
  const int mL = left_size(size, S.c);
  float lo, scale;
  threshold_bins((float)(mp + (double)ta), m, mL, size, (float)mp, (float)sqrt(vv / m), lane, &lo,
                 &scale);
  if (lane == 0) {
    ns[0] = 0;
    ns[1] = 0;
    ns[2] = 0;
    ns[3] = mL;
    ns[4] = start;
    ns[5] = size;
    ns[6] = __float_as_int(lo);
    ns[7] = (size + kChunk - 1) / kChunk;
    ns[8] = __float_as_int(scale);
    ns[9] = mL - 1;
    ns[10] = 0;
    ns[12] = 0;
  }
}

// The order after the last split level, copied to perm (basic splitting runs
// every level with the multi-block kernels, so no tail pass is needed).
__global__ __launch_bounds__(256) void copy_order_kernel(Ctx C, int parity0, int parity1) {
  const int pid = blockIdx.y, side = pid / C.BH, bh = pid % C.BH;
  const Side& S = C.s[side];
  const int32_t* src = ((side == 0 ? parity0 : parity1) ? C.idx1 : C.idx0) + (size_t)pid * C.nmax;
  int32_t* perm = S.perm + (size_t)bh * S.n;
  const bool identity = S.big == 0;
  for (int o = blockIdx.x * 256 + threadIdx.x; o < S.n; o += gridDim.x * 256)
    perm[o] = identity ? o : src[o];
}

// T_K = F_q and T_Q = F_k (basic splitting in the metric root space), and
// for the MFMA projection their transposed hi/lo bf16 operands: W_Q^T is the
// operand the Cholesky pass already packed for F_k, W_K^T is packed here.
__global__ __launch_bounds__(256) void copy_roots_kernel(Ctx C, int pack) {
  const int bh = blockIdx.x, d = C.d, dd = d * d;
  const float* Fq = mat(C, bh, M_E0);
  for (int e = threadIdx.x; e < dd; e += 256) {
    mat(C, bh, M_TK)[e] = Fq[e];
    mat(C, bh, M_TQ)[e] = mat(C, bh, M_EK)[e];
  }
  if (!pack) return;
  bf16* tk = wop(C, bh, O_TK);
  bf16* tq = wop(C, bh, O_TQ);
  const bf16* fk = wop(C, bh, O_FK);
  for (int e = threadIdx.x; e < dd; e += 256) {
    const int i = e / d, k = e % d;  // row i = output dim, column k = input dim
    const float w = Fq[k * d + i];
    const bf16 hi = (bf16)w;
    tk[e] = hi;
    tk[dd + e] = (bf16)(w - (float)hi);
    tq[e] = fk[e];
    tq[dd + e] = fk[dd + e];
  }
}

// Block-wide exclusive scan (NT threads).
template <int NT>
__device__ __forceinline__ int block_scan(int x, int* wsum, int* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int v = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(v, o, 64);
    if (lane >= o) v += y;
  }
  if (lane == 63) wsum[w] = v;
  __syncthreads();
  int base = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) {
    const int ws = wsum[i];
    base += i < w ? ws : 0;
    tot += ws;
  }
  __syncthreads();
  *total = tot;
  return base + v - x;
}

__device__ __forceinline__ int scan256(int x, int* wsum, int* total) {
  return block_scan<256>(x, wsum, total);
}

// Keys of one chunk and its linear-bin histogram.
// Projection keys of a thread's kPer rows on the direction dv (LDS): each row
// is read whole with 16-byte loads, R rows at a time (two at d = 64, one at
// d = 128 to bound registers), and its coordinates are summed in order with
// separately rounded products.
template <int D>
__device__ __forceinline__ void basic_keys(const float* __restrict__ Y, const int (&rows)[kPer],
                                           const float* dv, int nu, uint32_t (&kv)[kPer]) {
  constexpr int D4 = D / 4, R = D <= 64 ? 2 : 1;
#pragma unroll
  for (int u = 0; u < kPer; u += R) {
    if (u >= nu) break;  // block-uniform: no position of the chunk is left
    float4 x[R][D4];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float4* src = (const float4*)(Y + (size_t)rows[u + r] * D);
#pragma unroll
      for (int k = 0; k < D4; ++k) x[r][k] = src[k];
    }
    float a[R];
#pragma unroll
    for (int r = 0; r < R; ++r) a[r] = 0.f;
#pragma unroll
    for (int k = 0; k < D4; ++k) {
      const float4 w = *(const float4*)(dv + 4 * k);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        a[r] = add_rn(a[r], mul_rn(x[r][k].x, w.x));
        a[r] = add_rn(a[r], mul_rn(x[r][k].y, w.y));
        a[r] = add_rn(a[r], mul_rn(x[r][k].z, w.z));
        a[r] = add_rn(a[r], mul_rn(x[r][k].w, w.w));
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) kv[u + r] = ordered_bits(a[r]);
  }
}

// BD < 0: keys are the chosen coordinate (diagonalized splitting); BD >= 0:
// projections on the node's direction (basic splitting), BD = d when it is
// 64 or 128, else 0.
template <int BD>
__global__ __launch_bounds__(256) void split_keys_kernel(Ctx C, LevelArgs L) {
  __shared__ int lh[kBins];
  const int pid = blockIdx.z, side = pid / C.BH, bh = pid % C.BH, node = blockIdx.y;
  const Side& S = C.s[side];
  if (L.level >= S.big) return;
  int32_t* ns = node_ptr(C, pid, node);
  const int js = ns[0];
  if (js < 0) return;
  const int start = ns[4], size = ns[5];
  const float lo = __int_as_float(ns[6]), scale = __int_as_float(ns[8]);
  const int c0 = blockIdx.x * kChunk;
  if (c0 >= size) return;
  const int c1 = min(size, c0 + kChunk);
  for (int b = threadIdx.x; b < kBins; b += 256) lh[b] = 0;
  const float* Y = S.y + (size_t)bh * S.n * C.d;
  const int32_t* idx = L.idx_in + (size_t)pid * C.nmax;
  uint32_t* keys = C.keys + (size_t)pid * C.nmax;
  // All of a thread's loads are issued before any is used.
  int rows[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int o = c0 + threadIdx.x + 256 * u;
    rows[u] = o < c1 ? (L.first ? start + o : idx[start + o]) : 0;
  }
  uint32_t kv[kPer];
  if constexpr (BD >= 0) {
    // projection on the node's direction, coordinates summed in order
    __shared__ __attribute__((aligned(16))) float dv[kMaxD];
    const float* dir = dir_ptr(C, L.level, pid, node);
    for (int k = threadIdx.x; k < C.d; k += 256) dv[k] = dir[k];
    __syncthreads();
    if constexpr (BD > 0)
      basic_keys<BD>(Y, rows, dv, (c1 - c0 + 255) / 256, kv);
    else
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const float* yr = Y + (size_t)rows[u] * C.d;
        float a = 0.f;
        for (int k = 0; k < C.d; ++k) a = add_rn(a, mul_rn(yr[k], dv[k]));
        kv[u] = ordered_bits(a);
      }
  } else if (S.ycol && js < kColCopy) {
    // the node's coordinate from its contiguous column: the nodes of a level
    // share few columns, so the lines they read are mostly used in full
    const float* col = S.ycol + ((size_t)bh * kColCopy + js) * S.n;
#pragma unroll
    for (int u = 0; u < kPer; ++u) kv[u] = ordered_bits(col[rows[u]]);
  } else {
#pragma unroll
    for (int u = 0; u < kPer; ++u) kv[u] = ordered_bits(Y[(size_t)rows[u] * C.d + js]);
  }
  {
    if (size <= kChunk) {
      // The whole node is in this block: exact select of the rank-th key here
      // (four 8-bit digits, high first), and no histogram for the select pass.
      __shared__ int rh[256];
      __shared__ int sh_digit, sh_rank;
      const int tid = threadIdx.x, lane = tid & 63;
      uint32_t thr = 0u;
      int r = ns[9];
      for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        rh[tid] = 0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
          const int o = tid + 256 * u;
          if (o < c1 && (pass == 0 || (kv[u] >> (shift + 8)) == (thr >> (shift + 8))))
            atomicAdd(&rh[(kv[u] >> shift) & 255u], 1);
        }
        __syncthreads();
        if (tid < 64) {
          int cnt[4], sum = 0;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            cnt[i] = rh[4 * tid + i];
            sum += cnt[i];
          }
          int incl = sum;
#pragma unroll
          for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
          }
          int acc = incl - sum;
          if (r >= acc && r < incl) {
            for (int i = 0; i < 4; ++i) {
              if (r < acc + cnt[i]) {
                sh_digit = 4 * tid + i;
                sh_rank = r - acc;
                break;
              }
              acc += cnt[i];
            }
          }
        }
        __syncthreads();
        thr |= (uint32_t)sh_digit << shift;
        r = sh_rank;
      }
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int o = tid + 256 * u;
        if (o < c1) keys[start + o] = kv[u];
      }
      if (tid == 0) {
        ns[1] = (int)thr;
        ns[2] = r;
        ns[10] = 1;  // selected
      }
      return;
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int o = c0 + threadIdx.x + 256 * u;
    if (o < c1) {
      keys[start + o] = kv[u];
      atomicAdd(&lh[lin_bin(kv[u], lo, scale)], 1);
    }
  }
  __syncthreads();
  static_assert(kBins == 256, "one bin a thread");
  C.hist[((size_t)pid * C.hist_slots + (size_t)node * L.cpn + blockIdx.x) * kBins + threadIdx.x] =
      (uint32_t)lh[threadIdx.x];
  if (L.cpn > kGroupedFrom && lh[threadIdx.x] != 0)
    atomicAdd(&group_hist(C, L.cpn, pid, node)[(blockIdx.x / kGroup) * kBins + threadIdx.x],
              (uint32_t)lh[threadIdx.x]);
}

// Listed keys up to which every chunk block of a node selects for itself
// (16 a thread, in registers).
constexpr int kListed = 16 * 256;

// Exact select of a node with more than kListed listed keys, by one workgroup:
// whether the threshold is the most frequent of 64 of them (a run of equal
// keys), else 8-bit radix passes after the leading bytes that the smallest and
// the largest listed key share; and the numbers of keys below and equal to the
// threshold in the chunks before each.
struct NodeSelect {
  int hist[256];
  int wsum[4];
  uint32_t kmin, kmax;
  int digit, rank, lt, eq;
};
__device__ __forceinline__ void node_select(int32_t* ns, const uint32_t* cand, int32_t* cc, int n,
                                            int nch, int rank, NodeSelect& sh) {
  const int tid = threadIdx.x, lane = tid & 63;
  // Keys below and equal to thr in each chunk and in all. Chunks w, w + 4, ...
  // are wavefront w's: a lane for a chunk of at most 64 listed keys, then the
  // wavefront together for each of the others. (With a wavefront for every chunk
  // the bins pass of a node of 1,024 chunks with a dozen listed keys each took
  // 540 us; now 245.)
  auto count = [&](uint32_t thr) {
    if (tid == 0) sh.lt = sh.eq = 0;
    __syncthreads();
    for (int g0 = tid >> 6; g0 < nch; g0 += 256) {
      const int g = g0 + 4 * lane;
      int i0 = 0, i1 = 0, lt = 0, eq = 0;
      if (g < nch) {
        i0 = cc[kChunkInts * g + 1];
        i1 = g + 1 < nch ? cc[kChunkInts * (g + 1) + 1] : n;
      }
      const int len = i1 - i0;
      for (int i = 0; i < 64; i += 8) {
        const bool in = len <= 64 && i < len;
        if (__ballot(in) == 0ull) break;
        if (in) {
          uint32_t k[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) k[u] = cand[i0 + min(i + u, len - 1)];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            lt += i + u < len && k[u] < thr;
            eq += i + u < len && k[u] == thr;
          }
        }
      }
      for (uint64_t m = __ballot(len > 64); m != 0ull; m &= m - 1ull) {
        const int l = __builtin_ctzll(m);
        const int j0 = __builtin_amdgcn_readlane(i0, l), j1 = __builtin_amdgcn_readlane(i1, l);
        int wlt = 0, weq = 0;
        for (int i = j0 + lane; i - lane < j1; i += 64 * 16) {
          uint32_t k[16];
#pragma unroll
          for (int u = 0; u < 16; ++u) k[u] = i + 64 * u < j1 ? cand[i + 64 * u] : 0xFFFFFFFFu;
#pragma unroll
          for (int u = 0; u < 16; ++u) {
            wlt += i + 64 * u < j1 && k[u] < thr;
            weq += i + 64 * u < j1 && k[u] == thr;
          }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
          wlt += __shfl_xor(wlt, o, 64);
          weq += __shfl_xor(weq, o, 64);
        }
        if (lane == l) {
          lt = wlt;
          eq = weq;
        }
      }
      if (g < nch) {
        cc[kChunkInts * g + 2] = lt;
        cc[kChunkInts * g + 3] = eq;
        atomicAdd(&sh.lt, lt);
        atomicAdd(&sh.eq, eq);
      }
    }
    __syncthreads();
  };
  if (tid == 0) {
    sh.kmin = 0xFFFFFFFFu;
    sh.kmax = 0u;
  }
  __syncthreads();
  for (int i = tid; i < nch; i += 256) {
    atomicMin(&sh.kmin, (uint32_t)cc[kChunkInts * i + 2]);
    atomicMax(&sh.kmax, (uint32_t)cc[kChunkInts * i + 3]);
  }
  __syncthreads();
  const uint32_t kmin = sh.kmin, diff = sh.kmin ^ sh.kmax;
  uint32_t thr;
  {
    const uint32_t key = cand[(size_t)n * lane / 64];
    int same = 0;
    for (int j = 0; j < 64; ++j)
      same += (uint32_t)__builtin_amdgcn_readlane((int)key, j) == key;
    const int most = wave_max(same);
    thr = (uint32_t)__builtin_amdgcn_readlane((int)key, __builtin_ctzll(__ballot(same == most)));
    sh.lt = sh.eq = 0;
    if (most > 1) count(thr);  // the same in all wavefronts
  }
  __syncthreads();
  if (rank >= sh.lt && rank < sh.lt + sh.eq) {
    rank -= sh.lt;
  } else {
    const int skip = __builtin_clz(diff | 1u) / 8;  // common leading bytes
    thr = skip == 0 ? 0u : kmin & (0xFFFFFFFFu << (32 - 8 * skip));
    for (int shift = 24 - 8 * skip; shift >= 0; shift -= 8) {
      sh.hist[tid] = 0;
      __syncthreads();
      for (int i = tid; i - tid < n; i += 256 * 16) {
        uint32_t k[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) k[u] = i + 256 * u < n ? cand[i + 256 * u] : 0u;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          const bool in = i + 256 * u < n &&
                          (shift == 24 || (k[u] >> (shift + 8)) == (thr >> (shift + 8)));
          const uint64_t m = __ballot(in);
          if (!m) continue;
          // one addition for the lanes that share the first one's digit
          const int dg = (int)(k[u] >> shift) & 255;
          const int first = __builtin_ctzll(m), d0 = __builtin_amdgcn_readlane(dg, first);
          const uint64_t eq = __ballot(in && dg == d0);
          if (lane == first) atomicAdd(&sh.hist[d0], __popcll(eq));
          else if (in && dg != d0) atomicAdd(&sh.hist[dg], 1);
        }
      }
      __syncthreads();
      const int c = sh.hist[tid];
      int tot;
      const int before = scan256(c, sh.wsum, &tot);
      if (rank >= before && rank < before + c) {
        sh.digit = tid;
        sh.rank = rank - before;
      }
      __syncthreads();
      thr |= (uint32_t)sh.digit << shift;
      rank = sh.rank;
    }
    count(thr);
  }
  // of the chunks before each
  int lt0 = 0, eq0 = 0;
  for (int g0 = 0; g0 < nch; g0 += 256) {
    const int g = g0 + tid;
    const int lt = g < nch ? cc[kChunkInts * g + 2] : 0;
    const int eq = g < nch ? cc[kChunkInts * g + 3] : 0;
    int ltall, eqall;
    const int ltb = scan256(lt, sh.wsum, &ltall), eqb = scan256(eq, sh.wsum, &eqall);
    if (g < nch) {
      cc[kChunkInts * g] += lt0 + ltb;
      cc[kChunkInts * g + 1] = eq0 + eqb;
    }
    lt0 += ltall;
    eq0 += eqall;
  }
  if (tid == 0) {
    ns[1] = (int)thr;
    ns[2] = rank;
    ns[10] = 1;
  }
}

__global__ __launch_bounds__(256) void split_bins_kernel(Ctx C, LevelArgs L) {
  __shared__ NodeSelect sel;
  __shared__ int wsum[4];
  __shared__ int sh_last;
  __shared__ int sh_bin, sh_before, sh_base, sh_n, sh_cnt, sh_below;
  __shared__ uint32_t sh_min, sh_max;
  const int pid = blockIdx.z, node = blockIdx.y, side = pid / C.BH, ch = blockIdx.x;
  const Side& S = C.s[side];
  if (L.level >= S.big) return;
  int32_t* ns = node_ptr(C, pid, node);
  if (ns[0] < 0 || ns[10]) return;  // a leaf, or selected with its keys
  const int start = ns[4], size = ns[5], nch = ns[7];
  const float lo = __int_as_float(ns[6]), scale = __int_as_float(ns[8]);
  const int c0 = ch * kChunk;
  if (c0 >= size) return;
  const int c1 = min(size, c0 + kChunk);
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t* keys = C.keys + (size_t)pid * C.nmax + start;
  uint32_t kv[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int o = c0 + tid + 256 * u;
    kv[u] = o < c1 ? keys[o] : 0u;
  }
  // bin tid of the node, and of the chunks before this one
  const uint32_t* H = C.hist + ((size_t)pid * C.hist_slots + (size_t)node * L.cpn) * kBins + tid;
  int tot = 0, pre = 0;
  // adds h[0 .. n) to tot, and of them h[0 .. before) to pre
  auto add = [&](const uint32_t* h, int n, int before) __attribute__((always_inline)) {
    for (int g = 0; g < n; g += 16) {
      int hv[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) hv[u] = g + u < n ? (int)h[(size_t)(g + u) * kBins] : 0;
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        tot += hv[u];
        pre += g + u < before ? hv[u] : 0;
      }
    }
  };
  if (L.cpn <= kGroupedFrom) {
    add(H, nch, ch);
  } else {
    const int g0 = ch / kGroup * kGroup;  // the first chunk of this one's group
    add(H + (size_t)g0 * kBins, ch - g0, ch - g0);
    tot = 0;
    add(group_hist(C, L.cpn, pid, node) + tid, (nch + kGroup - 1) / kGroup, ch / kGroup);
  }
  if (tid == 0) {
    sh_cnt = 0;
    sh_below = 0;
    sh_min = 0xFFFFFFFFu;
    sh_max = 0u;
  }
  int all;
  const int before = scan256(tot, wsum, &all);
  const int rank = ns[9];
  if (rank >= before && rank < before + tot) {
    sh_bin = tid;
    sh_before = before;
    sh_base = pre;
    sh_n = tot;
  }
  __syncthreads();
  const int bin = sh_bin, base = sh_base;
  int below = tid < bin ? pre : 0;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) below += __shfl_xor(below, o, 64);
  if (lane == 0) atomicAdd(&sh_below, below);
  uint32_t* cand = C.cand + (size_t)pid * C.nmax + start;
  uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int o = c0 + tid + 256 * u;
    const bool in = o < c1 && lin_bin(kv[u], lo, scale) == bin;
    const uint64_t m = __ballot(in);
    if (!m) continue;
    // (the order inside a chunk is not used)
    int at = 0;
    if (lane == 0) at = atomicAdd(&sh_cnt, __popcll(m));
    at = __builtin_amdgcn_readfirstlane(at);
    if (in) {
      const int i = base + at + __popcll(m & ((1ull << lane) - 1ull));
      if (i < size) cand[i] = kv[u];
      kmin = min(kmin, kv[u]);
      kmax = max(kmax, kv[u]);
    }
  }
  if (kmin <= kmax) {
    atomicMin(&sh_min, kmin);
    atomicMax(&sh_max, kmax);
  }
  __syncthreads();
  int32_t* cc = C.chunk_cnt + ((size_t)pid * C.hist_slots + (size_t)node * L.cpn) * kChunkInts;
  const int n = sh_n;
  if (tid == 0) {
    cc[kChunkInts * ch] = sh_below;
    cc[kChunkInts * ch + 1] = base;
    cc[kChunkInts * ch + 2] = (int32_t)sh_min;
    cc[kChunkInts * ch + 3] = (int32_t)sh_max;
  }
  if (n <= kListed) {
    if (tid == 0 && ch == 0) {
      ns[1] = n;
      ns[2] = rank - sh_before;
      ns[11] = bin;
    }
    return;
  }
  // The same branch in all blocks of the node. The lists and chunk states are
  // released before this block's arrival is counted; the block that finds all
  // others arrived acquires them. No block waits for another.
  __threadfence();
  __syncthreads();
  if (tid == 0) sh_last = atomicAdd(&ns[12], 1) == nch - 1;
  __syncthreads();
  if (!sh_last) return;
  __threadfence();
  node_select(ns, cand, cc, n, nch, rank - sh_before, sel);
}

// Stable partition of every node: the m_L smallest (key, position) pairs go
// left in node order, the rest right in node order. Nodes that are already
// leaves are copied.
// LDS slot of position i of a chunk: one pad word per 16, so that the
// 16-position runs of consecutive threads start on different banks.
__device__ __forceinline__ int scat_slot(int i) { return i + (i >> 4); }

// Exact select among a node's at most kListed listed keys (the rank-th smallest)
// by one chunk block: their bin is cut into 256 again, and the rank found by
// counting among the at most 64 keys of its part, or, with more of them there
// (ties, an end bin), by 8-bit radix passes. Gives the threshold, the number of
// keys equal to it that go left (less one), and the numbers of keys below and
// equal to it in the chunks before this one.
struct ChunkSelect {
  int hist[256];
  int wsum[4];
  uint32_t list[64];
  int digit, rank, less, eq, nlist;
};
__device__ __forceinline__ void chunk_select(const Ctx& C, int pid, const int32_t* ns, int slot0,
                                             ChunkSelect& sh, uint32_t* thr_out, int* need_eq,
                                             int* less0, int* eq0) {
  constexpr int R = kListed / 256;  // keys per thread
  const int tid = threadIdx.x, lane = tid & 63, ch = blockIdx.x;
  const int n = ns[1], start = ns[4], bin = ns[11];
  const float lo = __int_as_float(ns[6]), scale = __int_as_float(ns[8]);
  int rank = ns[2];
  const uint32_t* cand = C.cand + (size_t)pid * C.nmax + start;
  const int32_t* cc = C.chunk_cnt + ((size_t)pid * C.hist_slots + slot0 + ch) * kChunkInts;
  uint32_t kr[R];
#pragma unroll
  for (int u = 0; u < R; ++u) {
    const int i = tid + 256 * u;
    kr[u] = i < n ? cand[i] : 0u;
  }
  const int base = cc[1];
  if (tid == 0) {
    sh.less = cc[0];
    sh.eq = 0;
    sh.nlist = 0;
  }
  sh.hist[tid] = 0;
  __syncthreads();
  // f(key, i) over the listed keys
  auto each = [&](auto&& f) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < R; ++u)
      if (256 * u < n) {  // uniform
        if (tid + 256 * u < n) f(kr[u], tid + 256 * u);
      }
  };
  // digit of the rank in hist (one entry a thread), the rank inside it
  auto find = [&]() __attribute__((always_inline)) {
    const int c = sh.hist[tid];
    int tot;
    const int before = scan256(c, sh.wsum, &tot);
    if (rank >= before && rank < before + c) {
      sh.digit = tid;
      sh.rank = rank - before;
    }
    __syncthreads();
    return sh.digit;
  };
  auto part_of = [&](uint32_t key) {
    if (key >= 0xFF800000u) return 255;  // +inf, positive NaNs
    if (key <= 0x007FFFFFu) return 0;    // -inf, negative NaNs
    const float t = ((key_value(key) - lo) * scale - (float)bin) * 256.f;
    return (int)fminf(fmaxf(t, 0.f), 255.f);
  };
  each([&](uint32_t key, int) { atomicAdd(&sh.hist[part_of(key)], 1); });
  __syncthreads();
  const int part = find();
  const int want = sh.rank;
  each([&](uint32_t key, int) {
    if (part_of(key) != part) return;
    const int i = atomicAdd(&sh.nlist, 1);
    if (i < 64) sh.list[i] = key;
  });
  __syncthreads();
  uint32_t thr = 0u;
  const int nl = __builtin_amdgcn_readfirstlane(sh.nlist);
  if (nl <= 64) {  // the same in every wavefront
    const uint32_t key = lane < nl ? sh.list[lane] : 0xFFFFFFFFu;
    int less = 0, eq = 0;
    for (int j = 0; j < nl; ++j) {
      const uint32_t kj = (uint32_t)__builtin_amdgcn_readlane((int)key, j);
      less += kj < key;
      eq += kj == key;
    }
    const uint64_t own = __ballot(lane < nl && want >= less && want < less + eq);
    const int l = own ? __builtin_ctzll(own) : 0;
    thr = (uint32_t)__builtin_amdgcn_readlane((int)key, l);
    rank = want - __builtin_amdgcn_readlane(less, l);
  } else {
    for (int shift = 24; shift >= 0; shift -= 8) {
      sh.hist[tid] = 0;
      __syncthreads();
      each([&](uint32_t key, int) {
        if (shift == 24 || (key >> (shift + 8)) == (thr >> (shift + 8)))
          atomicAdd(&sh.hist[(key >> shift) & 255u], 1);
      });
      __syncthreads();
      thr |= (uint32_t)find() << shift;
      rank = sh.rank;
    }
  }
  // the listed keys of the chunks before this one
  int lt = 0, eq = 0;
  each([&](uint32_t key, int i) {
    lt += i < base && key < thr;
    eq += i < base && key == thr;
  });
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lt += __shfl_xor(lt, o, 64);
    eq += __shfl_xor(eq, o, 64);
  }
  if (lane == 0) {
    atomicAdd(&sh.less, lt);
    atomicAdd(&sh.eq, eq);
  }
  __syncthreads();
  *thr_out = thr;
  *need_eq = rank + 1;
  *less0 = sh.less;
  *eq0 = sh.eq;
}

__global__ __launch_bounds__(256) void split_scatter_kernel(Ctx C, LevelArgs L) {
  __shared__ ChunkSelect sel;
  __shared__ int wsum[4];
  __shared__ uint32_t skey[kChunk + kChunk / 16];
  __shared__ int32_t srow[kChunk + kChunk / 16];
  __shared__ int32_t sout[kChunk];
  const int pid = blockIdx.z, side = pid / C.BH, node = blockIdx.y;
  const Side& S = C.s[side];
  if (L.level >= S.big) return;
  int start, size;
  node_range(S.n, S.c, L.level, node, &start, &size);
  const int c0 = blockIdx.x * kChunk;
  if (c0 >= size) return;
  const int c1 = min(size, c0 + kChunk), nc = c1 - c0;
  const int32_t* idx_in = L.idx_in + (size_t)pid * C.nmax;
  int32_t* idx_out = L.idx_out + (size_t)pid * C.nmax;
  const int32_t* ns = node_ptr(C, pid, node);
  const int t = threadIdx.x;
  if (size <= S.c) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int o = c0 + t + 256 * u;
      if (o < c1) idx_out[start + o] = L.first ? start + o : idx_in[start + o];
    }
    return;
  }
  const int mL = ns[3];
  const uint32_t* keys = C.keys + (size_t)pid * C.nmax;
  // coalesced loads of the chunk's keys and rows into LDS
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int i = t + 256 * u;
    if (i < nc) {
      skey[scat_slot(i)] = keys[start + c0 + i];
      srow[scat_slot(i)] = L.first ? start + c0 + i : idx_in[start + c0 + i];
    }
  }
  uint32_t thr = (uint32_t)ns[1];
  int less0 = 0, eq0 = 0, need_eq = ns[2] + 1;
  if (!ns[10]) {
    chunk_select(C, pid, ns, node * L.cpn, sel, &thr, &need_eq, &less0, &eq0);
  } else if (ns[7] > 1) {
    const int32_t* cc =
        C.chunk_cnt +
        ((size_t)pid * C.hist_slots + (size_t)node * L.cpn + blockIdx.x) * kChunkInts;
    less0 = cc[0];
    eq0 = cc[1];
  }
  __syncthreads();
  // Each thread owns kPer consecutive positions (the scan order).
  const int i0 = t * kPer;
  uint32_t kv[kPer];
  int less = 0, eq = 0;
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int i = i0 + u;
    kv[u] = i < nc ? skey[scat_slot(i)] : 0xFFFFFFFFu;
    less += i < nc && kv[u] < thr;
    eq += i < nc && kv[u] == thr;
  }
  int tot;
  const int packed = scan256((less << 16) | eq, wsum, &tot);
  // The chunk's left-goers land in one contiguous range of the node starting
  // at lmin, its right-goers in one starting at rmin: stage both in order,
  // left part first, then write them out coalesced.
  const int lmin = less0 + min(eq0, need_eq);
  const int rmin = mL + (c0 - lmin);
  const int tot_less = tot >> 16, tot_eq = tot & 0xFFFF;
  const int nleft = tot_less + min(eq0 + tot_eq, need_eq) - min(eq0, need_eq);
  int lb = less0 + (packed >> 16), eb = eq0 + (packed & 0xFFFF);
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int i = i0 + u;
    if (i >= nc) break;
    const uint32_t key = kv[u];
    const int Lo = lb + min(eb, need_eq);
    const bool left = key < thr || (key == thr && eb < need_eq);
    const int loc = left ? Lo - lmin : nleft + (c0 + i - Lo) - (c0 - lmin);
    if (loc >= 0 && loc < nc) sout[loc] = srow[scat_slot(i)];
    lb += key < thr;
    eb += key == thr;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int i = t + 256 * u;
    if (i < nc) {
      const int dst = i < nleft ? lmin + i : rmin + (i - nleft);
      if (dst >= 0 && dst < size) idx_out[start + dst] = sout[i];
    }
  }
}

// Remaining levels of one node (at most the side's tail size) in one
// workgroup. Thread t holds positions 256 w + 64 u + lane of the node (w, lane:
// its wavefront and lane; u = 0 .. 3) with their tokens and the range of the
// sub-node that each lies in. Per level:
//   choose     the coordinate of every sub-node (8 wavefronts share the sample
//              rows of the first levels' few sub-nodes)
//   keys       every position's coordinate, counted into linear bins of its
//              sub-node over mean +- 4 sd of the sample
//   select     the bin that holds the wanted rank, then the rank among that
//              bin's keys by counting (one wavefront a sub-node; more than 64
//              keys there: six radix passes of 6 bits over them)
//   partition  ballots of the keys below and equal to the threshold give every
//              position's place in its half
//
// What bounds it: small layers, the chain of barriers and memory trips, where
// choice, radix passes over the block and a partition through LDS prefix sums
// took 40,000 cycles a level for 1,024 tokens (now 17,000); large ones, the
// lines fetched for one coordinate of each scattered token. Times of the
// kernel: 63 -> 32 us (one head, 1,024 tokens), 123 -> 89 (8 heads,
// 65,521 tokens), 898 -> 668 (16 heads, 262,144), all at d = 64; 1,623 ->
// 742 (40 heads, 75,600 tokens, d = 128).
constexpr int kTailThreads = 512;
constexpr int kTailWaves = kTailThreads / 64;
constexpr int kTailPer = kTail / kTailThreads;
constexpr int kMaxSub = 32;
constexpr int kTailBins = 2048;  // bins of a level, shared evenly by its sub-nodes (at least 64 each)
static_assert(kTailPer == 4 && kTail / 64 <= 64, "position layout");

// Exact select by one wavefront: the rank-th smallest of keys[0, n), six bits
// at a time, high first (no pass for bits that all keys share). *rank becomes
// the rank among the keys equal to it.
__device__ uint32_t wave_radix_select(const uint32_t* keys, int n, int* rank, uint32_t* cnt,
                                      int lane) {
  uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
#pragma unroll 4
  for (int i = lane; i < n; i += 64) {
    kmin = min(kmin, keys[i]);
    kmax = max(kmax, keys[i]);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, o, 64));
    kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, o, 64));
  }
  uint32_t thr = 0u;
  int r = *rank;
  for (int shift = 26; shift >= -4; shift -= 6) {
    const int sh = shift < 0 ? 0 : shift;            // the last pass holds two bits
    const uint32_t mask = shift < 0 ? 3u : 63u;
    const int above = shift < 0 ? 2 : sh + 6;
    if (((kmin ^ kmax) >> sh) == 0u) {
      thr = kmin & (0xFFFFFFFFu << sh);
      continue;
    }
    cnt[lane] = 0u;
    wave_lds_order();
#pragma unroll 4
    for (int i = lane; i < n; i += 64) {
      const uint32_t key = keys[i];
      if (above >= 32 || (key >> above) == (thr >> above)) atomicAdd(&cnt[(key >> sh) & mask], 1u);
    }
    wave_lds_order();
    const int c = (int)cnt[lane];
    const int incl = wave_scan(c);
    const uint64_t hit = __ballot(r >= incl - c && r < incl);
    const int digit = hit ? __builtin_ctzll(hit) : 0;
    r -= __builtin_amdgcn_readlane(incl - c, digit);
    thr |= (uint32_t)digit << sh;
    wave_lds_order();
  }
  *rank = r;
  return thr;
}

template <int H>
__global__ __launch_bounds__(kTailThreads, 4) void split_tail_kernel(Ctx C, int parity0, int parity1) {
  __shared__ int32_t idx[kTail];
  __shared__ uint32_t keys[kTail];
  __shared__ int hist[kTailBins];
  __shared__ uint32_t cand[kTail];  // the ranks' bins' keys, kTail >> r for each sub-node
  __shared__ float2 part[kTailWaves][64 * H];
  __shared__ uint64_t mless[kTail / 64], meq[kTail / 64];
  __shared__ int sub_js[kMaxSub], sub_rank[kMaxSub], sub_bin[kMaxSub], sub_n[kMaxSub];
  __shared__ uint32_t sub_thr[kMaxSub];
  __shared__ float sub_lo[kMaxSub], sub_scale[kMaxSub];
  const int pid = blockIdx.y, side = pid / C.BH, bh = pid % C.BH, node = blockIdx.x;
  const Side& S = C.s[side];
  if (node >= (1 << S.big)) return;
  int start, size;
  node_range(S.n, S.c, S.big, node, &start, &size);
  const int par = side == 0 ? parity0 : parity1;
  const bool identity = S.big == 0;
  const int32_t* src = (par ? C.idx1 : C.idx0) + (size_t)pid * C.nmax;
  const float* Y = S.y + (size_t)bh * S.n * C.d;
  const float* ycol = S.ycol ? S.ycol + (size_t)bh * kColCopy * S.n : nullptr;
  const int d = C.d, c = S.c, lc = __builtin_ctz(c);
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto left = [&](int s) { return (((s + c - 1) >> lc) >> 1) << lc; };  // left_size
  // range of sub-node sl of level r
  auto sub_range = [&](int r, int sl, int* st, int* sz) {
    int a = 0, s = size;
    for (int b = r - 1; b >= 0; --b) {
      const int mL = s > c ? left(s) : s;
      if ((sl >> b) & 1) {
        a += mL;
        s -= mL;
      } else {
        s = mL;
      }
    }
    *st = a;
    *sz = s;
  };
  int row[kTailPer], st[kTailPer], sz[kTailPer], sl[kTailPer];
  uint32_t kv[kTailPer];
#pragma unroll
  for (int u = 0; u < kTailPer; ++u) {
    const int o = 256 * w + 64 * u + lane;
    row[u] = o < size ? (identity ? start + o : src[start + o]) : 0;
    st[u] = 0;
    sz[u] = o < size ? size : 0;  // positions past the node take part in nothing
    sl[u] = 0;
    idx[o] = row[u];
    hist[tid + kTailThreads * u] = 0;
  }
  if (tid < kMaxSub) sub_n[tid] = 0;
  __syncthreads();
  const int nclus = (size + c - 1) >> lc;
  const int nlev = S.levels - S.big;
  // a level splits nothing once every sub-node is one cluster (the right
  // halves are the larger ones: ceil(nclus / 2^r) clusters)
  for (int r = 0; r < nlev && ((nclus + (1 << r) - 1) >> r) >= 2; ++r) {
    const int nsub = 1 << r;
    const int nb = kTailBins >> r;       // bins per sub-node, 64 << lb of them
    const int lb = 5 - r;                // bin b is counted at (b % 2^lb) * 64 + b / 2^lb:
    const int cap = kTail >> r;          // the scan reads 64 of them side by side
    // ---- choose
    {
      const int P = nsub < kTailWaves ? kTailWaves >> r : 1;  // wavefronts per sub-node
      auto finish = [&](int s, int a, int z, int m, const Moments (&mo)[H]) {
        float mean, var;
        int js = choose_by_bounds<H>(mo, d, m, lane, &mean, &var);
        if (js < 0) js = choose_open<H, 16>(Y, d, idx, false, a, z, m, mo, lane, &mean, &var);
        if (lane == 0) {
          sub_js[s] = js;
          bin_range(mean, var, nb, &sub_lo[s], &sub_scale[s]);
        }
      };
      auto moments = [&](int a, int z, int m, int p, Moments (&mo)[H]) {
        uint32_t off[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
          off[h] = 4u * (uint32_t)d * (uint32_t)idx[a + sample_pos(min(lane + 64 * h, m - 1), z, m)];
        if (m <= 16 * P)
          sample_moments<H, 16>(Y, d, m, off, p, P, lane, mo);
        else
          sample_moments<H, 32>(Y, d, m, off, p, P, lane, mo);
      };
      if (P > 1) {
        const int s = w / P, p = w % P;
        int a, z;
        sub_range(r, s, &a, &z);
        const int m = min(z, d);
        const bool act = z > c;
        Moments mo[H];
        if (act) {
          moments(a, z, m, p, mo);
#pragma unroll
          for (int h = 0; h < H; ++h) part[w][lane + 64 * h] = make_float2(mo[h].S, mo[h].Q);
        }
        __syncthreads();
        if (act && p == 0) {
          for (int i = 1; i < P; ++i)
#pragma unroll
            for (int h = 0; h < H; ++h) {
              const float2 x = part[w + i][lane + 64 * h];
              mo[h].S += x.x;
              mo[h].Q += x.y;
            }
          finish(s, a, z, m, mo);
        }
      } else {
        for (int s = w; s < nsub; s += kTailWaves) {
          int a, z;
          sub_range(r, s, &a, &z);
          if (z <= c) continue;
          const int m = min(z, d);
          Moments mo[H];
          moments(a, z, m, 0, mo);
          finish(s, a, z, m, mo);
        }
      }
    }
    __syncthreads();
    // ---- keys and their bins
    float v[kTailPer];
#pragma unroll
    for (int u = 0; u < kTailPer; ++u) {
      v[u] = 0.f;
      if (sz[u] > c) {
        const int js = sub_js[sl[u]];
        // the chosen coordinate, from the coordinate-major copy when it holds
        // it (the nodes of a head run together, so they share its lines)
        v[u] = ycol && js < kColCopy ? ycol[(size_t)js * S.n + row[u]] : Y[(size_t)row[u] * d + js];
      }
    }
    int bin[kTailPer];
#pragma unroll
    for (int u = 0; u < kTailPer; ++u) {
      kv[u] = ordered_bits(v[u]);
      bin[u] = -1;
      if (sz[u] > c) {
        keys[256 * w + 64 * u + lane] = kv[u];
        bin[u] = lin_bin(kv[u], sub_lo[sl[u]], sub_scale[sl[u]], nb);
        atomicAdd(&hist[sl[u] * nb + ((bin[u] & ((1 << lb) - 1)) << 6) + (bin[u] >> lb)], 1);
      }
    }
    __syncthreads();
    // ---- select: the bin of the rank
    for (int s = w; s < nsub; s += kTailWaves) {
      int a, z;
      sub_range(r, s, &a, &z);
      if (z <= c) continue;
      const int rank = left(z) - 1;
      const int* hs = hist + s * nb;
      int sum = 0;  // of the 2^lb bins lane * 2^lb ..
      if (lb == 5) {
#pragma unroll
        for (int i = 0; i < 32; ++i) sum += hs[64 * i + lane];
      } else {
#pragma unroll 4
        for (int i = 0; i < (1 << lb); ++i) sum += hs[64 * i + lane];
      }
      const int before = wave_scan(sum) - sum;
      const uint64_t hl = __ballot(rank >= before && rank < before + sum);
      const int l = hl ? __builtin_ctzll(hl) : 0;
      const int cnt = lane < (1 << lb) ? hs[64 * lane + l] : 0;  // lane l's bins, one a lane
      const int acc = wave_scan(cnt) - cnt + __builtin_amdgcn_readlane(before, l);
      if (rank >= acc && rank < acc + cnt) {
        sub_bin[s] = (l << lb) + lane;
        sub_rank[s] = rank - acc;
      }
    }
    __syncthreads();
    // ---- that bin's keys
#pragma unroll
    for (int u = 0; u < kTailPer; ++u) {
      if (bin[u] >= 0 && bin[u] == sub_bin[sl[u]]) {
        const int i = atomicAdd(&sub_n[sl[u]], 1);
        if (i < cap) cand[sl[u] * cap + i] = kv[u];
      }
    }
    __syncthreads();
    // ---- the rank-th of them
    for (int s = w; s < nsub; s += kTailWaves) {
      int a, z;
      sub_range(r, s, &a, &z);
      if (z <= c) continue;
      const int n = __builtin_amdgcn_readfirstlane(sub_n[s]);
      uint32_t thr;
      int rank;
      if (n <= 64) {
        const int want = sub_rank[s];
        const uint32_t key = lane < n ? cand[s * cap + lane] : 0xFFFFFFFFu;
        int less = 0, eq = 0;
#pragma unroll 4
        for (int j = 0; j < n; ++j) {
          const uint32_t kj = (uint32_t)__builtin_amdgcn_readlane((int)key, j);
          less += kj < key;
          eq += kj == key;
        }
        const uint64_t hit = __ballot(lane < n && want >= less && want < less + eq);
        const int l = hit ? __builtin_ctzll(hit) : 0;
        thr = (uint32_t)__builtin_amdgcn_readlane((int)key, l);
        rank = want - __builtin_amdgcn_readlane(less, l);
      } else {
        const bool part_only = n <= cap;  // else more keys than the list holds: over all
        rank = part_only ? sub_rank[s] : left(z) - 1;
        thr = wave_radix_select(part_only ? cand + s * cap : keys + a, part_only ? n : z, &rank,
                                reinterpret_cast<uint32_t*>(hist) + 64 * s, lane);
      }
      if (lane == 0) {
        sub_thr[s] = thr;
        sub_rank[s] = rank;
        sub_n[s] = 0;
      }
    }
    __syncthreads();
    // ---- stable partition
    uint64_t bl[kTailPer], be[kTailPer];
#pragma unroll
    for (int u = 0; u < kTailPer; ++u) {
      const bool act = sz[u] > c;
      const uint32_t thr = act ? sub_thr[sl[u]] : 0u;
      hist[tid + kTailThreads * u] = 0;  // for the next level
      bl[u] = __ballot(act && kv[u] < thr);
      be[u] = __ballot(act && kv[u] == thr);
      if (lane == 0) {
        mless[4 * w + u] = bl[u];
        meq[4 * w + u] = be[u];
      }
    }
    __syncthreads();
    {
      // (below, equal) counts of the rows of 64 positions before row `lane`
      int pre = 0;
      if (lane < kTail / 64) pre = (__popcll(mless[lane]) << 16) | __popcll(meq[lane]);
      pre = wave_scan(pre) - pre;
#pragma unroll
      for (int u = 0; u < kTailPer; ++u) {
        const int o = 256 * w + 64 * u + lane;
        int dst = o;
        // the counts before the sub-node's first position
        const int sr = st[u] >> 6;
        const uint64_t low = (1ull << (st[u] & 63)) - 1ull;
        int at0 = __shfl(pre, sr, 64);
        at0 += (__popcll(mless[sr] & low) << 16) | __popcll(meq[sr] & low);
        if (sz[u] > c) {
          const uint64_t before = (1ull << lane) - 1ull;
          const int at = __builtin_amdgcn_readlane(pre, 4 * w + u) +
                         ((__popcll(bl[u] & before) << 16) | __popcll(be[u] & before));
          const int rel = at - at0, lb = rel >> 16, eb = rel & 0xFFFF;
          const uint32_t thr = sub_thr[sl[u]];
          const int need_eq = sub_rank[sl[u]] + 1;
          const int mL = left(sz[u]);
          const int Lo = lb + min(eb, need_eq);
          const bool goes = kv[u] < thr || (kv[u] == thr && eb < need_eq);
          const int rd = goes ? Lo : mL + (o - st[u] - Lo);
          dst = rd >= 0 && rd < sz[u] ? st[u] + rd : -1;
        }
        if (dst >= 0) idx[dst] = row[u];
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kTailPer; ++u) {
      const int o = 256 * w + 64 * u + lane;
      row[u] = idx[o];
      const int mL = sz[u] > c ? left(sz[u]) : sz[u];
      const bool right = o - st[u] >= mL && sz[u] > c;
      sl[u] = 2 * sl[u] + (right ? 1 : 0);
      st[u] += right ? mL : 0;
      sz[u] = right ? sz[u] - mL : mL;
    }
  }
  int32_t* perm = S.perm + (size_t)bh * S.n;
#pragma unroll
  for (int u = 0; u < kTailPer; ++u) {
    const int o = 256 * w + 64 * u + lane;
    if (o < size) perm[start + o] = row[u];
  }
}

// ---------------------------------------------------------------------------
// Gather: permuted copies (pad rows zero), centroids of the original vectors,
// counts, cluster ids. Values follow the key permutation and are stored per
// key cluster as a d x c tile (dimension-major), which is the operand layout
// of the value product in the attention kernels.
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(128) void gather_kernel(Ctx C) {
  extern __shared__ __attribute__((aligned(16))) float gsh[];  // value tile staging [c][d]
  const int pid = blockIdx.y, side = pid / C.BH, bh = pid % C.BH, a = blockIdx.x;
  const Side& S = C.s[side];
  if (a >= S.nc) return;
  const int d = C.d, c = S.c, t = threadIdx.x;
  const int cnt = min(c, S.n - a * c);
  const int32_t* perm = S.perm + (size_t)bh * S.n + (size_t)a * c;
  if (t == 0) S.count[(size_t)bh * S.nc + a] = cnt;
  if (S.cid)
    for (int r = t; r < cnt; r += 128) S.cid[(size_t)bh * S.n + perm[r]] = a;
  const size_t xrow0 = ((size_t)bh * S.npad + (size_t)a * c) * d;
  const bool vals = side == 1 && C.v != nullptr;
  for (int tt = t; tt < d; tt += 128) {
    float s = 0.f, sv = 0.f;
    for (int r = 0; r < c; ++r) {
      float x = 0.f, xv = 0.f;
      if (r < cnt) {
        const int i = perm[r];
        x = load_x(S.x, bh, i, S.lx, tt, C.dtype);
        s += x;
        if (vals) {
          xv = load_x(C.v, bh, i, C.lv, tt, C.dtype);
          sv += xv;
        }
      }
      store_elem(S.xp, xrow0 + (size_t)r * d + tt, C.dtype, x);
      if (vals) gsh[r * d + tt] = xv;
    }
    S.cent[((size_t)bh * S.nc + a) * d + tt] = s / (float)cnt;
    if (vals) C.cent_v[((size_t)bh * S.nc + a) * d + tt] = sv / (float)cnt;
  }
  if (vals) {
    __syncthreads();
    const size_t vt0 = ((size_t)bh * S.nc + a) * (size_t)d * c;
    for (int e = t; e < d * c; e += 128) {
      const int dd = e / c, r = e % c;
      store_elem(C.vp, vt0 + e, C.dtype, gsh[r * d + dd]);
    }
  }
}

// Fast gather for rows that are a whole number of 16-byte chunks: one
// workgroup per cluster copies the cluster's rows chunk by chunk (coalesced
// on both sides), sums the centroids in registers and then across the
// workgroup in a fixed order (deterministic), and transposes the value rows
// through LDS so that the value tiles are written 16 bytes at a time.
template <typename T>
__global__ __launch_bounds__(256) void gather_fast_kernel(Ctx C) {
  extern __shared__ __attribute__((aligned(16))) float gfs[];
  constexpr int EPC = 16 / sizeof(T);  // elements per 16-byte chunk
  const int pid = blockIdx.y, side = pid / C.BH, bh = pid % C.BH, a = blockIdx.x;
  const Side& S = C.s[side];
  if (a >= S.nc) return;
  const int d = C.d, c = S.c, tid = threadIdx.x;
  const int cpr = d / EPC;        // chunks per row (divides 256: d <= 128)
  const int rstep = 256 / cpr;    // row stride of one thread
  const int col = tid % cpr, r0 = tid / cpr;
  const int cnt = min(c, S.n - a * c);
  const int32_t* perm = S.perm + (size_t)bh * S.n + (size_t)a * c;
  const bool vals = side == 1 && C.v != nullptr;
  float* part = gfs;                            // [rstep][d] partial sums of x
  float* partv = gfs + rstep * d;               // [rstep][d] partial sums of v
  T* vstage = (T*)(gfs + 2 * rstep * d);        // [c][d] value rows
  if (tid == 0) S.count[(size_t)bh * S.nc + a] = cnt;
  if (S.cid)
    for (int r = tid; r < cnt; r += 256) S.cid[(size_t)bh * S.n + perm[r]] = a;
  float acc[EPC], accv[EPC];
#pragma unroll
  for (int u = 0; u < EPC; ++u) acc[u] = accv[u] = 0.f;
  T* dst = (T*)S.xp + ((size_t)bh * S.npad + (size_t)a * c) * d;
  // A thread's rows r0, r0 + rstep, ... (at most kGatherRows of them): all
  // loads are issued before the first is used.
  constexpr int kGatherRows = 8;
  for (int rb = r0; rb < c; rb += kGatherRows * rstep) {
    uint4 chunk[kGatherRows], vchunk[kGatherRows];
#pragma unroll
    for (int u = 0; u < kGatherRows; ++u) {
      const int r = rb + u * rstep;
      chunk[u] = vchunk[u] = make_uint4(0u, 0u, 0u, 0u);
      if (r < cnt) {
        const int i = perm[r];
        chunk[u] = *(const uint4*)((const T*)S.x + row_off(bh, i, S.lx) + col * EPC);
        if (vals)
          vchunk[u] =
              *(const uint4*)((const T*)C.v + row_off(bh, i, C.lv) + col * EPC);
      }
    }
#pragma unroll
    for (int u = 0; u < kGatherRows; ++u) {
      const int r = rb + u * rstep;
      if (r >= c) break;
      *(uint4*)(dst + (size_t)r * d + col * EPC) = chunk[u];
      union {
        uint4 v;
        T e[EPC];
      } cx, cv;
      cx.v = chunk[u];
#pragma unroll
      for (int e = 0; e < EPC; ++e) acc[e] += (float)cx.e[e];
      if (vals) {
        *(uint4*)(vstage + r * d + col * EPC) = vchunk[u];
        cv.v = vchunk[u];
#pragma unroll
        for (int e = 0; e < EPC; ++e) accv[e] += (float)cv.e[e];
      }
    }
  }
#pragma unroll
  for (int u = 0; u < EPC; ++u) {
    part[r0 * d + col * EPC + u] = acc[u];
    if (vals) partv[r0 * d + col * EPC + u] = accv[u];
  }
  __syncthreads();
  for (int f = tid; f < d; f += 256) {
    float sx = 0.f, sv = 0.f;
    for (int g = 0; g < rstep; ++g) {
      sx += part[g * d + f];
      if (vals) sv += partv[g * d + f];
    }
    S.cent[((size_t)bh * S.nc + a) * d + f] = sx / (float)cnt;
    if (vals) C.cent_v[((size_t)bh * S.nc + a) * d + f] = sv / (float)cnt;
  }
  if (vals) {
    // value tile [d][c]: chunk = EPC consecutive rows of one dimension
    T* vt = (T*)C.vp + ((size_t)bh * S.nc + a) * (size_t)d * c;
    const int cpc = c / EPC;  // chunks per tile row (c >= EPC)
    for (int e = tid; e < d * cpc; e += 256) {
      const int f = e / cpc, rr = (e % cpc) * EPC;
      union {
        uint4 v;
        T e[EPC];
      } tmp;
#pragma unroll
      for (int u = 0; u < EPC; ++u) tmp.e[u] = vstage[(rr + u) * d + f];
      *(uint4*)(vt + (size_t)f * c + rr) = tmp.v;
    }
  }
}

int tail_size(int c) { return c * 64 < kTail ? c * 64 : kTail; }

// Largest node of level l: the sizes of a level are few (whole clusters in two
// numbers, the node with the remainder, empty slots), so the levels are gone down by
// distinct size. With node_range of each of a level's slots a call's plan took 164
// us of host time where all levels are multi-block (basic splitting of 238,577
// tokens, 13 levels); now 9.
int level_max(int n, int c, int l) {
  int sizes[16] = {n}, m = 1;
  for (; l > 0; --l) {
    int next[16], k = 0;
    for (int i = 0; i < m; ++i) {
      const int s = sizes[i], mL = s > c ? left_size(s, c) : s;
      for (const int x : {mL, s - mL})
        if (k < 16 && std::find(next, next + k, x) == next + k) next[k++] = x;
    }
    std::copy(next, next + k, sizes);
    m = k;
  }
  return *std::max_element(sizes, sizes + m);
}

}  // namespace

int split_level_cpn(const Prob& P, int big_q, int big_k, int l) {
  int maxs = 0;
  for (int side = 0; side < 2; ++side) {
    const int n = side == 0 ? P.nq : P.nk, c = side == 0 ? P.cq : P.ck;
    if (l >= (side == 0 ? big_q : big_k)) continue;
    maxs = std::max(maxs, level_max(n, c, l));
  }
  return (maxs + kChunk - 1) / kChunk;
}

int split_hist_slots(const Prob& P, int big_q, int big_k) {
  const int big = big_q > big_k ? big_q : big_k;
  int slots = 1;
  for (int l = 0; l < big; ++l) {
    const int s = (1 << l) * split_level_cpn(P, big_q, big_k, l);
    if (s > slots) slots = s;
  }
  return slots;
}

int split_group_slots(const Prob& P, int big_q, int big_k) {
  const int big = big_q > big_k ? big_q : big_k;
  int slots = 0;
  for (int l = 0; l < big; ++l) {
    const int cpn = split_level_cpn(P, big_q, big_k, l);
    if (cpn > kGroupedFrom) slots = std::max(slots, (1 << l) * ((cpn + kGroup - 1) / kGroup));
  }
  return slots;
}

int split_big_levels(int n, int c, int L) {
  const int tail = tail_size(c);
  int l = 0;
  while (l < L && level_max(n, c, l) > tail) ++l;
  return l;
}

namespace {
// Kernels that use more than 64 KiB of dynamic LDS declare their size once. A
// refusal is not fatal here: the launch itself reports a real limit.
constexpr size_t kEighLds = eigh_lds_bytes(kMaxD);
constexpr size_t chol_lds_bytes(int dm) { return (size_t)dm * (dm + 1) * sizeof(float); }
constexpr size_t kQnormLds = (size_t)(kMaxD + 2 * kStage) * kDP * sizeof(float);
constexpr size_t kProjLds = (size_t)(kMaxD + kStage) * kDP * sizeof(float);
constexpr size_t kGatherLds = (size_t)kMaxC * kMaxD * sizeof(float);
hipError_t set_lds_limits() {
  static bool done = [] {
    (void)hipFuncSetAttribute((const void*)eigh_kernel<128>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)kEighLds);
    (void)hipFuncSetAttribute((const void*)eigh_kernel<64>,
                              hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)eigh_lds_bytes(64));
    (void)hipFuncSetAttribute((const void*)cholesky_kernel<128>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)chol_lds_bytes(128));
    (void)hipFuncSetAttribute((const void*)qnorm_partial_kernel,
                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)kQnormLds);
    (void)hipFuncSetAttribute((const void*)project_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                        (int)kProjLds);
    (void)hipFuncSetAttribute((const void*)gather_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                        (int)kGatherLds);
    for (const void* f : {(const void*)basic_choose_kernel<0>, (const void*)basic_choose_kernel<128>})
      (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)((size_t)kMaxD * (kMaxD + 1) * sizeof(float)));
    (void)hipFuncSetAttribute((const void*)gather_fast_kernel<bf16>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    (void)hipFuncSetAttribute((const void*)gather_fast_kernel<float>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    (void)hipGetLastError();
    return true;
  }();
  (void)done;
  return hipSuccess;
}
}  // namespace

hipError_t launch_cluster(const Prob& P, const void* q, const void* k, const void* v,
                          const ca_cluster_out* out, char* ws, const Workspace& W,
                          hipStream_t st) {
  {
    hipError_t le = set_lds_limits();
    if (le != hipSuccess) return le;
  }
  Ctx C = {};
  const int d = P.d;
  C.BH = P.BH;
  C.H = P.H;
  C.d = d;
  C.dtype = P.dtype;
  C.lv = P.lv;
  C.xf = P.xf;
  C.nmax = P.nq > P.nk ? P.nq : P.nk;
  C.nblk = W.nblk_mom;
  C.mom_rows = W.mom_rows;
  C.proj_rows = kProjRows;  // set for the projection launch below
  C.v = v;
  C.cent_v = out->cent_v;
  C.vp = out->vp;
  C.mats = (float*)(ws + W.mats);
  C.vecs = (float*)(ws + W.vecs);
  C.inv_q = (float*)(ws + W.inv_q);
  C.mom_part = (float*)(ws + W.mom_part);
  C.qn_part = (float*)(ws + W.qn_part);
  C.wops = (bf16*)(ws + W.wops);
  C.idx0 = (int32_t*)(ws + W.idx0);
  C.idx1 = (int32_t*)(ws + W.idx1);
  C.keys = (uint32_t*)(ws + W.keys);
  C.node_state = (int32_t*)(ws + W.node_state);
  C.hist = (uint32_t*)(ws + W.hist);
  C.cand = (uint32_t*)(ws + W.cand);
  C.chunk_cnt = (int32_t*)(ws + W.chunk_cnt);
  C.max_nodes = W.max_big_nodes;
  C.hist_slots = W.hist_slots;
  C.ghist = (uint32_t*)(ws + W.ghist);
  C.ghist_slots = W.ghist_slots;
  C.split = P.split;
  C.dirs = (float*)(ws + W.dirs);
  const bool basic = P.split == CA_SPLIT_BASIC;
  Side& Sq = C.s[0];
  Side& Sk = C.s[1];
  Sq.x = q;
  Sk.x = k;
  Sq.lx = P.lq;
  Sk.lx = P.lk;
  if (P.lq.H < 1 || P.lk.H < 1 || P.lv.H < 1) return hipErrorInvalidValue;
  Sq.y = out->yq_dbg ? out->yq_dbg : (float*)(ws + W.y_q);
  Sk.y = out->yk_dbg ? out->yk_dbg : (float*)(ws + W.y_k);
  // coordinate-major leading coordinates, where a multi-block level reads them
  const bool cols = col_copy_used(P);
  Sq.ycol = cols && W.big_q > 0 ? (float*)(ws + W.ycol_q) : nullptr;
  Sk.ycol = cols && W.big_k > 0 ? (float*)(ws + W.ycol_k) : nullptr;
  Sq.perm = out->perm_q;
  Sk.perm = out->perm_k;
  Sq.cid = out->cid_q;
  Sk.cid = out->cid_k;
  Sq.count = out->count_q;
  Sk.count = out->count_k;
  Sq.cent = out->cent_q;
  Sk.cent = out->cent_k;
  Sq.xp = out->qp;
  Sk.xp = out->kp;
  Sq.n = P.nq;
  Sk.n = P.nk;
  Sq.c = P.cq;
  Sk.c = P.ck;
  Sq.nc = P.nqc;
  Sk.nc = P.nkc;
  Sq.npad = P.nq_pad;
  Sk.npad = P.nk_pad;
  Sq.levels = W.levels_q;
  Sk.levels = W.levels_k;
  Sq.big = W.big_q;
  Sk.big = W.big_k;
  Sq.tail = tail_size(P.cq);
  Sk.tail = tail_size(P.ck);
  const int BH = P.BH;
  hipError_t e;
#define CA_CHECK()                          \
  do {                                      \
    e = hipGetLastError();                  \
    if (e != hipSuccess) return e;          \
  } while (0)

  const bool mfma = P.dtype == CA_BF16 && (d == 64 || d == 128);
  const bool transformed = P.xf != CA_XF_NONE && P.xf != CA_XF_RANDOM;
  if (transformed) {
    if (mfma && d == 64)
      hipLaunchKernelGGL(moments_mfma_kernel<64>, dim3(C.nblk, 2 * BH), dim3(256), 0, st, C);
    else if (mfma)
      hipLaunchKernelGGL(moments_mfma_kernel<128>, dim3(C.nblk, 2 * BH), dim3(256), 0, st, C);
    else
      hipLaunchKernelGGL(moments_partial_kernel, dim3(C.nblk, 2 * BH), dim3(256), 0, st, C);
    CA_CHECK();
    const bool few = (size_t)2 * BH * (d * d + d) <= (size_t)1 << 18;
    const int per = few ? 32 : 256;  // elements a workgroup of the finishing kernels
    hipLaunchKernelGGL((few ? moments_finish_kernel<8> : moments_finish_kernel<1>),
                       dim3((d * d + d + per - 1) / per, BH, 2), dim3(256), 0, st, C);
    CA_CHECK();
    const int wq = P.dtype == CA_BF16 ? (int)O_TQ : -1, wk = P.dtype == CA_BF16 ? (int)O_TK : -1;
    EighJobs J;
    if (P.xf == CA_XF_PCA) {
      // principal axes of the centred queries and keys, oriented by the means
      J.j[0] = {M_A0, -1, -1, 0, V_MUQ, -1, M_TQ, wq};
      J.j[1] = {M_CK, -1, -1, 0, V_MUK, -1, M_TK, wk};
    } else {
      const int fk = P.dtype == CA_BF16 ? (int)O_FK : -1;
      if (d <= 64)
        hipLaunchKernelGGL(cholesky_kernel<64>, dim3(BH, 2), dim3(chol_threads<64>()),
                           chol_lds_bytes(64), st, C, (int)M_A0, (int)M_E0, (int)M_CK, (int)M_EK, fk);
      else
        hipLaunchKernelGGL(cholesky_kernel<128>, dim3(BH, 2), dim3(chol_threads<128>()),
                           chol_lds_bytes(128), st, C, (int)M_A0, (int)M_E0, (int)M_CK, (int)M_EK, fk);
      CA_CHECK();
      if (P.xf == CA_XF_METRIC) {
        const size_t qlds = kQnormLds;
        if (mfma && d == 64)
          hipLaunchKernelGGL(qnorm_mfma_kernel<64>, dim3(C.nblk, BH), dim3(256), 0, st, C);
        else if (mfma)
          hipLaunchKernelGGL(qnorm_mfma_kernel<128>, dim3(C.nblk, BH), dim3(256), 0, st, C);
        else
          hipLaunchKernelGGL(qnorm_partial_kernel, dim3(C.nblk, BH), dim3(256), qlds, st, C);
        CA_CHECK();
        hipLaunchKernelGGL(qnorm_finish_kernel, dim3((d * d + d + 255) / 256, BH), dim3(256), 0,
                           st, C);
        CA_CHECK();
      }
      // keys: C2 = S_q^T C_K S_q, oriented by S_q^T mu_K, T_K = S_q U2
      J.j[0] = {M_CK, M_E0, V_MUK, 0, -1, M_E0, M_TK, wk};
      if (P.xf == CA_XF_ADAPTIVE)
        // queries: cov(q S_k) = S_k^T (Q^T Q / n - mu_Q mu_Q^T) S_k, oriented by
        // S_k^T mu_Q (the mean of q S_k), W_Q = S_k U3; no normalisation
        J.j[1] = {M_A0, M_EK, V_MUQ, 1, -1, M_EK, M_TQ, wq};
      else if (mfma)
        // queries: cov(r(q)), oriented by mu_r, W_Q = S_k U3
        J.j[1] = {M_C3, M_EK, V_MUR, 1, -1, M_EK, M_TQ, wq};
      else
        J.j[1] = {M_C3, -1, V_MUR, 1, -1, M_EK, M_TQ, wq};
    }
    if (basic)  // the metric root space: the Cholesky factors are the projections
      hipLaunchKernelGGL(copy_roots_kernel, dim3(BH), dim3(256), 0, st, C, (int)mfma);
    else if (d <= 64)
      hipLaunchKernelGGL(eigh_kernel<64>, dim3(BH, 2), dim3(eigh_threads<64>()), eigh_lds_bytes(64), st, C, J);
    else
      hipLaunchKernelGGL(eigh_kernel<128>, dim3(BH, 2), dim3(eigh_threads<128>()), kEighLds, st, C, J);
    CA_CHECK();
  }
  {
    const int nmax = C.nmax;
    const size_t plds = kProjLds;
    // the MFMA pass takes 128 rows per step, the fp32 one 32
    C.proj_rows = rows_per_block(nmax, mfma && transformed ? 128 : 32, kProjRows, 2 * BH);
    const dim3 pgrid((nmax + C.proj_rows - 1) / C.proj_rows, 2 * BH);
    if (mfma && transformed && d == 64)
      hipLaunchKernelGGL(project_mfma_kernel<64>, pgrid, dim3(256), 0, st, C);
    else if (mfma && transformed)
      hipLaunchKernelGGL(project_mfma_kernel<128>, pgrid, dim3(256), 0, st, C);
    else
      hipLaunchKernelGGL(project_kernel, pgrid, dim3(256), plds, st, C);
    CA_CHECK();
  }
  const int big = W.big_q > W.big_k ? W.big_q : W.big_k;
  for (int l = 0; l < big; ++l) {
    LevelArgs L;
    L.level = l;
    L.first = l == 0;
    L.idx_in = (l & 1) ? C.idx1 : C.idx0;
    L.idx_out = (l & 1) ? C.idx0 : C.idx1;
    const int cpn = split_level_cpn(P, W.big_q, W.big_k, l);
    L.cpn = cpn;
    if (basic) {
      const size_t blds = (size_t)d * (d + 1) * sizeof(float);
      if (d == 64)
        hipLaunchKernelGGL(basic_choose64_kernel, dim3(1 << l, 2 * BH), dim3(64), 0, st, C, L);
      else if (d == 128)
        hipLaunchKernelGGL(basic_choose_kernel<128>, dim3(1 << l, 2 * BH), dim3(kBasicThreads),
                           blds, st, C, L);
      else
        hipLaunchKernelGGL(basic_choose_kernel<0>, dim3(1 << l, 2 * BH), dim3(kBasicThreads),
                           blds, st, C, L);
    }
    else
      hipLaunchKernelGGL((d <= 64 ? split_choose_kernel<1> : split_choose_kernel<2>),
                         dim3(1 << l, 2 * BH), dim3(64 * kChooseWaves), 0, st, C, L);
    CA_CHECK();
    const dim3 kgrid(cpn, 1 << l, 2 * BH);
    if (!basic)
      hipLaunchKernelGGL(split_keys_kernel<-1>, kgrid, dim3(256), 0, st, C, L);
    else if (d == 64)
      hipLaunchKernelGGL(split_keys_kernel<64>, kgrid, dim3(256), 0, st, C, L);
    else if (d == 128)
      hipLaunchKernelGGL(split_keys_kernel<128>, kgrid, dim3(256), 0, st, C, L);
    else
      hipLaunchKernelGGL(split_keys_kernel<0>, kgrid, dim3(256), 0, st, C, L);
    CA_CHECK();
    if (cpn > 1) {  // nodes of one chunk are selected with their keys
      hipLaunchKernelGGL(split_bins_kernel, kgrid, dim3(256), 0, st, C, L);
      CA_CHECK();
    }
    hipLaunchKernelGGL(split_scatter_kernel, dim3(cpn, 1 << l, 2 * BH), dim3(256), 0, st, C, L);
    CA_CHECK();
  }
  {
    // After its last multi-block level, side s holds its order in idx[(big_s) & 1].
    const int nodes = 1 << big;
    if (basic)
      hipLaunchKernelGGL(copy_order_kernel, dim3((C.nmax + 255) / 256 < 1024 ? (C.nmax + 255) / 256 : 1024, 2 * BH),
                         dim3(256), 0, st, C, W.big_q & 1, W.big_k & 1);
    else
      hipLaunchKernelGGL((d <= 64 ? split_tail_kernel<1> : split_tail_kernel<2>), dim3(nodes, 2 * BH),
                         dim3(kTailThreads), 0, st, C, W.big_q & 1, W.big_k & 1);
    CA_CHECK();
  }
  {
    const int maxc = P.nqc > P.nkc ? P.nqc : P.nkc;
    const int epc = 16 / (int)P.esize;
    const bool fast = (d % epc == 0) && (P.ck % epc == 0) && ((256 / (d / epc)) * (d / epc) == 256);
    if (fast) {
      const int rstep = 256 / (d / epc);
      const size_t glds = (size_t)2 * rstep * d * sizeof(float) + (v ? (size_t)P.ck * d * P.esize : 0);
      if (P.dtype == CA_BF16)
        hipLaunchKernelGGL(gather_fast_kernel<bf16>, dim3(maxc, 2 * BH), dim3(256), glds, st, C);
      else
        hipLaunchKernelGGL(gather_fast_kernel<float>, dim3(maxc, 2 * BH), dim3(256), glds, st, C);
    } else {
      const size_t glds = v ? (size_t)P.ck * d * sizeof(float) : 0;
      hipLaunchKernelGGL(gather_kernel, dim3(maxc, 2 * BH), dim3(128), glds, st, C);
    }
    CA_CHECK();
  }
#undef CA_CHECK
  return hipSuccess;
}

// ---------------------------------------------------------------------------
// Checked mode: flag bits of the tensors holding a NaN or an infinity
// ---------------------------------------------------------------------------

namespace {

__global__ void flags_clear_kernel(int32_t* flags) { flags[0] = 0; }

// One block of 256 threads per 64 rows of one tensor (blockIdx.y: 0 q, 1 k,
// 2 v); a value is non-finite when its exponent bits are all ones.
__global__ __launch_bounds__(256) void check_finite_kernel(const void* q, const void* k,
                                                           const void* v, Lay lq, Lay lk, Lay lv,
                                                           int nq, int nk, int BH, int d,
                                                           int dtype, int32_t* flags) {
  const int t = blockIdx.y;
  const void* x = t == 0 ? q : (t == 1 ? k : v);
  const Lay& L = t == 0 ? lq : (t == 1 ? lk : lv);
  const int n = t == 0 ? nq : nk;
  const long long rows = (long long)BH * n;
  const long long r0 = (long long)blockIdx.x * 64;
  int bad = 0;
  if (x != nullptr) {
    for (int e = threadIdx.x; e < 64 * d; e += 256) {
      const long long r = r0 + e / d;
      if (r >= rows) break;
      const int bh = (int)(r / n), i = (int)(r % n), c = e % d;
      const size_t off = row_off(bh, i, L) + c;
      if (dtype == CA_BF16) {
        const uint16_t u = ((const uint16_t*)x)[off];
        bad |= (u & 0x7F80u) == 0x7F80u;
      } else {
        const uint32_t u = ((const uint32_t*)x)[off];
        bad |= (u & 0x7F800000u) == 0x7F800000u;
      }
    }
  }
  if (__syncthreads_or(bad) && threadIdx.x == 0) atomicOr(flags, 1 << t);
}

}  // namespace

hipError_t launch_check_finite(const Prob& P, const void* q, const void* k, const void* v,
                               int32_t* flags, hipStream_t st) {
  hipLaunchKernelGGL(flags_clear_kernel, dim3(1), dim3(1), 0, st, flags);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const long long rows = (long long)P.BH * (P.nq > P.nk ? P.nq : P.nk);
  const unsigned blocks = (unsigned)((rows + 63) / 64);
  hipLaunchKernelGGL(check_finite_kernel, dim3(blocks, v ? 3 : 2), dim3(256), 0, st, q, k, v,
                     P.lq, P.lk, P.lv, P.nq, P.nk, P.BH, P.d, P.dtype, flags);
  return hipGetLastError();
}

}  // namespace ca
