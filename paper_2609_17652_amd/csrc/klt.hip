// KLT-rotated store: Sec. 3.5 (basis rule).  The rotated variant stores the
// planes of (k - mu) V, mu the mean and V the orthonormal eigenbasis of the
// covariance of a unit's calibration keys, and allocates depths with
// g_j = sum_h ((q_h V)_j)^2 lambda_j -- i.e. the unchanged pack, depth
// allocation and scan run on rotated keys, rotated queries and var = lambda.
//
// fathom_klt_calibrate (one-time, per unit; the unit's own keys calibrate):
//   klt_cov_kernel    chunks of the keys: fp64 sums of y and y y^T, y the keys
//                     shifted by the unit's first, on the fp64 matrix cores.
//   klt_reduce_kernel the chunks' sums in chunk order: mean and covariance.
//   klt_eig_kernel    one workgroup per unit: Cholesky factor in fp64, cyclic
//                     one-sided Jacobi on it in fp32.
//   klt_refine_kernel the basis refined and the eigenvalues, in fp64.
//   klt_order_kernel  the columns ordered by eigenvalue (descending), with each
//                     column's largest-magnitude entry made positive.
// fathom_klt_rotate_keys (prefill) and fathom_klt_rotate_q (per step) compute
// in fp32 in a fixed order: d_j = fl(k_j - mu_j) (no mean for q), then for
// j = 0 .. D-1: acc_c = fl(acc_c + fl(d_j V[j][c])), no fused multiply-add, so
// the rotated operands (and every plane, depth and score built from them) are
// reproducible bit for bit.  The rotation is a dense contraction, but the MFMA
// accumulation order is not this one; it runs once per token at prefill.
#include "common.hpp"

namespace fathom {

constexpr size_t kCalUnitBytes = (size_t)32 * kD * (kD + 1) * sizeof(double);  // calibration workspace of one unit
constexpr int kCalChunks = 54;        // token chunks per unit in the calibration sums, at most (they fit the above)
constexpr int kEigThreads = 512;
// At most.  128 channels take 2 to 6 sweeps for fewer than 8 keys, 4 to 10 for
// eigenvalues over up to four decades, 11 to 14 over nine and up to all 16 over more
// than ten, where what is left is below the rounding of the largest.
constexpr int kJacobiSweeps = 16;
// A pair whose cosine is below 1.4e-6 (the rounding of a dot product) is not
// rotated.  The sweeps end when every rotation of a sweep was of a cosine below
// 1e-4 by a tangent below 2^-10: what the up to 127 rotations of a column leave
// of its other pairs' cosines is then about sqrt(127) * 1e-7.
constexpr float kJacobiSkip2 = 2e-12f, kJacobiTol2 = 1e-8f, kJacobiTan = 0x1p-10f;
constexpr double kCholShift = 1e-7;   // of the trace
// Rotations of the refinement are left out from this size on (its square stays in
// V^T V - I), and between eigenvalues closer than this share of the trace.
constexpr double kRefineMax = 0x1p-13, kRefineGap = 1e-10;
constexpr int kRotThreads = 256;
constexpr int kRotTokens = 4;         // tokens a wave rotates at a time

// Per unit: the covariance (fp64, 128 KB) and up to kCalChunks chunks' sums.
size_t klt_ws_bytes(int U) { return (size_t)U * kCalUnitBytes; }

template <typename KT>
__device__ __forceinline__ float key_at(const KT* p) {
  if constexpr (sizeof(KT) == 4) return *(const __attribute__((address_space(1))) float*)p;
  return half_bits_to_float(*(const __attribute__((address_space(1))) uint16_t*)p);
}

template <typename KT, bool VEC>
struct KeyRow {  // 8 consecutive channels of one token, as read
  uint32_t w[2 * sizeof(KT)];
  __device__ __forceinline__ void load(const KT* p) {
    if constexpr (VEC) {
#pragma unroll
      for (int i = 0; i < (int)sizeof(KT) / 2; ++i) {
        const uint4 r = reinterpret_cast<const uint4*>(p)[i];
        w[4 * i] = r.x; w[4 * i + 1] = r.y; w[4 * i + 2] = r.z; w[4 * i + 3] = r.w;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if constexpr (sizeof(KT) == 4) {
          w[e] = *(const __attribute__((address_space(1))) uint32_t*)(p + e);
        } else {
          const uint32_t h = *(const __attribute__((address_space(1))) uint16_t*)(p + e);
          w[e >> 1] = (e & 1) ? w[e >> 1] | (h << 16) : h;
        }
      }
    }
  }
  __device__ __forceinline__ float at(int e) const {
    if constexpr (sizeof(KT) == 4) return __uint_as_float(w[e]);
    return half_bits_to_float((uint16_t)(w[e >> 1] >> (16 * (e & 1))));
  }
};

// ---------------------------------------------------------------- calibration
// Chunks of a unit's keys: one workgroup each, one round of the chip (a
// workgroup per CU) where the workspace holds as many.
static inline int cal_chunks(int U, int64_t n_cap) {
  int64_t c = 256 / U;
  const int64_t most = n_cap / 256 + 1;  // not under 256 keys each
  c = c < most ? c : most;
  return (int)(c < 1 ? 1 : c > kCalChunks ? kCalChunks : c);
}

__device__ __forceinline__ void chunk_range(int64_t nu, int nch, int c, int64_t* t0, int64_t* t1) {
  const int64_t cs = (nu + nch - 1) / nch;
  *t0 = (int64_t)c * cs < nu ? (int64_t)c * cs : nu;
  *t1 = *t0 + cs < nu ? *t0 + cs : nu;
}

// fp64 sums of y and y y^T over a chunk, y = k - (the unit's first key), in one
// pass over the keys: shifting by a key keeps the covariance sum(y y^T) / n -
// mean(y) mean(y)^T free of cancellation however far the mean lies from zero.
// v_mfma_f64_16x16x4_f64 over 4 tokens a step: with channel 8 i + b at index i
// of channel block b, the A and the B operand of block b are the same register
// (lane (i, token)), a lane loads its 8 channels as one run, and no operand goes
// through LDS.  Only the 36 tiles with bi <= bj are formed, 18 in each of a
// pair of waves (144 accumulator registers, two waves per SIMD); four pairs
// take every fourth step and add up through LDS in a fixed order.
// Bound by the fp64 matrix rate (the 36 tiles: 0.25 ms at 78.6 TFLOP/s for 8 x
// 131072 keys): 0.35 ms (full 128 x 128 products from LDS operands and a
// pass of its own for the mean, before: 1.93 ms).
constexpr int kCovTiles = 36;
constexpr int kCovHalf = kCovTiles / 2;
constexpr int kCovPairs = 4;
constexpr int kCovThreads = 2 * kCovPairs * kWave;
constexpr size_t kPartDoubles = (size_t)kCovTiles * 256 + kD;  // of one chunk: tiles as the lanes hold them, sums
static_assert((kD * kD + kCalChunks * kPartDoubles) * sizeof(double) <= kCalUnitBytes, "calibration workspace");
typedef double v4f64 __attribute__((ext_vector_type(4)));
typedef float v4f32 __attribute__((ext_vector_type(4)));

__host__ __device__ constexpr int tile_row(int t) {  // tile t of the upper triangle in row order: its block row
  int r = 0;
  while (t >= 8 - r) t -= 8 - r++;
  return r;
}
__host__ __device__ constexpr int tile_col(int t) {
  int r = 0;
  while (t >= 8 - r) t -= 8 - r++;
  return r + t;
}

template <int HALF, int T>
__device__ __forceinline__ void cov_tiles(v4f64 (&acc)[kCovHalf], const double (&y)[8]) {
  if constexpr (T < kCovHalf) {
    constexpr int r = tile_row(HALF * kCovHalf + T), c = tile_col(HALF * kCovHalf + T);
    acc[T] = __builtin_amdgcn_mfma_f64_16x16x4f64(y[r], y[c], acc[T], 0, 0, 0);
    cov_tiles<HALF, T + 1>(acc, y);
  }
}

template <int HALF, typename KT, bool VEC>
__device__ __forceinline__ void cov_wave(const KT* Ku, int64_t ld_tok, int64_t t0, int64_t t1, int pair, double* red,
                                         double* out) {
  const int lane = threadIdx.x & 63, x = lane & 15, g = lane >> 4;
  const KT* p = Ku + 8 * x;
  KeyRow<KT, VEC> row;
  double shift[8], sum[8];
  v4f64 acc[kCovHalf];
  row.load(p);  // the first key
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    shift[b] = (double)row.at(b);
    sum[b] = 0.0;
  }
#pragma unroll
  for (int t = 0; t < kCovHalf; ++t) acc[t] = (v4f64){0.0, 0.0, 0.0, 0.0};
  int64_t i = t0 + 4 * pair + g;
  if (t0 < t1) row.load(p + (i < t1 ? i : t1 - 1) * ld_tok);
  for (int64_t s = t0 + 4 * pair; s < t1; s += 4 * kCovPairs) {
    double y[8];
    const bool valid = i < t1;
#pragma unroll
    for (int b = 0; b < 8; ++b) y[b] = valid ? (double)row.at(b) - shift[b] : 0.0;
    i += 4 * kCovPairs;
    row.load(p + (i < t1 ? i : t1 - 1) * ld_tok);  // the next step's keys
    if (HALF == 0) {
#pragma unroll
      for (int b = 0; b < 8; ++b) sum[b] += y[b];
    }
    cov_tiles<HALF, 0>(acc, y);
  }
  // ---- add up the four pairs: the others hand theirs to the first, in order ----
  double* mine = red + HALF * (kCovHalf * 256 + kD) + lane;
  for (int w = 1; w < kCovPairs; ++w) {
    if (pair == w) {
#pragma unroll
      for (int t = 0; t < kCovHalf; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) mine[(4 * t + r) * 64] = acc[t][r];
      if (HALF == 0) {
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          sum[b] += __shfl_xor(sum[b], 16, kWave);
          sum[b] += __shfl_xor(sum[b], 32, kWave);
          if (g == 0) red[kCovHalf * 256 + 8 * x + b] = sum[b];
        }
      }
    }
    __syncthreads();
    if (pair == 0) {
#pragma unroll
      for (int t = 0; t < kCovHalf; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[t][r] += mine[(4 * t + r) * 64];
      if (HALF == 0) {
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          if (w == 1) {
            sum[b] += __shfl_xor(sum[b], 16, kWave);
            sum[b] += __shfl_xor(sum[b], 32, kWave);
          }
          sum[b] += red[kCovHalf * 256 + 8 * x + b];
        }
      }
    }
    __syncthreads();
  }
  if (pair == 0) {
#pragma unroll
    for (int t = 0; t < kCovHalf; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) out[(HALF * kCovHalf + t) * 256 + r * 64 + lane] = acc[t][r];
    if (HALF == 0 && g == 0) {
#pragma unroll
      for (int b = 0; b < 8; ++b) out[kCovTiles * 256 + 8 * x + b] = sum[b];
    }
  }
}

template <typename KT, bool VEC>
__global__ __launch_bounds__(kCovThreads, 2) void klt_cov_kernel(const KT* __restrict__ K, int64_t ld_tok,
                                                                int64_t ld_unit, const int64_t* __restrict__ n,
                                                                int64_t n_cap, double* __restrict__ part,
                                                                uint32_t* __restrict__ st) {
  __shared__ double red[2 * (kCovHalf * 256 + kD)];
  const int c = blockIdx.x, u = blockIdx.y, nch = (int)gridDim.x, tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t nu = unit_tokens(n, u, n_cap, (c == 0 && tid == 0) ? st : nullptr);
  if (nu == 0) return;  // the reduction knows
  int64_t t0, t1;
  chunk_range(nu, nch, c, &t0, &t1);
  const KT* Ku = K + (int64_t)u * ld_unit;
  double* out = part + ((int64_t)u * nch + c) * kPartDoubles;
  if (wave & 1)
    cov_wave<1, KT, VEC>(Ku, ld_tok, t0, t1, wave >> 1, red, out);
  else
    cov_wave<0, KT, VEC>(Ku, ld_tok, t0, t1, wave >> 1, red, out);
}

// Covariance and mean of a unit from its chunks' sums, added in chunk order
// (tile blockIdx.x; thread (r, lane) as the accumulators lie: row r4 + 4 r of
// block bi, column of block bj).
template <typename KT>
__global__ __launch_bounds__(256) void klt_reduce_kernel(const KT* __restrict__ K, int64_t ld_unit,
                                                        const int64_t* __restrict__ n, int64_t n_cap, int nch,
                                                        const double* __restrict__ part, double* __restrict__ cov,
                                                        float* __restrict__ mu_out) {
  const int u = blockIdx.y, t = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int bi = tile_row(t), bj = tile_col(t);
  const int i = 8 * ((lane >> 4) + 4 * (tid >> 6)) + bi, j = 8 * (lane & 15) + bj;
  int64_t nu = n[u];
  if (nu < 0 || nu > n_cap) nu = 0;  // flagged by the covariance pass
  double s = 0.0, si = 0.0, sj = 0.0;
  if (nu > 0) {
    const double* pu = part + (int64_t)u * nch * kPartDoubles;
#pragma unroll 8
    for (int c = 0; c < nch; ++c) {
      s += pu[c * kPartDoubles + t * 256 + tid];
      si += pu[c * kPartDoubles + kCovTiles * 256 + i];
      sj += pu[c * kPartDoubles + kCovTiles * 256 + j];
    }
    const double inv = 1.0 / (double)nu;
    s *= inv;
    si *= inv;
    sj *= inv;
  }
  const double v = s - si * sj;
  cov[((int64_t)u * kD + i) * kD + j] = v;
  if (bi != bj) cov[((int64_t)u * kD + j) * kD + i] = v;
  if (i == j) mu_out[(int64_t)u * kD + i] = nu > 0 ? (float)((double)key_at(K + (int64_t)u * ld_unit + i) + si) : 0.0f;
}

// ---- eigen-decomposition: one-sided Jacobi on a Cholesky factor ----
// C + delta I = L L^T (pivoted, fp64; delta = 1e-7 of the trace keeps every
// column of L well above zero for a singular C and leaves the eigenvectors
// as they are).  Rotations of L's columns until all are orthogonal turn them
// into multiples of the eigenvectors: one 128 x 128 fp32 matrix, no separate
// basis, and only columns are ever combined, so a pair of columns stays in the
// registers of 8 lanes (16 rows each) and its dot product is 16 multiply-adds
// and three DPP additions.
//
// The order of rotations: the 128 columns are 16 blocks of 8; each of the 8
// waves holds two blocks, one as "top" and one as "bottom" columns, lane group i
// pairing top i with bottom i ^ r for r = 0 .. 7 (the bottom columns move
// between lane groups along a Gray code).  Then the blocks move to the next
// wave through LDS (circle method, 15 meetings a sweep); at the first meeting of
// a sweep the wave also pairs its 16 columns among themselves, by permlane
// swaps of half of the top with half of the bottom columns.
// What bounds it: the rotations' VALU work on one CU per unit (a sweep of 127
// rounds takes 49 us; 9 sweeps for the decaying spectrum measured) and the
// serial steps of the factorisation (about 0.11 ms).  8 units: 0.62 ms
// (two-sided Jacobi with matrix and basis in LDS, three barriers a round and 12
// fixed sweeps, before: 5.6 ms).
__device__ __forceinline__ float dpp_xor1(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));
}
__device__ __forceinline__ float dpp_xor2(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, true));
}
__device__ __forceinline__ float dpp_half_mirror(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, true));
}
// Sum over a group of 8 lanes, in every lane.
__device__ __forceinline__ float sum8(float v) {
  v = __fadd_rn(v, dpp_xor1(v));
  v = __fadd_rn(v, dpp_xor2(v));
  return __fadd_rn(v, dpp_half_mirror(v));
}

// Largest value of the wave, in every lane.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true));
  auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = max(r[0], r[1]);
  r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return max(r[0], r[1]);
}

// 1 / sqrt(x): the hardware's estimate and two Newton steps (x > 0).
__device__ __forceinline__ double rsqrt_f64(double x) {
  double y = __builtin_amdgcn_rsq(x);
#pragma unroll
  for (int i = 0; i < 2; ++i) y = __fma_rn(__dmul_rn(0.5, y), __fma_rn(-__dmul_rn(x, y), y, 1.0), y);
  return y;
}

constexpr int kColRows = 16;  // rows of a column per lane

// A column across 8 lanes: its values are scale * v, |column|^2 = norm.
struct JacobiCol {
  float v[kColRows], norm, scale, inv;
};

template <int M>
__device__ __forceinline__ float lane_xor(float v) {
  if constexpr (M == 8) return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xF, 0xF, true));
  return __shfl_xor(v, M, kWave);
}
template <int M>
__device__ __forceinline__ void move_col(JacobiCol& c) {
#pragma unroll
  for (int e = 0; e < kColRows; ++e) c.v[e] = lane_xor<M>(c.v[e]);
  c.norm = lane_xor<M>(c.norm);
  c.scale = lane_xor<M>(c.scale);
  c.inv = lane_xor<M>(c.inv);
}

// Top columns of the upper half of each 2M lanes against bottom columns of the lower half.
template <int M>
__device__ __forceinline__ void swap_halves(float& a, float& b) {
  if constexpr (M == 8) {
    const int t = __float_as_int(a);
    a = __int_as_float(__builtin_amdgcn_update_dpp(t, __float_as_int(b), 0x128, 0xF, 0xC, false));
    b = __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(b), t, 0x128, 0xF, 0x3, false));
  } else {
    const auto r = M == 32 ? __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false)
                           : __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
  }
}
template <int M>
__device__ __forceinline__ void swap_cols(JacobiCol& a, JacobiCol& b) {
#pragma unroll
  for (int e = 0; e < kColRows; ++e) swap_halves<M>(a.v[e], b.v[e]);
  swap_halves<M>(a.norm, b.norm);
  swap_halves<M>(a.scale, b.scale);
  swap_halves<M>(a.inv, b.inv);
}

// Rotate the pair (p, q) orthogonal; true if another sweep has to follow.  (Norms
// are at least delta, so a_pq above the skipped cosines keeps its square.)
__device__ __forceinline__ bool rotate_pair(JacobiCol& p, JacobiCol& q) {
  float d0 = 0.0f, d1 = 0.0f;
#pragma unroll
  for (int e = 0; e < kColRows; e += 2) {
    d0 = __fmaf_rn(p.v[e], q.v[e], d0);
    d1 = __fmaf_rn(p.v[e + 1], q.v[e + 1], d1);
  }
  const float apq = __fmul_rn(sum8(__fadd_rn(d0, d1)), __fmul_rn(p.scale, q.scale));
  // t = tan of the smaller rotation angle: 2 a_pq / (d + sign(d) sqrt(d^2 + 4 a_pq^2)), d = a_qq - a_pp
  const float d = __fsub_rn(q.norm, p.norm), a2 = __fadd_rn(apq, apq);
  const float r = __builtin_amdgcn_sqrtf(__fmaf_rn(a2, a2, __fmul_rn(d, d)));
  const float den = __fadd_rn(d, __builtin_copysignf(r, d));
  const float cos2 = __fmul_rn(apq, apq), len2 = __fmul_rn(p.norm, q.norm);
  const float t = cos2 < __fmul_rn(kJacobiSkip2, len2) ? 0.0f : __fmul_rn(a2, __builtin_amdgcn_rcpf(den));
  const float c = __builtin_amdgcn_rsqf(__fmaf_rn(t, t, 1.0f));
  const float fp = __fmul_rn(t, __fmul_rn(q.scale, p.inv)), fq = __fmul_rn(t, __fmul_rn(p.scale, q.inv));
#pragma unroll
  for (int e = 0; e < kColRows; ++e) {
    const float x = p.v[e];
    p.v[e] = __fmaf_rn(-fp, q.v[e], x);
    q.v[e] = __fmaf_rn(fq, x, q.v[e]);
  }
  const bool big = cos2 > __fmul_rn(kJacobiTol2, len2) || fabsf(t) > kJacobiTan;
  p.norm = __fmaf_rn(-t, apq, p.norm);
  q.norm = __fmaf_rn(t, apq, q.norm);
  const float ic = __fmul_rn(__fmaf_rn(t, t, 1.0f), c);  // 1 / c
  p.scale = __fmul_rn(p.scale, c);
  q.scale = __fmul_rn(q.scale, c);
  p.inv = __fmul_rn(p.inv, ic);
  q.inv = __fmul_rn(q.inv, ic);
  return big;
}

// What the decomposition's kernels hand on of a unit (in the chunks' sums' place).
struct alignas(256) EigUnit {
  float basis[kD * kD];    // unit columns, row-major
  float refined[kD * kD];  // after the refinement
  double approx[kD];       // eigenvalues to fp32 rounding
  float lam[kD];           // Rayleigh quotients
};
static_assert(kD * kD * sizeof(double) + sizeof(EigUnit) <= kCalUnitBytes, "calibration workspace");

// A basis in LDS as rows: every 4 rows shift their 4-column groups, so that a
// column's reads use other banks.
__device__ __forceinline__ int basis_col(int row, int col) { return col ^ (4 * ((row >> 2) & 7)); }

// Columns in LDS: 128 rows each; the 32-row quarters of odd columns change
// places in pairs, so that two columns' 16-byte reads use all banks.
__device__ __forceinline__ int col_addr(int col, int quarter, int li) {
  return col * kD + ((quarter ^ (col & 1)) << 5) + 4 * li;
}
__device__ __forceinline__ void load_col(const float* X, int col, int li, JacobiCol& c) {
  float n = 0.0f;
#pragma unroll
  for (int i = 0; i < kColRows / 4; ++i) {
    const float4 v = *reinterpret_cast<const float4*>(&X[col_addr(col, i, li)]);
    c.v[4 * i] = v.x; c.v[4 * i + 1] = v.y; c.v[4 * i + 2] = v.z; c.v[4 * i + 3] = v.w;
  }
#pragma unroll
  for (int e = 0; e < kColRows; ++e) n = __fmaf_rn(c.v[e], c.v[e], n);
  c.norm = sum8(n);
  c.scale = c.inv = 1.0f;
}
__device__ __forceinline__ void store_col(float* X, int col, int li, const JacobiCol& c) {
#pragma unroll
  for (int i = 0; i < kColRows / 4; ++i)
    *reinterpret_cast<float4*>(&X[col_addr(col, i, li)]) =
        make_float4(__fmul_rn(c.v[4 * i], c.scale), __fmul_rn(c.v[4 * i + 1], c.scale),
                    __fmul_rn(c.v[4 * i + 2], c.scale), __fmul_rn(c.v[4 * i + 3], c.scale));
}

__global__ __launch_bounds__(kEigThreads, 2) void klt_eig_kernel(const double* __restrict__ cov, EigUnit* __restrict__ eig) {
  __shared__ __attribute__((aligned(16))) float X[2][kD * kD];  // columns; at the end one holds the basis as rows
  __shared__ double colj[kD], diag[kD];
  __shared__ int again[2];
  const int u = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double* Cu = cov + (int64_t)u * kD * kD;
  // thread (rg, cg) owns rows 8 rg .., columns 4 cg .. of what is left of the matrix
  const int rg = tid >> 5, cg = tid & 31;
  double a[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const v4f64 v = *reinterpret_cast<const v4f64*>(Cu + (8 * rg + i) * kD + 4 * cg);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      a[i][j] = v[j];
      if (8 * rg + i == 4 * cg + j) diag[8 * rg + i] = a[i][j];
    }
  }
  __syncthreads();
  double tr = diag[lane] + diag[lane + 64];
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) tr += __shfl_xor(tr, m, kWave);
  EigUnit& out = eig[u];
  if (tr == 0.0) {  // no keys, or all equal: every basis is one, the identity is given
    for (int e = tid; e < kD * kD; e += kEigThreads) out.basis[e] = e / kD == e % kD ? 1.0f : 0.0f;
    if (tid < kD) out.approx[tid] = 0.0;
    return;
  }
  // ---- pivoted Cholesky of C / trace + delta I; the factor's column k goes to X[0] ----
  const double itr = 1.0 / tr;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) a[i][j] = a[i][j] * itr + (8 * rg + i == 4 * cg + j ? kCholShift : 0.0);
  __syncthreads();
  double dg = 0.0;  // thread x < 128: what is left of diagonal x, negative once used
  if (tid < kD) {
    dg = diag[tid] * itr + kCholShift;
    diag[tid] = dg;
  }
  __syncthreads();
  for (int k = 0; k < kD; ++k) {
    // the largest diagonal (to 16 mantissa bits) is the pivot; every wave finds it
    uint32_t key = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const double v = diag[lane + 64 * h];
      const uint32_t kk = v < 0.0 ? 0u : (__float_as_uint((float)v) & 0x7FFFFF80u) | (uint32_t)(lane + 64 * h);
      key = key > kk ? key : kk;
    }
    key = wave_max_u32(key);
    const int j = __builtin_amdgcn_readfirstlane((int)(key & 127u));
    if (cg == (j >> 2)) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const double a0 = a[i][0], a1 = a[i][1], a2 = a[i][2], a3 = a[i][3];  // values: no indexing of registers
        const double lo = (j & 1) ? a1 : a0, hi = (j & 1) ? a3 : a2;
        colj[8 * rg + i] = (j & 2) ? hi : lo;
      }
    }
    __syncthreads();
    const double is = rsqrt_f64(colj[j]);
    double lr[8], lc[4];
#pragma unroll
    for (int i = 0; i < 8; ++i) lr[i] = colj[8 * rg + i] * is;
#pragma unroll
    for (int i = 0; i < 4; ++i) lc[i] = colj[4 * cg + i] * is;
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) a[i][jj] = __fma_rn(-lr[i], lc[jj], a[i][jj]);
    if (tid < kD) {
      const double l = dg < 0.0 ? 0.0 : colj[tid] * is;  // rows used before hold nothing
      X[0][col_addr(k, tid >> 5, 0) + (tid & 31)] = (float)l;
      dg = tid == j ? -1.0 : dg < 0.0 ? dg : fmax(dg - l * l, 0.0);
      diag[tid] = dg;
    }
    __syncthreads();
  }
  // ---- Jacobi sweeps ----
  const int gi = lane >> 3, li = lane & 7;
  // slots of this wave's blocks now, and where they go after a meeting
  const int s0 = wave, s1 = 15 - wave;
  const int t0 = s0 == 0 ? 0 : s0 + 1, t1 = s1 == 15 ? 1 : s1 + 1;
  if (tid < 2) again[tid] = 0;
  int buf = 0;
  for (int sweep = 0; sweep < kJacobiSweeps; ++sweep) {
    bool big = false;
    for (int meet = 0; meet < 15; ++meet) {
      JacobiCol p, q;
      load_col(X[buf], 8 * s0 + gi, li, p);
      load_col(X[buf], 8 * s1 + gi, li, q);
      big |= rotate_pair(p, q);
      move_col<8>(q);
      big |= rotate_pair(p, q);
      move_col<16>(q);
      big |= rotate_pair(p, q);
      move_col<8>(q);
      big |= rotate_pair(p, q);
      move_col<32>(q);
      big |= rotate_pair(p, q);
      move_col<8>(q);
      big |= rotate_pair(p, q);
      move_col<16>(q);
      big |= rotate_pair(p, q);
      move_col<8>(q);
      big |= rotate_pair(p, q);
      if (meet == 0) {  // the pairs inside the two blocks: 4 + 2 + 1 rounds
        swap_cols<32>(p, q);
        big |= rotate_pair(p, q);
        move_col<8>(q);
        big |= rotate_pair(p, q);
        move_col<16>(q);
        big |= rotate_pair(p, q);
        move_col<8>(q);
        big |= rotate_pair(p, q);
        swap_cols<16>(p, q);
        big |= rotate_pair(p, q);
        move_col<8>(q);
        big |= rotate_pair(p, q);
        swap_cols<8>(p, q);
        big |= rotate_pair(p, q);
      }
      buf ^= 1;
      store_col(X[buf], 8 * t0 + gi, li, p);
      store_col(X[buf], 8 * t1 + gi, li, q);
      if (meet == 14 && __ballot(big) && lane == 0) again[sweep & 1] = 1;
      __syncthreads();
    }
    if (again[sweep & 1] == 0) break;  // nothing was left to rotate but what this sweep did
    if (tid == 0) again[(sweep & 1) ^ 1] = 0;
  }
  __syncthreads();
  // ---- unit columns, as rows of the basis (through the other buffer), and their
  // eigenvalues to fp32 rounding ----
  const float* Xf = X[buf];
  float* Vs = X[buf ^ 1];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int col = 8 * wave + gi + 64 * h;
    double s = 0.0;
    float v[kColRows];
#pragma unroll
    for (int e = 0; e < kColRows; ++e) {
      v[e] = Xf[col_addr(col, e >> 2, li) + (e & 3)];
      s = __fma_rn((double)v[e], (double)v[e], s);
    }
#pragma unroll
    for (int m = 1; m < 8; m <<= 1) s += __shfl_xor(s, m, kWave);
    const double is = 1.0 / sqrt(s);
#pragma unroll
    for (int e = 0; e < kColRows; ++e) {
      const int row = 32 * (e >> 2) + 4 * li + (e & 3);
      Vs[row * kD + basis_col(row, col)] = (float)((double)v[e] * is);
    }
    if (li == 0) out.approx[col] = (s - kCholShift) * tr;
  }
  __syncthreads();
  for (int e = tid; e < kD * kD; e += kEigThreads) out.basis[e] = Vs[(e / kD) * kD + basis_col(e / kD, e % kD)];
}

// ---- eigenvalues, and one step of Ogita and Aishima's refinement ("Iterative
// refinement for symmetric eigenvalue decomposition", 2018).  The rotations leave
// the rounding of their 1000 fp32 steps: |V^T V - I|_F 5e-5 and an off-diagonal of
// V^T C V of 7e-6 of |C|_F.  With R = I - V^T V and S = V^T C V in fp64,
//   V <- V (I + R / 2 + X),  X_ij = (S_ij + (l_i + l_j) R_ij / 2) / (l_j - l_i),
// leaves 4e-7 and 4e-8 (under 2e-6 where many eigenvalues are close), the rounding
// of V's entries.  X is left out
// where it is not small: close eigenvalues, whose vectors may be any of their plane.
// Workgroup x takes columns 16 x .. 16 x + 15 and wave t the rows 16 t .. of C V (C is
// symmetric: its rows serve as the A operand's columns), R, S and the result; C V goes
// through LDS as the B operand of S.  Bound by the latency of its operands: 16 us for 8
// units (on the CU of the kernel above 22, and its code cost the rotations a tenth of
// their time).
constexpr int kRefThreads = 512;
constexpr int kRefSteps = kD / 4;
__global__ __launch_bounds__(kRefThreads) void klt_refine_kernel(const double* __restrict__ cov, EigUnit* __restrict__ eig) {
  __shared__ __attribute__((aligned(16))) float Vs[kD * kD];
  __shared__ double cv[kD * 16], la[kD];
  __shared__ float E[kD * 16];
  const int u = blockIdx.y, tid = threadIdx.x, lane = tid & 63, i16 = lane & 15, g = lane >> 4, t = tid >> 6;
  const int c = 16 * (int)blockIdx.x + i16;
  const double* Cu = cov + (int64_t)u * kD * kD;
  EigUnit& out = eig[u];
  double cu[kRefSteps];
#pragma unroll
  for (int s = 0; s < kRefSteps; ++s) cu[s] = Cu[(4 * s + g) * kD + 16 * t + i16];
#pragma unroll
  for (int x = 0; x < kD * kD / 4 / kRefThreads; ++x) {
    const int e = 4 * (tid + x * kRefThreads), row = e / kD;
    *reinterpret_cast<float4*>(&Vs[row * kD + basis_col(row, e % kD)]) = *reinterpret_cast<const float4*>(&out.basis[e]);
  }
  if (tid < kD) la[tid] = out.approx[tid];
  __syncthreads();
  auto at = [&](int row, int col) { return Vs[row * kD + basis_col(row, col)]; };
  v4f64 w = {0.0, 0.0, 0.0, 0.0}, rr = w, ss = w;
#pragma unroll
  for (int s = 0; s < kRefSteps; ++s) w = __builtin_amdgcn_mfma_f64_16x16x4f64(cu[s], (double)at(4 * s + g, c), w, 0, 0, 0);
#pragma unroll
  for (int r = 0; r < 4; ++r) cv[(16 * t + 4 * r + g) * 16 + i16] = w[r];
  __syncthreads();
#pragma unroll 8
  for (int k = g; k < kD; k += 4) {
    const double y = (double)at(k, 16 * t + i16);
    rr = __builtin_amdgcn_mfma_f64_16x16x4f64(y, (double)at(k, c), rr, 0, 0, 0);
    ss = __builtin_amdgcn_mfma_f64_16x16x4f64(y, cv[k * 16 + i16], ss, 0, 0, 0);
  }
  double tr = la[lane] + la[lane + 64];
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) tr += __shfl_xor(tr, m, kWave);
  const double lj = la[c];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = 16 * t + 4 * r + g;
    const double h = 0.5 * ((i == c ? 1.0 : 0.0) - rr[r]), gap = lj - la[i];
    const double q = __fma_rn(la[i] + lj, h, ss[r]);
    E[i * 16 + i16] = (float)(fabs(gap) > kRefineGap * tr && fabs(q) < kRefineMax * fabs(gap) ? h + q / gap : h);
    // The Rayleigh quotient is that of the refined vector too (the step is of first
    // order).  A covariance has no negative eigenvalue: a null direction's quotient is
    // rounding error of either sign, and a negative variance is no input to the depth
    // allocation (the test leaves a NaN as it is).
    if (i == c) out.lam[c] = ss[r] < 0.0 ? 0.0f : (float)(ss[r] / rr[r]);
  }
  __syncthreads();
  v4f32 d = {0.0f, 0.0f, 0.0f, 0.0f};  // V (R / 2 + X), a correction of 1e-6, in fp32
#pragma unroll 8
  for (int k = g; k < kD; k += 4) d = __builtin_amdgcn_mfma_f32_16x16x4f32(at(16 * t + i16, k), E[k * 16 + i16], d, 0, 0, 0);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = 16 * t + 4 * g + r;
    out.refined[row * kD + c] = __fadd_rn(at(row, c), d[r]);
  }
}

// Columns by eigenvalue (descending, ties by position), each with its
// largest-magnitude entry (the first of equal ones) positive.  Four threads a column.
__global__ __launch_bounds__(kEigThreads) void klt_order_kernel(const EigUnit* __restrict__ eig, float* __restrict__ V_out,
                                                                float* __restrict__ lam_out) {
  __shared__ float Vs[kD * (kD + 1)], lam[kD];
  __shared__ int order[kD];
  const int u = blockIdx.x, tid = threadIdx.x;
  const EigUnit& in = eig[u];
#pragma unroll
  for (int x = 0; x < kD * kD / kEigThreads; ++x) {
    const int e = tid + x * kEigThreads;
    Vs[(e / kD) * (kD + 1) + e % kD] = in.refined[e];
  }
  if (tid < kD) lam[tid] = in.lam[tid];
  __syncthreads();
  const int c = tid >> 2, part = tid & 3;
  const float lc = lam[c];
  int rank = 0, first = 0;
  float best = -1.0f, at = 0.0f;
#pragma unroll 8
  for (int i = 32 * part; i < 32 * part + 32; ++i) {
    rank += (lam[i] > lc) || (lam[i] == lc && i < c);
    const float v = Vs[i * (kD + 1) + c];
    if (fabsf(v) > best) {
      best = fabsf(v);
      at = v;
      first = i;
    }
  }
#pragma unroll
  for (int m = 1; m < 4; m <<= 1) {
    rank += __shfl_xor(rank, m, kWave);
    const float ob = __shfl_xor(best, m, kWave), oa = __shfl_xor(at, m, kWave);
    const int of = __shfl_xor(first, m, kWave);
    if (ob > best || (ob == best && of < first)) {
      best = ob;
      at = oa;
      first = of;
    }
  }
  if (part == 0) {
    order[rank & (kD - 1)] = at < 0.0f ? c | kD : c;
    lam_out[(int64_t)u * kD + (rank & (kD - 1))] = lc;
  }
  __syncthreads();
  float* Vo = V_out + (int64_t)u * kD * kD;
  for (int e = tid; e < kD * kD; e += kEigThreads) {
    const int o = order[e % kD];
    const float v = Vs[(e / kD) * (kD + 1) + (o & (kD - 1))];
    Vo[e] = (o & kD) ? -v : v;
  }
}

// ---------------------------------------------------------------- rotations
// The fixed order allows no fused multiply-add, so the contraction is 2 VALU
// operations per (token, j, channel) at best; everything else is kept out of
// the loop.  A wave owns 64 channels and holds its half of V in registers (lane
// = channel, 128 VGPRs); of a token row every 16 lanes hold a copy (8 channels a
// lane), and the multiply broadcasts d_j from lane j / 8 of each row by its
// DPP operand: no LDS, no scalar moves, four tokens' chains interleaved.
// 8 x 131072 fp16 keys: 0.98 ms, of which the two operations are 0.87 (V and
// the keys through LDS, one wave per SIMD, before: 2.70 ms).
// acc[t] += pr[t], then pr[t] = d[t] of lane X of each row of 16 times v.  The
// four additions stand first, so that a register written just before has the
// two wait states that a DPP read needs.
template <int X>
__device__ __forceinline__ void rot_step(float (&acc)[kRotTokens], float (&pr)[kRotTokens], float d0, float d1,
                                         float d2, float d3, float v) {
  static_assert(kRotTokens == 4, "one asm block per four tokens");
  asm("v_add_f32 %0, %0, %4\n\t"
      "v_add_f32 %1, %1, %5\n\t"
      "v_add_f32 %2, %2, %6\n\t"
      "v_add_f32 %3, %3, %7\n\t"
      "v_mul_f32_dpp %4, %8, %12 row_newbcast:%13 row_mask:0xf bank_mask:0xf\n\t"
      "v_mul_f32_dpp %5, %9, %12 row_newbcast:%13 row_mask:0xf bank_mask:0xf\n\t"
      "v_mul_f32_dpp %6, %10, %12 row_newbcast:%13 row_mask:0xf bank_mask:0xf\n\t"
      "v_mul_f32_dpp %7, %11, %12 row_newbcast:%13 row_mask:0xf bank_mask:0xf"
      : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2]), "+&v"(acc[3]), "+&v"(pr[0]), "+&v"(pr[1]), "+&v"(pr[2]),
        "+&v"(pr[3])
      : "v"(d0), "v"(d1), "v"(d2), "v"(d3), "v"(v), "n"(X));
}

template <int X>
__device__ __forceinline__ void rot_steps(const float (&d)[kRotTokens][8], const float (&v)[kD],
                                          float (&acc)[kRotTokens], float (&pr)[kRotTokens]) {
  if constexpr (X < 16) {
#pragma unroll
    for (int e = 0; e < 8; ++e) rot_step<X>(acc, pr, d[0][e], d[1][e], d[2][e], d[3][e], v[8 * X + e]);
    rot_steps<X + 1>(d, v, acc, pr);
  }
}

// INPLACE: out's rows are K's.  Both waves of a run read whole rows and each
// writes its own half of them, so neither may store a group of tokens before the
// other has read it: one barrier a group, between the two, with as many groups
// for every wave of the workgroup (a wave past its run's end re-reads a row and
// stores nothing).
template <typename KT, bool VEC, bool INPLACE>
__device__ __forceinline__ void rotate_keys(const KT* K, int64_t ld_tok, int64_t ld_unit, const int64_t* n,
                                            int64_t n_cap, const float* mu, const float* V, float* out, int64_t ld_out,
                                            int chunk, uint32_t* st) {
  const int u = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t nu = unit_tokens(n, u, n_cap, (blockIdx.x == 0 && tid == 0) ? st : nullptr);
  // two waves (the channel halves) share a run of chunk / 2 tokens
  const int c = 64 * (wave & 1) + lane, x = lane & 15;
  const int64_t b0 = (int64_t)blockIdx.x * chunk, t0 = b0 + (wave >> 1) * (chunk / 2);
  const int64_t t1 = t0 + chunk / 2 < nu ? t0 + chunk / 2 : nu;
  if ((INPLACE ? b0 : t0) >= nu) return;
  // in place the workgroup's first run, which is no shorter, sets the count of groups
  const int64_t end = !INPLACE ? t1 : t0 + (nu - b0 < chunk / 2 ? nu - b0 : chunk / 2);
  const KT* Ku = K + (int64_t)u * ld_unit + 8 * x;
  KeyRow<KT, VEC> row[kRotTokens];
#pragma unroll
  for (int t = 0; t < kRotTokens; ++t) row[t].load(Ku + (t0 + t < t1 ? t0 + t : t1 - 1) * ld_tok);
  float m[8], v[kD];
#pragma unroll
  for (int e = 0; e < 8; ++e) m[e] = mu[(int64_t)u * kD + 8 * x + e];
  const float* Vu = V + (int64_t)u * kD * kD + c;
#pragma unroll
  for (int j = 0; j < kD; ++j) v[j] = Vu[j * kD];
  float* Ou = out + (int64_t)u * ld_out + c;
  for (int64_t i = t0; i < end; i += kRotTokens) {
    float d[kRotTokens][8], acc[kRotTokens], pr[kRotTokens];
#pragma unroll
    for (int t = 0; t < kRotTokens; ++t) {
      acc[t] = pr[t] = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) d[t][e] = __fsub_rn(row[t].at(e), m[e]);
    }
    // the next tokens' rows are in flight while these are rotated (past the end: the last row again)
#pragma unroll
    for (int t = 0; t < kRotTokens; ++t) {
      const int64_t nx = i + kRotTokens + t;
      row[t].load(Ku + (nx < t1 ? nx : t1 - 1) * ld_tok);
    }
    rot_steps<0>(d, v, acc, pr);
    if constexpr (INPLACE) __syncthreads();
#pragma unroll
    for (int t = 0; t < kRotTokens; ++t)
      if (i + t < t1) Ou[(i + t) * kD] = __fadd_rn(acc[t], pr[t]);
  }
}

template <typename KT, bool VEC>
__global__ __launch_bounds__(kRotThreads, 2) void klt_rotate_keys_kernel(const KT* __restrict__ K, int64_t ld_tok,
                                                                        int64_t ld_unit, const int64_t* __restrict__ n,
                                                                        int64_t n_cap, const float* __restrict__ mu,
                                                                        const float* __restrict__ V,
                                                                        float* __restrict__ out, int64_t ld_out,
                                                                        int chunk, uint32_t* __restrict__ st) {
  rotate_keys<KT, VEC, false>(K, ld_tok, ld_unit, n, n_cap, mu, V, out, ld_out, chunk, st);
}

template <bool VEC>
__global__ __launch_bounds__(kRotThreads, 2) void klt_rotate_in_place_kernel(float* K, int64_t ld_unit, const int64_t* n,
                                                                            int64_t n_cap, const float* mu,
                                                                            const float* V, int64_t ld_out, int chunk,
                                                                            uint32_t* st) {
  rotate_keys<float, VEC, true>(K, kD, ld_unit, n, n_cap, mu, V, K, ld_out, chunk, st);
}

// One workgroup per unit: V and the unit's queries are staged in LDS with all
// loads in flight, then thread (h, c) forms its dot product from LDS.
__global__ __launch_bounds__(kMaxG * kD) void klt_rotate_q_kernel(const void* __restrict__ q, fathom_dtype qdt,
                                                                 int G, const float* __restrict__ V,
                                                                 float* __restrict__ out) {
  __shared__ float4 Vs4[kD * kD / 4];
  __shared__ float qs[kMaxG * kD];
  const int u = blockIdx.x, tid = threadIdx.x, h = tid / kD, c = tid % kD;
  const float4* Vu = reinterpret_cast<const float4*>(V + (int64_t)u * kD * kD);
  float4 r[kD * kD / 4 / (kMaxG * kD)];
#pragma unroll
  for (int x = 0; x < kD * kD / 4 / (kMaxG * kD); ++x) r[x] = Vu[tid + x * kMaxG * kD];
  const int64_t qo = (int64_t)u * G * kD;
  if (h < G) qs[tid] = load_q(q, qdt, qo + tid);
#pragma unroll
  for (int x = 0; x < kD * kD / 4 / (kMaxG * kD); ++x) Vs4[tid + x * kMaxG * kD] = r[x];
  __syncthreads();
  if (h >= G) return;
  const float* Vs = reinterpret_cast<const float*>(Vs4);
  float acc = 0.0f;
  for (int j = 0; j < kD; ++j) acc = __fadd_rn(acc, __fmul_rn(qs[h * kD + j], Vs[j * kD + c]));
  out[qo + tid] = acc;
}

// ---------------------------------------------------------------- launches
fathom_status launch_klt_calibrate(const void* K, fathom_dtype kdt, int64_t ld_tok, int64_t ld_unit,
                                   const int64_t* n, int64_t n_cap, int U, float* mu, float* V, float* lam, void* ws,
                                   uint32_t* st, hipStream_t s) {
  if (U == 0) return FATHOM_OK;
  double* cov = reinterpret_cast<double*>(ws);
  double* part = cov + (size_t)U * kD * kD;
  const int nch = cal_chunks(U, n_cap);
  const dim3 g((unsigned)nch, (unsigned)U), gr((unsigned)kCovTiles, (unsigned)U);
  // 16-byte loads of a lane's 8 channels when every row start is 16-byte aligned
  const int64_t vec = kdt == FATHOM_F32 ? 4 : 8;
  const bool al = (reinterpret_cast<uintptr_t>(K) & 15) == 0 && ld_tok % vec == 0 && ld_unit % vec == 0;
  const float* Kf = reinterpret_cast<const float*>(K);
  const __half* Kh = reinterpret_cast<const __half*>(K);
  if (kdt == FATHOM_F32 && al)
    hipLaunchKernelGGL((klt_cov_kernel<float, true>), g, dim3(kCovThreads), 0, s, Kf, ld_tok, ld_unit, n, n_cap, part, st);
  else if (kdt == FATHOM_F32)
    hipLaunchKernelGGL((klt_cov_kernel<float, false>), g, dim3(kCovThreads), 0, s, Kf, ld_tok, ld_unit, n, n_cap, part, st);
  else if (al)
    hipLaunchKernelGGL((klt_cov_kernel<__half, true>), g, dim3(kCovThreads), 0, s, Kh, ld_tok, ld_unit, n, n_cap, part, st);
  else
    hipLaunchKernelGGL((klt_cov_kernel<__half, false>), g, dim3(kCovThreads), 0, s, Kh, ld_tok, ld_unit, n, n_cap, part, st);
  if (kdt == FATHOM_F32)
    hipLaunchKernelGGL(klt_reduce_kernel<float>, gr, dim3(256), 0, s, Kf, ld_unit, n, n_cap, nch, part, cov, mu);
  else
    hipLaunchKernelGGL(klt_reduce_kernel<__half>, gr, dim3(256), 0, s, Kh, ld_unit, n, n_cap, nch, part, cov, mu);
  EigUnit* eig = reinterpret_cast<EigUnit*>(part);  // the chunks' sums are read by then
  hipLaunchKernelGGL(klt_eig_kernel, dim3((unsigned)U), dim3(kEigThreads), 0, s, cov, eig);
  hipLaunchKernelGGL(klt_refine_kernel, dim3(kD / 16, (unsigned)U), dim3(kRefThreads), 0, s, cov, eig);
  hipLaunchKernelGGL(klt_order_kernel, dim3((unsigned)U), dim3(kEigThreads), 0, s, eig, V, lam);
  FATHOM_LAUNCH_CHECK();
  return FATHOM_OK;
}

fathom_status launch_klt_rotate_keys(const void* K, fathom_dtype kdt, int64_t ld_tok, int64_t ld_unit,
                                     const int64_t* n, int64_t n_cap, int U, const float* mu, const float* V,
                                     float* out, int64_t ld_out, uint32_t* st, hipStream_t s) {
  if (U == 0 || n_cap == 0) return FATHOM_OK;
  // Tokens per workgroup: about 2048 workgroups (four rounds of two per CU, so
  // that one's loads of V run beside another's rotations and ragged units even
  // out), of 16 to 512 tokens (at 512 a wave's 32 KB of V is 1 % of its time).
  // One round only: 131072 keys 140 us against 134, 4 x 8346 keys 47 against 45.
  int64_t chunk = (n_cap * U / 2048 + 15) & ~(int64_t)15;
  chunk = chunk < 16 ? 16 : chunk > 512 ? 512 : chunk;
  const dim3 g((unsigned)((n_cap + chunk - 1) / chunk), (unsigned)U);
  // 16-byte row loads when every row start is 16-byte aligned
  const int64_t vec = kdt == FATHOM_F32 ? 4 : 8;
  const bool al = (reinterpret_cast<uintptr_t>(K) & 15) == 0 && ld_tok % vec == 0 && ld_unit % vec == 0;
  const float* Kf = reinterpret_cast<const float*>(K);
  const __half* Kh = reinterpret_cast<const __half*>(K);
  // keys rotated into their own rows: 8 x 131072 keys 931 us in place, 993 into rows of their own
  if (kdt == FATHOM_F32 && Kf == out && ld_tok == kD) {
    if (al)
      hipLaunchKernelGGL(klt_rotate_in_place_kernel<true>, g, dim3(kRotThreads), 0, s, out, ld_unit, n, n_cap, mu, V,
                         ld_out, (int)chunk, st);
    else
      hipLaunchKernelGGL(klt_rotate_in_place_kernel<false>, g, dim3(kRotThreads), 0, s, out, ld_unit, n, n_cap, mu, V,
                         ld_out, (int)chunk, st);
  } else if (kdt == FATHOM_F32 && al)
    hipLaunchKernelGGL((klt_rotate_keys_kernel<float, true>), g, dim3(kRotThreads), 0, s, Kf, ld_tok, ld_unit, n, n_cap,
                       mu, V, out, ld_out, (int)chunk, st);
  else if (kdt == FATHOM_F32)
    hipLaunchKernelGGL((klt_rotate_keys_kernel<float, false>), g, dim3(kRotThreads), 0, s, Kf, ld_tok, ld_unit, n,
                       n_cap, mu, V, out, ld_out, (int)chunk, st);
  else if (al)
    hipLaunchKernelGGL((klt_rotate_keys_kernel<__half, true>), g, dim3(kRotThreads), 0, s, Kh, ld_tok, ld_unit, n,
                       n_cap, mu, V, out, ld_out, (int)chunk, st);
  else
    hipLaunchKernelGGL((klt_rotate_keys_kernel<__half, false>), g, dim3(kRotThreads), 0, s, Kh, ld_tok, ld_unit, n,
                       n_cap, mu, V, out, ld_out, (int)chunk, st);
  FATHOM_LAUNCH_CHECK();
  return FATHOM_OK;
}

fathom_status launch_klt_rotate_q(const void* q, fathom_dtype qdt, int U, int G, const float* V, float* out,
                                  hipStream_t s) {
  if (U == 0) return FATHOM_OK;
  hipLaunchKernelGGL(klt_rotate_q_kernel, dim3((unsigned)U), dim3(kMaxG * kD), 0, s, q, qdt, G, V, out);
  FATHOM_LAUNCH_CHECK();
  return FATHOM_OK;
}

}  // namespace fathom
