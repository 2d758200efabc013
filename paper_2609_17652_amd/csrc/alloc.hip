// fathom_alloc_depths: Sec. 3.3, Eq. (g) and Eq. (wf) (water-filling), and the
// grouped top-r channel rule of Sec. 2 (uniform-depth mode).
//
// One wave per unit; lane l owns channels l and l + 64.  The water line is
// found exactly: the 4D candidates g_j * 2^-(2m-1) are non-negative, so their
// IEEE bit patterns order like their values, and a bitwise search over the
// pattern (each step a wave-wide count from ballots) yields the (B+1)-th
// largest candidate with no log, exp or rounding -- a bisection on log(theta).
// Each candidate is an fp32 value times a power of two between 2^-156 and
// 2^127: 23 mantissa bits and a 9-bit exponent, one 32-bit key.  The search
// starts at the highest bit in which candidates differ and ends as soon as
// exactly B + 1 of them remain, whose smallest is the answer (about 12 of the
// 32 steps for continuous data).  Latency bound: one wave's loads, then that
// serial chain.  8 units: 4.4 us, of which 2 are the launch (64-bit keys, 34 steps, before: 5.9).
#include "common.hpp"

namespace fathom {

template <fathom_dtype QDT>
__device__ __forceinline__ float load_q_as(const void* q, int64_t i) {
  if (QDT == FATHOM_F16)
    return __half2float(__ushort_as_half(((const __attribute__((address_space(1))) uint16_t*)q)[i]));
  return ((const __attribute__((address_space(1))) float*)q)[i];
}

// Outside the defined inputs, in the order of their bit patterns as doubles: above
// every candidate.
constexpr uint32_t kKeyInf = 0xFFFFFFFDu, kKeyNan = 0xFFFFFFFEu, kKeyNeg = 0xFFFFFFFFu;
constexpr int kExpBias = 160;  // a candidate's exponent, -156 .. 126, plus this fits 9 bits and is not 0

__device__ __forceinline__ uint32_t wave_max_u(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true));  // row_half_mirror
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true));  // row_mirror
  return max(max((uint32_t)__builtin_amdgcn_readlane((int)v, 0), (uint32_t)__builtin_amdgcn_readlane((int)v, 16)),
             max((uint32_t)__builtin_amdgcn_readlane((int)v, 32), (uint32_t)__builtin_amdgcn_readlane((int)v, 48)));
}
__device__ __forceinline__ uint32_t wave_or(uint32_t v) {
  v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);
  v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);
  v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);
  v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true);
  return (uint32_t)(__builtin_amdgcn_readlane((int)v, 0) | __builtin_amdgcn_readlane((int)v, 16) |
                    __builtin_amdgcn_readlane((int)v, 32) | __builtin_amdgcn_readlane((int)v, 48));
}

template <fathom_dtype QDT>
__global__ __launch_bounds__(kWave) void alloc_waterfill_kernel(const void* __restrict__ q, int G,
                                                                const float* __restrict__ var,
                                                                int B, uint8_t* __restrict__ depths,
                                                                float* __restrict__ theta,
                                                                uint32_t* __restrict__ st) {
  const int u = blockIdx.x, lane = threadIdx.x;
  __builtin_assume(G >= 1 && G <= kMaxG);
  // every load is issued before the first use: heads past G re-read head G-1
  const float v0 = var[(int64_t)u * kD + lane], v1 = var[(int64_t)u * kD + lane + 64];
  float x[2][kMaxG];
#pragma unroll
  for (int h = 0; h < kMaxG; ++h) {
    const int64_t row = ((int64_t)u * G + min(h, G - 1)) * kD;
    x[0][h] = load_q_as<QDT>(q, row + lane);
    x[1][h] = load_q_as<QDT>(q, row + lane + 64);
  }
  uint32_t key[2][4];
  uint32_t flags = 0;
  uint32_t any = 0, all = 0xFFFFFFFFu;  // bits set in some, in every candidate
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    float s = 0.0f;  // heads in ascending order
#pragma unroll
    for (int h = 0; h < kMaxG; ++h)
      if (h < G) s = __fadd_rn(s, __fmul_rn(x[r][h], x[r][h]));
    const float g = __fmul_rn(s, r ? v1 : v0);
    const bool fine = g >= 0.0f && g <= 3.402823466e38f;
    if (!fine) flags |= FATHOM_DEV_NONFINITE;
    const uint32_t odd = g != g ? kKeyNan : g < 0.0f ? kKeyNeg : kKeyInf;
    const uint64_t w = (uint64_t)__double_as_longlong((double)g);  // subnormal g is normal here
    const uint32_t k0 = (uint32_t)(w >> 29) - ((uint32_t)(1023 - kExpBias) << 23);  // (exponent + kExpBias, mantissa)
#pragma unroll
    for (int m = 1; m <= 4; ++m) {
      key[r][m - 1] = !fine ? odd : g == 0.0f ? 0u : k0 - ((uint32_t)(2 * m - 1) << 23);
      any |= key[r][m - 1];
      all &= key[r][m - 1];
    }
  }
  // T = largest pattern with #{keys >= T} >= B + 1, i.e. the (B+1)-th largest key
  uint32_t T = 0;
  if (B < 4 * kD) {
    const uint32_t diff = wave_or(any) & wave_or(~all);
    T = wave_or(any) & ~diff;  // what every key has
    for (int bit = diff ? 31 - __builtin_clz(diff) : -1; bit >= 0; --bit) {
      const uint32_t cand = (T & ~((1u << bit) - 1u)) | (1u << bit);
      int c = 0;  // wave-wide count from ballots: no cross-lane data movement
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int m = 0; m < 4; ++m) c += __popcll(__ballot(key[r][m] >= cand));
      if (c >= B + 1) T = cand;
      if (c == B + 1) {  // the smallest of exactly these (as the largest complement)
        uint32_t low = 0;
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
          for (int m = 0; m < 4; ++m) low = max(low, key[r][m] >= cand ? ~key[r][m] : 0u);
        T = ~wave_max_u(low);
        break;
      }
    }
  }
  T = min(T, kKeyNan);  // a water line is no negative value: at NaN
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    int t = 0;
#pragma unroll
    for (int m = 0; m < 4; ++m) t += key[r][m] > T;
    depths[(int64_t)u * kD + lane + 64 * r] = (uint8_t)t;
  }
  if (lane == 0 && theta) {
    const uint64_t w = ((uint64_t)T + ((uint64_t)(1023 - kExpBias) << 23)) << 29;
    theta[u] = T == 0u         ? 0.0f
               : T == kKeyInf ? __builtin_huge_valf()
               : T == kKeyNan ? __builtin_nanf("")
                              : (float)__longlong_as_double((long long)w);
  }
  uint32_t f = flags;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) f |= __shfl_xor(f, m, kWave);
  if (lane == 0) set_status(st, f);
}

// Thread j ranks channel j against all others, whose weights it reads from LDS
// four at a time.  8 units: 6.2 us (one wave with two channels a lane and one
// weight a read, before: 10.8).
template <fathom_dtype QDT>
__global__ __launch_bounds__(kD) void alloc_topr_kernel(const void* __restrict__ q, int G, int r,
                                                        uint8_t* __restrict__ depths, float* __restrict__ theta,
                                                        uint32_t* __restrict__ st) {
  __shared__ __attribute__((aligned(16))) float w[kD];
  const int u = blockIdx.x, j = threadIdx.x;
  __builtin_assume(G >= 1 && G <= kMaxG);
  float x[kMaxG];  // every load issued before the first use: heads past G re-read head G - 1
#pragma unroll
  for (int h = 0; h < kMaxG; ++h) x[h] = load_q_as<QDT>(q, ((int64_t)u * G + min(h, G - 1)) * kD + j);
  float wj = 0.0f;  // heads in ascending order
#pragma unroll
  for (int h = 0; h < kMaxG; ++h)
    if (h < G) wj = __fadd_rn(wj, fabsf(x[h]));
  w[j] = wj;
  __syncthreads();
  int rank = 0;  // position of j in (w desc, j asc) order
#pragma unroll 8
  for (int i = 0; i < kD; i += 4) {
    const float4 v = *reinterpret_cast<const float4*>(&w[i]);
    rank += (v.x > wj) || (v.x == wj && i < j);
    rank += (v.y > wj) || (v.y == wj && i + 1 < j);
    rank += (v.z > wj) || (v.z == wj && i + 2 < j);
    rank += (v.w > wj) || (v.w == wj && i + 3 < j);
  }
  depths[(int64_t)u * kD + j] = rank < r ? 4 : 0;
  if (theta && rank == r - 1) theta[u] = wj;
  if (theta && r == 0 && j == 0) theta[u] = 0.0f;
  if (__ballot(!(wj <= 3.402823466e38f)) && (j & 63) == 0) set_status(st, FATHOM_DEV_NONFINITE);
}

fathom_status launch_alloc(const void* q, fathom_dtype qdt, int U, int G, const float* var,
                           fathom_mode mode, int budget_or_r, uint8_t* depths, float* theta,
                           uint32_t* st, hipStream_t s) {
  if (U == 0) return FATHOM_OK;
  if (mode == FATHOM_WATERFILL)
  {
    if (qdt == FATHOM_F16)
      hipLaunchKernelGGL(alloc_waterfill_kernel<FATHOM_F16>, dim3(U), dim3(kWave), 0, s, q, G, var,
                         budget_or_r, depths, theta, st);
    else
      hipLaunchKernelGGL(alloc_waterfill_kernel<FATHOM_F32>, dim3(U), dim3(kWave), 0, s, q, G, var,
                         budget_or_r, depths, theta, st);
  }
  else if (qdt == FATHOM_F16)
    hipLaunchKernelGGL(alloc_topr_kernel<FATHOM_F16>, dim3(U), dim3(kD), 0, s, q, G, budget_or_r, depths, theta, st);
  else
    hipLaunchKernelGGL(alloc_topr_kernel<FATHOM_F32>, dim3(U), dim3(kD), 0, s, q, G, budget_or_r, depths, theta, st);
  FATHOM_LAUNCH_CHECK();
  return FATHOM_OK;
}

}  // namespace fathom
