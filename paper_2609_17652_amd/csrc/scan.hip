// fathom_scan: Sec. 3.2-3.3 -- approximate scores from per-channel plane
// prefixes, all G query heads of a unit at once (the plan is shared by the
// group, so each plane word is read once for all G heads).
//
// A workgroup of 4 waves scores 16 consecutive blocks of one unit, 4 a wave (1
// a wave where the keys are few),
// lane i = key 64b + i.  The plane words of up to 32 active channels at a time
// are staged in LDS (runs of 128 bytes a row, every load of a stage in flight
// at once), split into halves so that one 16-byte broadcast read gives a lane
// the dwords of its wave's four blocks; per plane a lane then extracts its bit
// (two instructions), dequantises its key exactly, and every head accumulates
// one fused multiply-add in the documented order:
//   khat = (c^(t) + 1/2 - 2^(t-1)) * a16 * 2^(1-t)   (exact in fp32),
//   acc_h = fmaf(q_hj, khat, acc_h),  channels ascending, acc from +0.
// Bound by that VALU work (about 9 instructions a channel and key at 4 heads
// and 80 bits).  8 x 131072 keys at 80 bits, 4 heads: 34 us (one block a wave,
// its words fetched by dependent wave-uniform loads, before: 73 us).
#include "common.hpp"

namespace fathom {

constexpr int kScanThreads = 256;
constexpr int kScanWaves = kScanThreads / kWave;
constexpr int kScanChannels = 32;  // channels per stage

struct ScanPlan {
  int nact, ncell;
  uint32_t chan[kD];            // active channels ascending: j | t << 8 | first cell << 16
  uint16_t cell[kD * kPlanes];  // row j * 4 + p of each cell
};

// Active channels and their plane cells of one unit (128 threads' worth).
__device__ __forceinline__ void build_scan_plan(const uint8_t* __restrict__ d, ScanPlan& pl, int (*tot)[2]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int t = 0;
  if (tid < kD) t = d[tid] > kPlanes ? kPlanes : d[tid];  // depths above 4 read as 4
  const uint64_t lt = (1ull << lane) - 1;
  const uint64_t on = __ballot(t > 0), b0 = __ballot(t & 1), b1 = __ballot(t & 2), b2 = __ballot(t & 4);
  int a = __popcll(on & lt), c = __popcll(b0 & lt) + 2 * __popcll(b1 & lt) + 4 * __popcll(b2 & lt);
  if (tid < kD && lane == 0) {
    tot[wave][0] = __popcll(on);
    tot[wave][1] = __popcll(b0) + 2 * __popcll(b1) + 4 * __popcll(b2);
  }
  __syncthreads();
  if (wave == 1) {
    a += tot[0][0];
    c += tot[0][1];
  }
  if (t > 0) {
    pl.chan[a] = (uint32_t)tid | (uint32_t)t << 8 | (uint32_t)c << 16;
    for (int p = 0; p < t; ++p) pl.cell[c + p] = (uint16_t)(tid * kPlanes + p);
  }
  if (tid == 0) {
    pl.nact = tot[0][0] + tot[1][0];
    pl.ncell = tot[0][1] + tot[1][1];
  }
  __syncthreads();
}

template <int PW>
struct ScanRun {  // a wave's PW blocks: one LDS read
  typedef uint32_t words __attribute__((ext_vector_type(PW)));
  typedef float scales __attribute__((ext_vector_type(PW)));
};
template <>
struct ScanRun<1> {
  struct words { uint32_t v; __device__ uint32_t operator[](int) const { return v; } };
  struct scales { float v; __device__ float operator[](int) const { return v; } };
};

// One channel of T planes: the code bits, keys and heads of the wave's PW blocks.
template <int G, int PW, int T>
__device__ __forceinline__ void scan_channel(const uint32_t* __restrict__ w, const float* __restrict__ sc,
                                             const float (&q)[G], int bit, float (&acc)[PW][G]) {
  typename ScanRun<PW>::words x[T];
#pragma unroll
  for (int p = 0; p < T; ++p)
    x[p] = *reinterpret_cast<const typename ScanRun<PW>::words*>(w + p * 2 * kScanWaves * PW);
  const auto s = *reinterpret_cast<const typename ScanRun<PW>::scales*>(sc);
#pragma unroll
  for (int b = 0; b < PW; ++b) {
    uint32_t c = 0;
#pragma unroll
    for (int p = 0; p < T; ++p) c = (c << 1) | __builtin_amdgcn_ubfe(x[p][b], bit, 1);
    const float y = (float)c + (0.5f - (float)(1 << (T - 1)));  // exact half-integer
    const float khat = __fmul_rn(y, s[b]);                       // exact: <= 16 significant bits
#pragma unroll
    for (int h = 0; h < G; ++h) acc[b][h] = __fmaf_rn(q[h], khat, acc[b][h]);
  }
}

template <int G, int PW>
__global__ __launch_bounds__(kScanThreads) void scan_kernel(const uint64_t* __restrict__ planes,
                                                            const uint16_t* __restrict__ scales,
                                                            const int64_t* __restrict__ n, int64_t nb_cap,
                                                            const void* __restrict__ q, fathom_dtype qdt,
                                                            const uint8_t* __restrict__ depths,
                                                            float* __restrict__ scores, int64_t ld_s,
                                                            uint32_t* __restrict__ st) {
  constexpr int kScanPerWave = PW, kScanBlocks = kScanWaves * PW;  // blocks per wave, per workgroup
  constexpr int GP = G <= 1 ? 1 : G <= 2 ? 2 : G <= 4 ? 4 : 8;  // heads of a channel as one LDS run
  __shared__ ScanPlan pl;
  __shared__ int tot[2][2];
  __shared__ __attribute__((aligned(16))) uint32_t word[kScanChannels * kPlanes][2][kScanBlocks];
  __shared__ __attribute__((aligned(16))) float scl[kScanChannels][kScanBlocks];  // a16 * 2^(1-t)
  __shared__ __attribute__((aligned(16))) float qs[kD][GP];
  const int u = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t nu = unit_tokens(n, u, nb_cap * kBlockTokens, (blockIdx.x == 0 && tid == 0) ? st : nullptr);
  const int64_t b0 = (int64_t)blockIdx.x * kScanBlocks;
  if (b0 * kBlockTokens >= nu) return;
  for (int x = tid; x < G * kD; x += kScanThreads) qs[x % kD][x / kD] = load_q(q, qdt, (int64_t)u * G * kD + x);
  build_scan_plan(depths + (int64_t)u * kD, pl, tot);
  // staging: 16 threads a row, one word each (blocks past the store's end re-read its last)
  const int sb = tid & (kScanBlocks - 1), sr = tid / kScanBlocks;
  const int64_t bl = b0 + sb < nb_cap ? b0 + sb : nb_cap - 1;
  const uint64_t* Pu = planes + (int64_t)u * kD * kPlanes * nb_cap + bl;
  const uint16_t* Su = scales + (int64_t)u * kD * nb_cap + bl;
  const int bit = lane & 31, half = lane >> 5;
  float acc[kScanPerWave][G];
#pragma unroll
  for (int b = 0; b < kScanPerWave; ++b)
#pragma unroll
    for (int h = 0; h < G; ++h) acc[b][h] = 0.0f;
  const int nact = pl.nact;
  for (int a0 = 0; a0 < nact; a0 += kScanChannels) {
    const int a1 = a0 + kScanChannels < nact ? a0 + kScanChannels : nact;
    const int c0 = (int)(pl.chan[a0] >> 16), c1 = a1 < nact ? (int)(pl.chan[a1] >> 16) : pl.ncell;
    constexpr int kRowsAtOnce = kScanThreads / kScanBlocks;
    constexpr int kLoads = kScanChannels * kPlanes / kRowsAtOnce;
    uint64_t w[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int c = c0 + sr + i * kRowsAtOnce;
      if (c < c1) w[i] = Pu[(int64_t)pl.cell[c] * nb_cap];
    }
    constexpr int kScaleLoads = (kScanChannels + kRowsAtOnce - 1) / kRowsAtOnce;
    uint16_t a16[kScaleLoads];
#pragma unroll
    for (int i = 0; i < kScaleLoads; ++i) {
      const int a = a0 + sr + i * kRowsAtOnce;
      if (a < a1) a16[i] = Su[(int64_t)(pl.chan[a] & 0xFF) * nb_cap];
    }
    if (a0 > 0) __syncthreads();  // the stage before is read
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int c = sr + i * kRowsAtOnce;
      if (c < c1 - c0) {
        word[c][0][sb] = (uint32_t)w[i];
        word[c][1][sb] = (uint32_t)(w[i] >> 32);
      }
    }
#pragma unroll
    for (int i = 0; i < kScaleLoads; ++i) {
      const int a = sr + i * kRowsAtOnce;
      if (a < a1 - a0) {
        const uint32_t t = (pl.chan[a0 + a] >> 8) & 0xFF;
        scl[a][sb] = __fmul_rn(half_bits_to_float(a16[i]), __uint_as_float((128u - t) << 23));  // exact
      }
    }
    __syncthreads();
    if ((b0 + wave * kScanPerWave) * kBlockTokens < nu) {
      const int mine = (int)pl.chan[a0 + (lane & (kScanChannels - 1)) < nact ? a0 + (lane & (kScanChannels - 1)) : a0];
      for (int a = a0; a < a1; ++a) {
        const uint32_t e = (uint32_t)__builtin_amdgcn_readlane(mine, a - a0);
        const int j = e & 0xFF, t = (e >> 8) & 0xFF;
        const uint32_t* wp = &word[(int)(e >> 16) - c0][half][wave * kScanPerWave];
        const float* sp = &scl[a - a0][wave * kScanPerWave];
        float qv[G];
#pragma unroll
        for (int h = 0; h < G; ++h) qv[h] = qs[j][h];
        switch (t) {
          case 1: scan_channel<G, PW, 1>(wp, sp, qv, bit, acc); break;
          case 2: scan_channel<G, PW, 2>(wp, sp, qv, bit, acc); break;
          case 3: scan_channel<G, PW, 3>(wp, sp, qv, bit, acc); break;
          default: scan_channel<G, PW, 4>(wp, sp, qv, bit, acc); break;
        }
      }
    }
  }
#pragma unroll
  for (int b = 0; b < kScanPerWave; ++b) {
    const int64_t i = (b0 + wave * kScanPerWave + b) * kBlockTokens + lane;
    if (i < nu && i < ld_s) {
#pragma unroll
      for (int h = 0; h < G; ++h) scores[((int64_t)u * G + h) * ld_s + i] = acc[b][h];
    }
  }
}

template <int G>
static void launch_scan_g(const uint64_t* planes, const uint16_t* scales, const int64_t* n, int U, int64_t nb_cap,
                          const void* q, fathom_dtype qdt, const uint8_t* depths, float* scores, int64_t ld_s,
                          uint32_t* st, hipStream_t s) {
  // 4 blocks a wave where that gives every CU more than one workgroup (the more so
  // the more heads: their accumulators lengthen a wave), else 1.  A unit of 3000
  // keys takes 13.9 us with one and 21.6 with four; at 48 bits, 2 x 131072 keys (256
  // workgroups of four) 9.6 and 10.4 us at 1 head, 13.2 and 18.3 at 8; 3 x 131072
  // (384) 12.7 and 11.3, 16.7 and 18.6; 4 x 131072 15.0 and 11.5, 19.4 and 18.5.
  if ((nb_cap + 15) / 16 * U >= 256 + 16 * G)
    hipLaunchKernelGGL((scan_kernel<G, 4>), dim3((unsigned)((nb_cap + 15) / 16), (unsigned)U), dim3(kScanThreads), 0, s,
                       planes, scales, n, nb_cap, q, qdt, depths, scores, ld_s, st);
  else
    hipLaunchKernelGGL((scan_kernel<G, 1>), dim3((unsigned)((nb_cap + 3) / 4), (unsigned)U), dim3(kScanThreads), 0, s,
                       planes, scales, n, nb_cap, q, qdt, depths, scores, ld_s, st);
}

fathom_status launch_scan(const uint64_t* planes, const uint16_t* scales, const int64_t* n, int U, int64_t nb_cap,
                          const void* q, fathom_dtype qdt, int G, const uint8_t* depths, float* scores,
                          int64_t ld_s, uint32_t* st, hipStream_t s) {
  if (U == 0 || nb_cap == 0) return FATHOM_OK;
  switch (G) {
    case 1: launch_scan_g<1>(planes, scales, n, U, nb_cap, q, qdt, depths, scores, ld_s, st, s); break;
    case 2: launch_scan_g<2>(planes, scales, n, U, nb_cap, q, qdt, depths, scores, ld_s, st, s); break;
    case 3: launch_scan_g<3>(planes, scales, n, U, nb_cap, q, qdt, depths, scores, ld_s, st, s); break;
    case 4: launch_scan_g<4>(planes, scales, n, U, nb_cap, q, qdt, depths, scores, ld_s, st, s); break;
    case 5: launch_scan_g<5>(planes, scales, n, U, nb_cap, q, qdt, depths, scores, ld_s, st, s); break;
    case 6: launch_scan_g<6>(planes, scales, n, U, nb_cap, q, qdt, depths, scores, ld_s, st, s); break;
    case 7: launch_scan_g<7>(planes, scales, n, U, nb_cap, q, qdt, depths, scores, ld_s, st, s); break;
    default: launch_scan_g<8>(planes, scales, n, U, nb_cap, q, qdt, depths, scores, ld_s, st, s); break;
  }
  FATHOM_LAUNCH_CHECK();
  return FATHOM_OK;
}

}  // namespace fathom
