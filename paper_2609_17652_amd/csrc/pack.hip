// fathom_pack: Sec. 3.2, Eq. (2) -- per-channel 4-bit quantisation with fp16
// block scales, written channel-major as bit planes.
//
// One wave quantises an item: 64 tokens x 256 bytes of key row (64 fp32 or 128
// fp16 channels).  Lane (x = lane & 15, g = lane >> 4) loads 16 bytes of the
// rows 16g .. 16g + 15, so it holds 4 (8) channels x 16 tokens in registers
// and the block maximum, the codes and the plane bits need no lane exchange per
// key:
//   - maximum: one v_maximum3_f32 per two keys, then a 4 x 4 transpose over the
//     four lane rows (permlane swaps) so that lane (x, g) owns channel 4x + g;
//   - code: the four plane bits are the signs of v, v -+ 4s, v -+ 4s -+ 2s, ...
//     (s the cell width): every threshold is an exact multiple of s and one
//     rounded subtraction keeps the sign of the exact difference, so the bits
//     are those of floor(v / s) clipped to [-8, 7];
//   - plane words: v_alignbit_b32 shifts each sign into the plane's word, 16
//     tokens per lane; the same transpose joins the four quarters.
// About 14 VALU instructions per key and channel: fp32 packs are bound by
// reading the keys once, fp16 packs by both about equally.  8 x 2^20 keys: fp32
// 1.00 ms (4.89 TB/s, the rate of a large copy), fp16 0.65 ms (4.18 TB/s); one
// token per lane, wave-wide shuffle maxima and one LDS column read per key
// took 4.30 and 4.24 ms.
//
// pack_tile_kernel: a workgroup of 8 waves packs 16 consecutive blocks of one
// unit, whose words collect in LDS and leave as 128-byte runs per (channel,
// plane).  70 KB of LDS and 128 VGPRs: two workgroups, 4 waves per SIMD (8
// blocks a workgroup: 1.06 ms; 6 waves and 3 per SIMD: fp16 0.76 ms).
// pack_direct_kernel: one wave per item (two for an append's fp16 item), words
// stored as they are (8 bytes each, every one in its own line); it serves large
// appends and the packs whose 16-block workgroups would leave CUs idle (below).
// pack_append_kernel: a token a lane; it serves the appends of a decode step.
//
// Append (n_old given): a block's fp16 scale depends on every token in it, so
// a unit growing from n_old to n tokens re-packs blocks floor(n_old/64) ..
// ceil(n/64)-1 from the keys (the last partial block together with the new
// tokens); the grid then covers at most max_blocks blocks per unit.
#include "common.hpp"

namespace fathom {

constexpr int kPackWaves = 8;
constexpr int kPackThreads = kPackWaves * kWave;
constexpr int kTileBlocks = 16;                          // blocks per workgroup
constexpr int kTileWords = kTileBlocks * kPlanes;        // plane words per channel
constexpr int kTilePitch = 2 * kTileWords + 2;           // dwords per channel in LDS (2 of padding)
constexpr int kRows = 16;                                // tokens per lane
// Fewer 16-block tiles than CUs: one wave per item.  At 256 tiles (2 x 131072
// keys) the tiles take 28.0 us (fp32) and 27.8 us (fp16) against 42.6 and 42.1
// one wave per item, whose 8-byte stores cost three times the traffic; at 128
// tiles half of the chip would idle and one wave per item takes 22.2 us.
constexpr int64_t kDirectTiles = 256;

template <typename KT>
struct PackItem {
  static constexpr int kCh = 16 / (int)sizeof(KT);     // channels per lane
  static constexpr int kSets = kCh / 4;                // groups of 4 channels per lane
  static constexpr int kPerBlock = kD / (16 * kCh);    // items per block
};

typedef unsigned short v2u16 __attribute__((ext_vector_type(2)));
typedef _Float16 v2f16 __attribute__((ext_vector_type(2)));

// Lane row g of result register q holds what row q of register g held.
__device__ __forceinline__ void transpose_rows(uint32_t (&a)[4]) {
  auto r = __builtin_amdgcn_permlane32_swap(a[0], a[2], false, false);
  a[0] = r[0]; a[2] = r[1];
  r = __builtin_amdgcn_permlane32_swap(a[1], a[3], false, false);
  a[1] = r[0]; a[3] = r[1];
  r = __builtin_amdgcn_permlane16_swap(a[0], a[1], false, false);
  a[0] = r[0]; a[1] = r[1];
  r = __builtin_amdgcn_permlane16_swap(a[2], a[3], false, false);
  a[2] = r[0]; a[3] = r[1];
}

// Channel e of a lane's 16 bytes as fp32.
template <typename KT>
__device__ __forceinline__ float item_value(const uint4& r, int e) {
  const uint32_t w[4] = {r.x, r.y, r.z, r.w};
  if constexpr (sizeof(KT) == 4) return __uint_as_float(w[e]);
  return half_bits_to_float((uint16_t)(w[e >> 1] >> (16 * (e & 1))));
}

// The register of channel e becomes opaque here: nothing computed from it moves up.
template <typename KT>
__device__ __forceinline__ void pin_channel(uint4& r, int e) {
  const int i = sizeof(KT) == 4 ? e : e >> 1;
  if (i == 0) asm volatile("" : "+v"(r.x));
  else if (i == 1) asm volatile("" : "+v"(r.y));
  else if (i == 2) asm volatile("" : "+v"(r.z));
  else asm volatile("" : "+v"(r.w));
}

// Largest |key| per channel over the lane's rows; true if one is NaN or infinite.
template <typename KT>
__device__ __forceinline__ bool item_max(const uint4 (&r)[kRows], float (&m)[PackItem<KT>::kCh]) {
  bool bad = false;
  if constexpr (sizeof(KT) == 4) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      m[e] = fabsf(item_value<KT>(r[0], e));
#pragma unroll
      for (int t = 1; t < kRows; ++t) m[e] = __builtin_elementwise_maximum(m[e], fabsf(item_value<KT>(r[t], e)));
      bad |= !(m[e] <= 3.402823466e38f);
    }
  } else {  // magnitudes order like their bits, two channels per instruction
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v2u16 a = {0, 0};
#pragma unroll
      for (int t = 0; t < kRows; ++t) {
        const uint32_t w = i == 0 ? r[t].x : i == 1 ? r[t].y : i == 2 ? r[t].z : r[t].w;
        a = __builtin_elementwise_max(a, __builtin_bit_cast(v2u16, w & 0x7FFF7FFFu));
      }
      m[2 * i] = half_bits_to_float(a[0]);
      m[2 * i + 1] = half_bits_to_float(a[1]);
      bad |= a[0] >= 0x7C00u || a[1] >= 0x7C00u;
    }
  }
  return bad;
}

template <typename KT>
__device__ __forceinline__ void add_zero(uint4& r) {
  uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (sizeof(KT) == 4) {
      w[i] = __float_as_uint(__fadd_rn(__uint_as_float(w[i]), 0.0f));
    } else {
      const v2f16 zero = {(_Float16)0.0f, (_Float16)0.0f};
      w[i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(v2f16, w[i]) + zero);
    }
  }
  r = make_uint4(w[0], w[1], w[2], w[3]);
}

// The item's rows: row t of a lane is token tok0 + 16g + t, channels from c
// (tokens past nu read as zero).
template <typename KT>
__device__ __forceinline__ void load_item(const KT* __restrict__ Ku, int64_t ld_tok, int64_t tok0, int64_t nu, int c,
                                          uint4 (&r)[kRows]) {
  const int g = (threadIdx.x & 63) >> 4;
  const KT* p = Ku + (tok0 + kRows * g) * ld_tok + c;
  if (tok0 + kBlockTokens <= nu) {
#pragma unroll
    for (int t = 0; t < kRows; ++t) r[t] = *reinterpret_cast<const uint4*>(p + t * ld_tok);
  } else {
    const int left = (int)(nu - tok0) - kRows * g;  // valid rows of this lane, when in 1 .. 15
#pragma unroll
    for (int t = 0; t < kRows; ++t) {  // rows past the end re-read the last token and drop it
      r[t] = *reinterpret_cast<const uint4*>(p + (int64_t)min(t, left - 1) * ld_tok);
      if (t >= left) r[t] = make_uint4(0u, 0u, 0u, 0u);
    }
  }
}

// Quantise sets S0 .. S0 + SN - 1 of an item.  word[s][p] and a16[s] belong to
// channel 4 (S0 + s) + g of the lane's kCh channels; vmask has the bits of the
// block's valid tokens.
template <typename KT, int S0, int SN>
__device__ __forceinline__ void quantise_item(uint4 (&r)[kRows], uint64_t vmask, uint64_t (&word)[SN][kPlanes],
                                              uint16_t (&a16)[SN], uint32_t& flags) {
#pragma unroll
  for (int t = 0; t < kRows; ++t) add_zero<KT>(r[t]);  // -0 counts as +0
  float m[PackItem<KT>::kCh];
  const bool bad = item_max<KT>(r, m);
  const bool any_bad = __ballot(bad) != 0;
  if (any_bad) {  // rare: NaN keys leave the maximum (and take code 8 below)
    if (bad) flags |= FATHOM_DEV_NONFINITE;
#pragma unroll
    for (int e = 0; e < PackItem<KT>::kCh; ++e) {
      m[e] = 0.0f;
#pragma unroll
      for (int t = 0; t < kRows; ++t) m[e] = fmaxf(m[e], fabsf(item_value<KT>(r[t], e)));
    }
  }
#pragma unroll
  for (int s = 0; s < SN; ++s) {
    uint32_t x[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = __float_as_uint(m[4 * (S0 + s) + e]);
    transpose_rows(x);
    const float a = fmaxf(fmaxf(__uint_as_float(x[0]), __uint_as_float(x[1])),
                          fmaxf(__uint_as_float(x[2]), __uint_as_float(x[3])));
    const __half ah = __float2half_rn(a);
    a16[s] = __half_as_ushort(ah);
    const bool over = (a16[s] & 0x7FFFu) == 0x7C00u;
    if (over) flags |= FATHOM_DEV_SCALE_OVERFLOW;
    const uint32_t half_range = __float_as_uint(__fmul_rn(__half2float(ah), 0.5f));  // 4 cells, exact
    uint32_t q4[4] = {half_range, half_range, half_range, half_range};
    transpose_rows(q4);  // every lane of a column: the four channels' widths
    uint32_t lo[4], hi[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float s4 = __uint_as_float(q4[e]), s2 = __fmul_rn(s4, 0.5f), s1 = __fmul_rn(s4, 0.25f);
#pragma unroll
      for (int t = 0; t < kRows; ++t) pin_channel<KT>(r[t], 4 * (S0 + s) + e);
      uint32_t b0 = 0, b1 = 0, b2 = 0, b3 = 0;  // sign bits, the last token processed at bit 0
#pragma unroll
      for (int t = kRows - 1; t >= 0; --t) {
        const float v = item_value<KT>(r[t], 4 * (S0 + s) + e);
        const float t1 = __builtin_copysignf(s4, v);
        const float d1 = __fsub_rn(v, t1);
        float d2, d3;
        if constexpr (sizeof(KT) == 4) {
          const float t2 = __fadd_rn(t1, __builtin_copysignf(s2, d1));
          d2 = __fsub_rn(v, t2);
          const float t3 = __fadd_rn(t2, __builtin_copysignf(s1, d2));
          d3 = __fsub_rn(v, t3);
        } else {
          // 11-bit keys and widths: the differences are exact, except below
          // 2^-13 of the range, where no later threshold is near
          d2 = __fsub_rn(d1, __builtin_copysignf(s2, d1));
          d3 = __fsub_rn(d2, __builtin_copysignf(s1, d2));
        }
        b0 = __builtin_amdgcn_alignbit(b0, __float_as_uint(v), 31);
        b1 = __builtin_amdgcn_alignbit(b1, __float_as_uint(d1), 31);
        b2 = __builtin_amdgcn_alignbit(b2, __float_as_uint(d2), 31);
        b3 = __builtin_amdgcn_alignbit(b3, __float_as_uint(d3), 31);
      }
      if (any_bad) {
        uint32_t nan = 0;
#pragma unroll
        for (int t = 0; t < kRows; ++t) {
          const float v = item_value<KT>(r[t], 4 * (S0 + s) + e);
          if (v != v) nan |= 1u << t;
        }
        b0 &= ~nan;  // code 8: not negative, below every threshold above 0
        b1 |= nan;
        b2 |= nan;
        b3 |= nan;
      }
      lo[e] = b0 | (b1 << 16);
      hi[e] = b2 | (b3 << 16);
      // one channel's chains at a time, or the converted keys of all of them are live at once
      asm volatile("" : "+v"(lo[e]), "+v"(hi[e]));
    }
    transpose_rows(lo);  // now register q: tokens 16q .. 16q + 15 of channel 4s + g
    transpose_rows(hi);
    const bool zero_code = a16[s] == 0 || over;  // code 8 for every key
    const uint32_t ml = (uint32_t)vmask, mh = (uint32_t)(vmask >> 32);
#pragma unroll
    for (int p = 0; p < kPlanes; ++p) {
      const uint32_t* w = p < 2 ? lo : hi;
      const uint32_t sel = (p & 1) ? 0x07060302u : 0x05040100u;  // high or low halves of two registers
      uint32_t wl = ~__builtin_amdgcn_perm(w[1], w[0], sel) & ml;
      uint32_t wh = ~__builtin_amdgcn_perm(w[3], w[2], sel) & mh;
      if (zero_code) {
        wl = p == 0 ? ml : 0u;
        wh = p == 0 ? mh : 0u;
      }
      word[s][p] = ((uint64_t)wh << 32) | wl;
    }
  }
}

// One status update per wave.
__device__ __forceinline__ void wave_status(uint32_t* st, uint32_t flags) {
  if (__ballot(flags != 0)) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) flags |= __shfl_xor(flags, m, kWave);
    if ((threadIdx.x & 63) == 0) set_status(st, flags);
  }
}

__device__ __forceinline__ uint64_t valid_mask(int64_t left) {
  return left >= kBlockTokens ? ~0ull : left <= 0 ? 0ull : (1ull << left) - 1;
}

template <typename KT>
__global__ __launch_bounds__(kPackThreads, 4) void pack_tile_kernel(const KT* __restrict__ K, int64_t ld_tok,
                                                                   int64_t ld_unit, const int64_t* __restrict__ n,
                                                                   int64_t nb_cap, uint64_t* __restrict__ planes,
                                                                   uint16_t* __restrict__ scales,
                                                                   uint32_t* __restrict__ st) {
  using P = PackItem<KT>;
  __shared__ __attribute__((aligned(16))) uint32_t outw[kD * kTilePitch];
  __shared__ uint16_t outs[kD * kTileBlocks];
  const int u = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int x = lane & 15, g = lane >> 4;
  const int64_t nu = unit_tokens(n, u, nb_cap * kBlockTokens, tid == 0 ? st : nullptr);
  const int64_t b0 = (int64_t)blockIdx.x * kTileBlocks;
  const int nbw = nb_cap - b0 < kTileBlocks ? (int)(nb_cap - b0) : kTileBlocks;
  const KT* Ku = K + (int64_t)u * ld_unit;
  uint32_t flags = 0;
  for (int it = wave; it < nbw * P::kPerBlock; it += kPackWaves) {
    const int bb = it / P::kPerBlock, c = (it % P::kPerBlock) * 16 * P::kCh + x * P::kCh;
    const int64_t tok0 = (b0 + bb) * kBlockTokens;
    uint64_t w[P::kSets][kPlanes];
    uint16_t a16[P::kSets];
    if (tok0 < nu) {
      uint4 r[kRows];
      load_item<KT>(Ku, ld_tok, tok0, nu, c, r);
      quantise_item<KT, 0, P::kSets>(r, valid_mask(nu - tok0), w, a16, flags);
    } else {
#pragma unroll
      for (int s = 0; s < P::kSets; ++s) {
        a16[s] = 0;
#pragma unroll
        for (int p = 0; p < kPlanes; ++p) w[s][p] = 0ull;
      }
    }
#pragma unroll
    for (int s = 0; s < P::kSets; ++s) {
      const int j = c + 4 * s + g;
#pragma unroll
      for (int p = 0; p < kPlanes; ++p)
        *reinterpret_cast<uint64_t*>(&outw[j * kTilePitch + 2 * (p * kTileBlocks + bb)]) = w[s][p];
      outs[j * kTileBlocks + bb] = a16[s];
    }
  }
  __syncthreads();
  // ---- runs of up to 16 words per (channel, plane), up to 16 scales per channel ----
  uint64_t* Pu = planes + (int64_t)u * kD * kPlanes * nb_cap + b0;
#pragma unroll 4
  for (int i = tid; i < kD * kTileWords; i += kPackThreads) {
    const int row = i / kTileBlocks, bb = i % kTileBlocks;  // row = channel * 4 + plane
    const uint64_t v =
        *reinterpret_cast<const uint64_t*>(&outw[(row >> 2) * kTilePitch + 2 * ((row & 3) * kTileBlocks + bb)]);
    if (bb < nbw) Pu[(int64_t)row * nb_cap + bb] = v;
  }
  uint16_t* Su = scales + (int64_t)u * kD * nb_cap + b0;
#pragma unroll
  for (int i = tid; i < kD * kTileBlocks; i += kPackThreads) {
    const int row = i / kTileBlocks, bb = i % kTileBlocks;
    if (bb < nbw) Su[(int64_t)row * nb_cap + bb] = outs[i];
  }
  wave_status(st, flags);
}

// Sets S0 .. S0 + SN - 1 of the item of block b from channel c of unit u, stored as they are.
template <typename KT, int S0, int SN>
__device__ __forceinline__ void direct_item(const KT* Ku, int64_t ld_tok, int64_t b, int64_t nu, int u, int c,
                                            int64_t nb_cap, uint64_t* __restrict__ planes, uint16_t* __restrict__ scales,
                                            uint32_t& flags) {
  const int g = (threadIdx.x & 63) >> 4;
  const int64_t tok0 = b * kBlockTokens;
  uint64_t w[SN][kPlanes] = {};
  uint16_t a16[SN] = {};
  if (tok0 < nu) {
    uint4 r[kRows];
    load_item<KT>(Ku, ld_tok, tok0, nu, c, r);
    quantise_item<KT, S0, SN>(r, valid_mask(nu - tok0), w, a16, flags);
  }
#pragma unroll
  for (int s = 0; s < SN; ++s) {
    const int64_t j = (int64_t)u * kD + c + 4 * (S0 + s) + g;
#pragma unroll
    for (int p = 0; p < kPlanes; ++p) planes[(j * kPlanes + p) * nb_cap + b] = w[s][p];
    scales[j * nb_cap + b] = a16[s];
  }
}

// Tokens of a unit and the blocks [bs, be) that an append re-packs, from the first
// block holding a new token; false leaves the unit as it was.
__device__ __forceinline__ bool append_range(const int64_t* n, const int64_t* n_old, int u, int64_t max_blocks,
                                             int64_t nb_cap, uint32_t* st, int64_t* nu, int64_t* bs, int64_t* be) {
  const int64_t no = n_old[u];
  *nu = unit_tokens(n, u, nb_cap * kBlockTokens, st);
  *bs = no / kBlockTokens;
  *be = (*nu + kBlockTokens - 1) / kBlockTokens;
  if (no >= 0 && no <= *nu && *be - *bs <= max_blocks) return true;
  set_status(st, FATHOM_DEV_BAD_N);
  return false;
}

// An append of few blocks: one wave takes 16 bytes of a block's 64 key rows, a
// token a lane, so that a plane word is the ballot of its bits and the chain from
// the loads to the stores is short: it is one wave's latency.  8 units' one token:
// fp32 2.7 us, fp16 3.4 (16 tokens a lane, in one or two waves an item: 4.3 and 4.5;
// a tile in LDS with wave-wide shuffles: 4.3 and 4.3).
template <typename KT>
__global__ __launch_bounds__(kWave) void pack_append_kernel(const KT* __restrict__ K, int64_t ld_tok, int64_t ld_unit,
                                                           const int64_t* __restrict__ n,
                                                           const int64_t* __restrict__ n_old, int64_t max_blocks,
                                                           int64_t nb_cap, uint64_t* __restrict__ planes,
                                                           uint16_t* __restrict__ scales, uint32_t* __restrict__ st) {
  constexpr int kCh = PackItem<KT>::kCh, kItems = kD / kCh;
  const int u = blockIdx.y, lane = threadIdx.x;
  int64_t nu, bs, be;
  if (!append_range(n, n_old, u, max_blocks, nb_cap, lane == 0 ? st : nullptr, &nu, &bs, &be)) return;
  const int64_t b = bs + blockIdx.x / kItems;
  if (b >= be) return;
  const int c = (int)(blockIdx.x % kItems) * kCh;
  const int64_t tok = b * kBlockTokens + lane;
  const bool valid = tok < nu;
  uint4 r = make_uint4(0u, 0u, 0u, 0u);
  if (valid) r = *reinterpret_cast<const uint4*>(K + (int64_t)u * ld_unit + tok * ld_tok + c);
  add_zero<KT>(r);  // -0 counts as +0
  const uint64_t vm = __ballot(valid);
  uint32_t mx[kCh / 4][4], flags = 0;
#pragma unroll
  for (int e = 0; e < kCh; ++e) {  // NaN keys leave the maximum (and take code 8 below)
    const float a = fabsf(item_value<KT>(r, e));
    if (!(a <= 3.402823466e38f)) flags |= FATHOM_DEV_NONFINITE;
    mx[e / 4][e % 4] = a != a ? 0u : __float_as_uint(a);
  }
#pragma unroll
  for (int i = 0; i < kCh / 4; ++i) wave_max4_u(mx[i]);
  uint32_t lo = 0, hi = 0, a16w = 0;
#pragma unroll
  for (int e = 0; e < kCh; ++e) {
    const __half ah = __float2half_rn(__uint_as_float(mx[e / 4][e % 4]));
    const uint16_t a16 = __half_as_ushort(ah);
    const bool over = (a16 & 0x7FFFu) == 0x7C00u, zero_code = a16 == 0 || over;  // code 8 for every key
    if (over) flags |= FATHOM_DEV_SCALE_OVERFLOW;
    // the signs of v and of its distances to the thresholds, as in quantise_item
    const float v = item_value<KT>(r, e), s4 = __fmul_rn(__half2float(ah), 0.5f);
    const float t1 = __builtin_copysignf(s4, v), d1 = __fsub_rn(v, t1);
    const float t2 = __fadd_rn(t1, __builtin_copysignf(__fmul_rn(s4, 0.5f), d1)), d2 = __fsub_rn(v, t2);
    const float t3 = __fadd_rn(t2, __builtin_copysignf(__fmul_rn(s4, 0.25f), d2)), d3 = __fsub_rn(v, t3);
    const uint64_t nan = __ballot(v != v), on = zero_code ? 0ull : vm & ~nan;
    const uint64_t w[kPlanes] = {(zero_code ? vm : (~__ballot(__float_as_int(v) < 0) | nan) & vm),
                                 ~__ballot(__float_as_int(d1) < 0) & on, ~__ballot(__float_as_int(d2) < 0) & on,
                                 ~__ballot(__float_as_int(d3) < 0) & on};
#pragma unroll
    for (int p = 0; p < kPlanes; ++p)
      if (lane == kPlanes * e + p) {
        lo = (uint32_t)w[p];
        hi = (uint32_t)(w[p] >> 32);
      }
    if (lane == e) a16w = a16;
  }
  const int64_t j = (int64_t)u * kD + c;
  if (lane < kPlanes * kCh) planes[(j * kPlanes + lane) * nb_cap + b] = ((uint64_t)hi << 32) | lo;
  if (lane < kCh) scales[(j + lane) * nb_cap + b] = (uint16_t)a16w;
  wave_status(st, flags);
}

// SPLIT: an item's sets of 4 channels a lane go to waves of their own.  An append
// is one wave's latency: one unit's fp16 block takes 4.1 us, 5.7 in one wave.
template <typename KT, bool SPLIT>
__global__ __launch_bounds__(kWave) void pack_direct_kernel(const KT* __restrict__ K, int64_t ld_tok, int64_t ld_unit,
                                                           const int64_t* __restrict__ n,
                                                           const int64_t* __restrict__ n_old, int64_t max_blocks,
                                                           int64_t nb_cap, uint64_t* __restrict__ planes,
                                                           uint16_t* __restrict__ scales, uint32_t* __restrict__ st) {
  using P = PackItem<KT>;
  constexpr int kParts = SPLIT ? P::kSets : 1;  // waves per item
  const int u = blockIdx.y, lane = threadIdx.x, x = lane & 15;
  int64_t nu, bs = 0, be = nb_cap;
  if (!n_old) nu = unit_tokens(n, u, nb_cap * kBlockTokens, lane == 0 ? st : nullptr);
  else if (!append_range(n, n_old, u, max_blocks, nb_cap, lane == 0 ? st : nullptr, &nu, &bs, &be)) return;
  const int it = (int)(blockIdx.x / kParts), part = (int)(blockIdx.x % kParts);
  const int64_t b = bs + it / P::kPerBlock;
  if (b >= be) return;
  const int c = (it % P::kPerBlock) * 16 * P::kCh + x * P::kCh;
  const KT* Ku = K + (int64_t)u * ld_unit;
  uint32_t flags = 0;
  if constexpr (kParts == 1)
    direct_item<KT, 0, P::kSets>(Ku, ld_tok, b, nu, u, c, nb_cap, planes, scales, flags);
  else if (part == 0)
    direct_item<KT, 0, 1>(Ku, ld_tok, b, nu, u, c, nb_cap, planes, scales, flags);
  else
    direct_item<KT, 1, 1>(Ku, ld_tok, b, nu, u, c, nb_cap, planes, scales, flags);
  wave_status(st, flags);
}

template <typename KT>
static void launch_pack_t(const KT* K, int64_t ld_tok, int64_t ld_unit, const int64_t* n, const int64_t* n_old,
                          int64_t max_new, int U, int64_t nb_cap, uint64_t* planes, uint16_t* scales, uint32_t* st,
                          hipStream_t s) {
  // append: new tokens span at most ceil(max_new / 64) + 1 blocks per unit
  int64_t mb = nb_cap;
  if (n_old) {
    mb = (max_new + kBlockTokens - 1) / kBlockTokens + 1;
    if (mb > nb_cap) mb = nb_cap;
  }
  const int64_t tiles = (nb_cap + kTileBlocks - 1) / kTileBlocks;
  const unsigned items = (unsigned)(mb * PackItem<KT>::kPerBlock);
  // An append's rows are read 16 bytes at a time by 16 (fp32: 32) waves a token each
  // lane, which up to about 100 blocks is the faster (32 units' 128 tokens, 96 blocks: fp32
  // 3.8 us against 4.9, fp16 4.8 and 5.1; 256 tokens, 160 blocks: 6.5 and 5.5, 6.1 and 5.6).
  if (n_old && mb * U <= 96)
    hipLaunchKernelGGL(pack_append_kernel<KT>, dim3((unsigned)(mb * (kD / PackItem<KT>::kCh)), (unsigned)U), dim3(kWave), 0,
                       s, K, ld_tok, ld_unit, n, n_old, mb, nb_cap, planes, scales, st);
  else if (n_old)
    hipLaunchKernelGGL((pack_direct_kernel<KT, true>), dim3(items * PackItem<KT>::kSets, (unsigned)U), dim3(kWave), 0, s,
                       K, ld_tok, ld_unit, n, n_old, mb, nb_cap, planes, scales, st);
  else if (tiles * U < kDirectTiles)
    hipLaunchKernelGGL((pack_direct_kernel<KT, false>), dim3(items, (unsigned)U), dim3(kWave), 0, s, K, ld_tok, ld_unit,
                       n, n_old, mb, nb_cap, planes, scales, st);
  else
    hipLaunchKernelGGL(pack_tile_kernel<KT>, dim3((unsigned)tiles, (unsigned)U), dim3(kPackThreads), 0, s, K, ld_tok,
                       ld_unit, n, nb_cap, planes, scales, st);
}

fathom_status launch_pack(const void* K, fathom_dtype kdt, int64_t ld_tok, int64_t ld_unit,
                          const int64_t* n, const int64_t* n_old, int64_t max_new, int U, int64_t nb_cap,
                          uint64_t* planes, uint16_t* scales, uint32_t* st, hipStream_t s) {
  if (U == 0 || nb_cap == 0) return FATHOM_OK;
  if (kdt == FATHOM_F32)
    launch_pack_t(reinterpret_cast<const float*>(K), ld_tok, ld_unit, n, n_old, max_new, U, nb_cap, planes, scales,
                  st, s);
  else
    launch_pack_t(reinterpret_cast<const __half*>(K), ld_tok, ld_unit, n, n_old, max_new, U, nb_cap, planes, scales,
                  st, s);
  FATHOM_LAUNCH_CHECK();
  return FATHOM_OK;
}

}  // namespace fathom
