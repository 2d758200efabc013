// fathom_topk: Sec. 2 (top-k decoding) -- per query head, the k largest
// scores over an eligible window, ordered by (score desc, index asc).
//
// Exact radix select on an order-preserving uint32 key (score_key), digits of
// 12, 10 and 10 bits, that stops refining as soon as the keys not yet ruled
// out fit a list of lcap entries (about 4k + 2048):
//   - a pass over the row either histograms the next digit (the workgroup that
//     arrives last at a row picks the digit holding the k-th key), or, once
//     the row's remaining keys fit, collects them (key, index) into its list.
//     Each row decides for itself; a row that is done leaves the later passes at
//     once.  Scores spread over a few binades take one histogram and one
//     collection: the scores are read twice.
//   - the rank pass orders the lists and writes the top k: up to 8 workgroups a
//     row share its output positions by a counting sort on sub-buckets, so that
//     only keys sharing a sub-bucket are compared: interpolated ones, or, where
//     the scores are uneven, ones between entries of the list.
//   - more equal keys at the threshold than a list holds: the list gets the
//     keys above, the collecting pass counts the equal ones of every chunk, and
//     the rank pass writes the first of them in index order from those counts.
// Rows are split into chunks of kChunk elements so that a launch has many
// workgroups even for a few rows.  32 rows of 131072 scores, k = 1024, in 6
// launches: 38 us, 58 with ties at the threshold, 46 rounded to quarters, 63 in
// one binade (13 launches with three histograms and single-thread pivots, count,
// scan and write passes and a bitonic sort, before: 104, 155, 122, 112 us).
#include <algorithm>
#include <type_traits>

#include "common.hpp"

namespace fathom {

constexpr int kTopkThreads = 256;
constexpr int kPerThread = 16;
constexpr int kChunk = kTopkThreads * kPerThread;  // 4096 elements per workgroup
constexpr int kDigits = 3;
constexpr int kBins = 4096;
constexpr int kNever = 1 << 30;

struct RowState {
  uint32_t prefix;   // digits fixed so far
  uint32_t mask;     // bits of `prefix` that are fixed
  int32_t need;      // how many still to take among keys matching `prefix`
  int32_t collect;   // the pass that collects the row's keys >= prefix (kNever: not known yet)
  uint32_t strict;   // collect only keys > prefix (the equal ones do not fit)
  uint32_t arrived;  // workgroups that have added their histogram
  uint32_t count;    // keys in the list
  uint32_t k;        // k once the first digit is known
};

struct TopkWs {
  uint32_t* hist;   // [R][kBins]
  RowState* state;  // [R]
  uint64_t* list;   // [R][lcap] composites (key << 32 | ~index), any order
  int lcap;
};

static inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

static inline int64_t topk_chunks(int64_t max_n) { return (max_n + kChunk - 1) / kChunk; }

static inline int topk_lcap(int k) {
  const int c = 4 * k + 2048;
  return c < 2 * FATHOM_MAX_K ? c : 2 * FATHOM_MAX_K;
}

size_t topk_ws_bytes(int R, int64_t, int k) {
  return align_up((size_t)R * kBins * 4) + align_up((size_t)R * sizeof(RowState)) +
         align_up((size_t)R * topk_lcap(k) * 8);
}

static TopkWs carve(void* ws, int R, int k) {
  char* p = reinterpret_cast<char*>(ws);
  TopkWs w;
  w.hist = reinterpret_cast<uint32_t*>(p); p += align_up((size_t)R * kBins * 4);
  w.state = reinterpret_cast<RowState*>(p); p += align_up((size_t)R * sizeof(RowState));
  w.list = reinterpret_cast<uint64_t*>(p);
  w.lcap = topk_lcap(k);
  return w;
}

struct RowRange {
  int64_t lo, hi;  // eligible window [lo, hi)
};

__device__ __forceinline__ RowRange row_range(const int64_t* n, int u, int64_t cap, int64_t lo,
                                              int64_t tail, uint32_t* st) {
  const int64_t nu = unit_tokens(n, u, cap, st);
  RowRange r;
  r.lo = lo;
  r.hi = nu - tail;
  if (r.hi < r.lo) r.hi = r.lo;
  return r;
}

__global__ __launch_bounds__(1024) void topk_init_kernel(RowState* __restrict__ state, uint4* __restrict__ hist,
                                                         int k) {
  const int r = blockIdx.x;
  hist[(int64_t)r * (kBins / 4) + threadIdx.x] = make_uint4(0u, 0u, 0u, 0u);
  if (threadIdx.x == 0) {
    RowState s = {};
    s.need = k;
    s.collect = kNever;
    state[r] = s;
  }
}
static_assert(kBins == 4 * 1024, "topk_init_kernel clears 4 bins per thread");

// Chunks whose equal keys at the threshold are counted together.
__device__ __forceinline__ int64_t tie_chunks(const RowRange& rr) {
  return ((rr.hi - rr.lo + kChunk - 1) / kChunk + kBins - 1) / kBins;
}

// Pass `pass` over the scores (see above).  Every workgroup of a row sees the
// state the pass before left, and only the one that arrives last changes it.
__global__ __launch_bounds__(kTopkThreads) void topk_pass_kernel(const float* __restrict__ scores, int64_t ld_s,
                                                                 const int64_t* __restrict__ n, int G, int64_t lo,
                                                                 int64_t tail, int pass, TopkWs ws,
                                                                 uint32_t* __restrict__ st) {
  __shared__ __attribute__((aligned(16))) uint32_t h[kBins];
  __shared__ uint32_t part[kTopkThreads / kWave];
  __shared__ int s_digit;
  __shared__ uint32_t s_above, s_last;
  const int r = blockIdx.y, u = r / G, tid = threadIdx.x, lane = tid & 63;
  RowState* S = ws.state + r;
  const int collect = S->collect;
  if (collect < pass) return;
  const RowRange rr = row_range(n, u, ld_s, lo, tail, (pass == 0 && blockIdx.x == 0 && tid == 0) ? st : nullptr);
  const int64_t step = (int64_t)gridDim.x * kChunk;  // a workgroup takes every gridDim.x-th chunk
  int64_t c0 = rr.lo + (int64_t)blockIdx.x * kChunk;
  if (c0 >= rr.hi) return;
  const uint32_t prefix = S->prefix;
  const float* row = scores + (int64_t)r * ld_s;
  float v[kPerThread];
  auto load = [&]() {
#pragma unroll
    for (int e = 0; e < kPerThread; ++e) {
      const int64_t i = c0 + (int64_t)e * kTopkThreads + tid;
      v[e] = row[i < rr.hi ? i : rr.hi - 1];
    }
  };
  if (collect == pass) {
    const bool strict = S->strict != 0;
    uint64_t* list = ws.list + (int64_t)r * ws.lcap;
    for (; c0 < rr.hi; c0 += step) {
      load();
      uint32_t take = 0;
      int mine = 0, same = 0;
#pragma unroll
      for (int e = 0; e < kPerThread; ++e) {
        const uint32_t key = score_key(v[e]);
        const bool ok = c0 + (int64_t)e * kTopkThreads + tid < rr.hi, in = ok && (strict ? key > prefix : key >= prefix);
        take |= (uint32_t)in << e;
        mine += in;
        same += ok && key == prefix;
      }
      if (strict) {  // the equal keys of the chunk (the histogram is all zeros by now)
        same = wave_sum_int(same);
        if (lane == 0 && same > 0)
          atomicAdd(&ws.hist[(int64_t)r * kBins + ((c0 - rr.lo) / kChunk) / tie_chunks(rr)], (uint32_t)same);
      }
      if (__ballot(take != 0) == 0) continue;
      int inc = mine;  // positions: one reservation per wave
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += x;
      }
      uint32_t base = 0;
      if (lane == 63) base = atomicAdd(&S->count, (uint32_t)inc);
      base = __shfl(base, 63, kWave) + (uint32_t)(inc - mine);
#pragma unroll
      for (int e = 0; e < kPerThread; ++e) {
        if (take & (1u << e)) {
          const int64_t i = c0 + (int64_t)e * kTopkThreads + tid;
          // the histograms bound the count; the test only keeps a changed input inside the list
          if (base < (uint32_t)ws.lcap) list[base] = ((uint64_t)score_key(v[e]) << 32) | (uint64_t)(~(uint32_t)i);
          ++base;
        }
      }
    }
    return;
  }
  const int shift = pass == 0 ? 20 : pass == 1 ? 10 : 0, nb = pass == 0 ? 4096 : 1024;
  const uint32_t mask = S->mask;
#pragma unroll
  for (int i = 0; i < kBins / 4 / kTopkThreads; ++i)
    reinterpret_cast<uint4*>(h)[tid + i * kTopkThreads] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  bool nonfinite = false;
  const uint64_t lanes_lt = (1ull << lane) - 1;
  for (; c0 < rr.hi; c0 += step) {
    load();
    auto bin_of = [&](int e) -> uint32_t {  // ~0: not counted
      const uint32_t key = score_key(v[e]);
      return c0 + (int64_t)e * kTopkThreads + tid < rr.hi && (key & mask) == prefix ? (key >> shift) & (uint32_t)(nb - 1) : ~0u;
    };
    if (pass == 0) {
#pragma unroll
      for (int e = 0; e < kPerThread; ++e) nonfinite |= !(fabsf(v[e]) <= 3.402823466e38f);  // past the end: the last score
    }
    // Additions to one address queue.  In the first pass, where most of a wave's
    // keys share a bin those add up before; the later ones keep four copies of
    // their fewer bins.  512 rows of 40000 scores of one binade: 44 us the first
    // pass and 29 the next two (plain additions: 151, 80 and 50).
    const uint32_t b0 = bin_of(0);
    const uint64_t lead = __ballot(b0 == (uint32_t)__builtin_amdgcn_readfirstlane((int)b0) && b0 != ~0u);
    if (pass == 0 && __popcll(lead) >= 48) {
#pragma unroll
      for (int e = 0; e < kPerThread; ++e) {
        const uint32_t b = bin_of(e);
        if (b != ~0u) {
          const uint64_t one = __ballot(b == (uint32_t)__builtin_amdgcn_readfirstlane((int)b));
          if (!((one >> lane) & 1ull)) atomicAdd(&h[b], 1u);
          else if ((one & lanes_lt) == 0ull) atomicAdd(&h[b], (uint32_t)__popcll(one));
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < kPerThread; ++e) {
        const uint32_t b = bin_of(e);
        if (b != ~0u) atomicAdd(&h[pass == 0 ? b : 4u * b + (uint32_t)(lane & 3)], 1u);
      }
    }
  }
  if (pass == 0 && __ballot(nonfinite) && lane == 0) set_status(st, FATHOM_DEV_NONFINITE);
  __syncthreads();
  uint32_t* gh = ws.hist + (int64_t)r * kBins;
  // The counts are only ever touched by device-scope atomics, so an addition is
  // done once its old value has come back: no fence, whose write-back of the L2
  // by every workgroup took 100 us.
  uint32_t back = 0;
  auto batches = [&](auto fn) {  // every bin of this thread, up to 16 in flight
    if (nb == 4096) fn(std::integral_constant<int, 4096 / kTopkThreads>{});
    else fn(std::integral_constant<int, 1024 / kTopkThreads>{});
  };
  batches([&](auto N) {
    uint32_t x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int b = tid + i * kTopkThreads;
      if (pass == 0) {
        x[i] = h[b];
      } else {
        const uint4 q = reinterpret_cast<const uint4*>(h)[b];
        x[i] = q.x + q.y + q.z + q.w;
      }
    }
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (x[i]) x[i] = atomicAdd(&gh[tid + i * kTopkThreads], x[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) back |= x[i];
  });
  asm volatile("" ::"v"(back) : "memory");
  __syncthreads();
  if (tid == 0) {
    const int64_t chunks = (rr.hi - rr.lo + kChunk - 1) / kChunk;
    const uint32_t groups = chunks < (int64_t)gridDim.x ? (uint32_t)chunks : gridDim.x;
    s_last = atomicAdd(&S->arrived, 1u) + 1u == groups;
  }
  __syncthreads();
  if (!s_last) return;
  batches([&](auto N) {
    uint32_t x[N];
#pragma unroll
    for (int i = 0; i < N; ++i)
      x[i] = __hip_atomic_load(&gh[tid + i * kTopkThreads], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      h[tid + i * kTopkThreads] = x[i];
      gh[tid + i * kTopkThreads] = 0u;  // for the next pass
    }
  });
  __syncthreads();
  const int need = S->need;
  find_crossing(h, nb, (uint32_t)need, part, &s_digit, &s_above);
  if (tid == 0) {
    // keys above the digit's own: all of the k wanted so far but `need`, and s_above
    const int left = need - (int)s_above, k = pass > 0 ? (int)S->k : need;
    const uint32_t fits = (uint32_t)(k - left) + h[s_digit];
    S->k = (uint32_t)k;
    S->prefix = prefix | (uint32_t)s_digit << shift;
    S->mask = mask | (uint32_t)(nb - 1) << shift;
    S->need = left;
    S->arrived = 0u;
    if (fits <= (uint32_t)ws.lcap) {
      S->collect = pass + 1;
    } else if (pass == kDigits - 1) {
      S->collect = pass + 1;
      S->strict = 1u;
    }
  }
}

// ---------------------------------------------------------------- ranks
constexpr int kRankT = 512;
constexpr int kRankWaves = kRankT / kWave;
constexpr int kRankShare = 8;     // workgroups per row at most
constexpr int kRankMaxSub = 4096; // sub-buckets at most
constexpr int kRankGroup = 4096;  // keys one workgroup groups at most
constexpr int kRankSame = 64;     // keys of one interpolated sub-bucket at most (else splitters)
constexpr int kRankRegs = 8;      // list entries per thread kept in registers
constexpr int kRankSplit = 255;   // splitters: 256 sub-buckets, an entry's in one byte
constexpr int kRankFew = 512;     // lists up to here are ranked key against key

static_assert(4 * (kRankMaxSub + 320 - (kRankSplit + 2)) >= 2 * FATHOM_MAX_K, "a byte for every entry of a list");

struct RankLds {
  __attribute__((aligned(16))) uint64_t grp[kRankGroup];
  uint32_t hist[kRankMaxSub + 320];  // with splitters: 257 counts, then the entries' sub-buckets
  uint64_t split[kRankSplit + 1];
  uint32_t at[kRankSplit + 1];
  uint32_t red[3][kRankWaves];
  uint32_t first[kRankShare + 1];
};

// Exclusive prefix of hist[0 .. ns) in place (thread t owns a run of ns / kRankT,
// or one), hist[ns] = c; first[y] = the sub-bucket where part y of 2^lp starts, the
// first whose first position is at least y K / 2^lp.  Returns the largest count.
__device__ __forceinline__ uint32_t rank_prefix(RankLds& L, int ns, uint32_t c, uint32_t K, int lp) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int kPer = kRankMaxSub / kRankT;
  const int per = (ns + kRankT - 1) / kRankT, x0 = tid * per;
  uint32_t hv[kPer], run = 0, most = 0;  // this thread's run (0 past it)
#pragma unroll
  for (int x = 0; x < kPer; ++x) hv[x] = x < per && x0 + x < ns ? L.hist[x0 + x] : 0u;
#pragma unroll
  for (int x = 0; x < kPer; ++x) {
    run += hv[x];
    most = hv[x] > most ? hv[x] : most;
  }
  uint32_t inc = run;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(inc, o, kWave);
    if (lane >= o) inc += y;
    const uint32_t m = __shfl_xor(most, o, kWave);
    most = m > most ? m : most;
  }
  if (lane == 63) {
    L.red[0][wave] = inc;
    L.red[2][wave] = most;
  }
  if (tid <= 1 << lp && (uint32_t)tid * K >> lp == 0u) L.first[tid] = 0u;
  __syncthreads();
  uint32_t acc = inc - run;
#pragma unroll
  for (int x = 0; x < kRankWaves; ++x) {
    if (x < wave) acc += L.red[0][x];
    most = L.red[2][x] > most ? L.red[2][x] : most;
  }
  uint32_t at[kPer + 1];
  at[0] = acc;
#pragma unroll
  for (int x = 0; x < kPer; ++x) {
    at[x + 1] = at[x] + hv[x];
    if (x < per && x0 + x < ns) L.hist[x0 + x] = at[x];
  }
#pragma unroll
  for (int y = 1; y <= kRankShare; ++y) {  // bounds among this thread's positions
    const uint32_t b = (uint32_t)y * K >> lp;
    if (y <= 1 << lp && acc < b && at[kPer] >= b) {
      int f = x0 + 1;
#pragma unroll
      for (int x = 1; x <= kPer; ++x) f += at[x] < b;
      L.first[y] = (uint32_t)f;
    }
  }
  if (tid == 0) L.hist[ns] = c;
  __syncthreads();
  return most;
}

// A row's list in order: `parts` workgroups share its K output positions by a
// counting sort on sub-buckets interpolated between the smallest and the largest
// key, so that only keys sharing a sub-bucket are compared.  Where those come out
// uneven (equal scores, an outlier) the sub-buckets lie between 256 entries of the
// list instead, taken at scattered places: composites are distinct, so these are
// even whatever the scores (a sub-bucket of 8 times the mean among 16384 entries:
// one row in 30).  Short uneven lists, and what still does not fit, are ranked
// key against key.
__global__ __launch_bounds__(kRankT) void topk_rank_kernel(const float* __restrict__ scores, int64_t ld_s,
                                                           const int64_t* __restrict__ n, int G, int R, int64_t lo,
                                                           int64_t tail, int k, int lp, TopkWs ws,
                                                           int32_t* __restrict__ idx, float* __restrict__ val,
                                                           uint32_t* __restrict__ st) {
  __shared__ RankLds L;
  // a row's workgroups on one XCD (workgroups are dealt to the 8 XCDs in turn): its list comes into one L2
  const int parts = 1 << lp;
  const int r = (int)(blockIdx.x >> (3 + lp)) * 8 + (int)(blockIdx.x % 8);
  const int z = (int)(blockIdx.x / 8) & (parts - 1);
  if (r >= R) return;
  const int u = r / G, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t* list = ws.list + (int64_t)r * ws.lcap;
  uint64_t pv[kRankRegs];
#pragma unroll
  for (int x = 0; x < kRankRegs; ++x) {  // entries past the count are read but not used
    const int e = tid + kRankT * x;
    pv[x] = e < ws.lcap ? list[e] : 0ull;
  }
  const RowState S = ws.state[r];
  const float* row = scores + (int64_t)r * ld_s;
  const uint32_t c = S.count < (uint32_t)ws.lcap ? S.count : (uint32_t)ws.lcap;
  auto emit = [&](uint32_t rank, int32_t i) {
    idx[(int64_t)r * k + rank] = i;
    if (val) val[(int64_t)r * k + rank] = row[i];
  };
  if (S.strict) {
    // behind the c keys above stand the first k - c equal ones in index order: the
    // counts of the chunks give their positions, and the parts share the chunks
    const RowRange rr = row_range(n, u, ld_s, lo, tail, nullptr);
    const int64_t per = tie_chunks(rr) * kChunk;
    const int nb = (int)((rr.hi - rr.lo + per - 1) / per);
    for (int b = tid; b < nb; b += kRankT) L.hist[b] = ws.hist[(int64_t)r * kBins + b];
    __syncthreads();
    const uint32_t need = (uint32_t)k - c;
    rank_prefix(L, nb, 0u, 0u, 0);
    for (int b = z; b < nb && L.hist[b] < need; b += parts) {
      uint32_t at0 = L.hist[b];
      if (b + 1 < nb && L.hist[b + 1] == at0) continue;  // none
      const int64_t end = rr.lo + (b + 1) * per < rr.hi ? rr.lo + (b + 1) * per : rr.hi;
      for (int64_t i = rr.lo + b * per; i < end && at0 < need; i += kChunk) {
        const int64_t i0 = i + tid * kRankRegs;  // eight in a row per thread: thread order is index order
        uint32_t eq = 0;
#pragma unroll
        for (int x = 0; x < kRankRegs; ++x)
          if (i0 + x < end && score_key(row[i0 + x]) == S.prefix) eq |= 1u << x;
        const int mine = __popc(eq);
        int inc = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int y = __shfl_up(inc, o, kWave);
          if (lane >= o) inc += y;
        }
        if (lane == 63) L.red[0][wave] = (uint32_t)inc;
        __syncthreads();
        uint32_t at = at0 + (uint32_t)(inc - mine);
        for (int x = 0; x < kRankWaves; ++x) {
          if (x < wave) at += L.red[0][x];
          at0 += L.red[0][x];
        }
#pragma unroll
        for (int x = 0; x < kRankRegs; ++x)
          if (eq & (1u << x)) {
            if (at < need) emit(c + at, (int32_t)(i0 + x));
            ++at;
          }
        __syncthreads();  // red read by all
      }
    }
    __syncthreads();
  }
  const uint32_t K = c < (uint32_t)k ? c : (uint32_t)k;
  if (z == 0 && !S.strict && K < (uint32_t)k) {  // fewer eligible keys than k
    for (int e = (int)K + tid; e < k; e += kRankT) {
      idx[(int64_t)r * k + e] = -1;
      if (val) val[(int64_t)r * k + e] = __uint_as_float(0x7FC00000u);
    }
    if (tid == 0) set_status(st, FATHOM_DEV_TOPK_SHORT);
  }
  if (K == 0) return;
  auto each = [&](auto fn) {  // every list entry and its place
#pragma unroll
    for (int x = 0; x < kRankRegs; ++x)
      if (tid + kRankT * x < (int)c) fn(pv[x], (uint32_t)(tid + kRankT * x));
    for (uint32_t e = tid + kRankT * kRankRegs; e < c; e += kRankT) fn(list[e], e);
  };
  // (hist zeroed before:) counts the sub-buckets, finds this part's and orders its keys; false (to every
  // thread of every part alike) if a sub-bucket or a part's share is too large
  auto order = [&](int ns, uint32_t same, auto sub_of, auto keep, auto kept) {
    each([&](uint64_t v, uint32_t e) {
      const int sb = sub_of(v);
      keep(e, sb);
      atomicAdd(&L.hist[sb], 1u);
    });
    __syncthreads();
    bool over = rank_prefix(L, ns, c, K, lp) > same;
    for (int y = 0; y < parts; ++y) over |= L.hist[L.first[y + 1]] - L.hist[L.first[y]] > (uint32_t)kRankGroup;
    if (over) {
      __syncthreads();  // the bounds are read before the next attempt's
      return false;
    }
    const int s0 = (int)L.first[z], s1 = (int)L.first[z + 1];
    if (s0 == s1) return true;
    const uint32_t start = L.hist[s0], share = L.hist[s1] - start;
    __syncthreads();  // every bound read before hist[s0 .. s1) serve as cursors
    each([&](uint64_t v, uint32_t e) {  // group by sub-bucket; hist[s] ends at the group's end
      const int sb = kept(v, e);
      if (sb >= s0 && sb < s1) L.grp[atomicAdd(&L.hist[sb], 1u) - start] = v;
    });
    __syncthreads();
    for (uint32_t e = tid; e < share; e += kRankT) {
      const uint64_t v = L.grp[e];
      const int sb = sub_of(v);
      const uint32_t g0 = sb > s0 ? L.hist[sb - 1] : start, g1 = L.hist[sb];
      uint32_t rank = g0;
      for (uint32_t x = g0; x < g1; ++x) rank += L.grp[x - start] > v;
      if (rank < K) emit(rank, (int32_t)(~(uint32_t)v));
    }
    return true;
  };
  int ns = 64;  // sub-buckets: a power of two, at least the entries
  while (ns < (int)c && ns < kRankMaxSub) ns <<= 1;
  for (int x = tid; x < ns; x += kRankT) L.hist[x] = 0u;
  uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
  each([&](uint64_t v, uint32_t) {
    const uint32_t key = (uint32_t)(v >> 32);
    kmin = key < kmin ? key : kmin;
    kmax = key > kmax ? key : kmax;
  });
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    const uint32_t a = __shfl_xor(kmin, m, kWave), b = __shfl_xor(kmax, m, kWave);
    kmin = a < kmin ? a : kmin;
    kmax = b > kmax ? b : kmax;
  }
  if (lane == 0) {
    L.red[0][wave] = kmin;
    L.red[1][wave] = kmax;
  }
  __syncthreads();
  for (int x = 0; x < kRankWaves; ++x) {
    kmin = L.red[0][x] < kmin ? L.red[0][x] : kmin;
    kmax = L.red[1][x] > kmax ? L.red[1][x] : kmax;
  }
  // sub-bucket: floor((kmax - key) * scale), not decreasing as the key falls
  const float scale = kmax > kmin ? (float)(ns - 1) / (float)(kmax - kmin) : 0.0f;
  auto sub_even = [&](uint64_t v) {
    const int sb = (int)__fmul_rn((float)(kmax - (uint32_t)(v >> 32)), scale);
    return sb < ns - 1 ? sb : ns - 1;
  };
  if (order(ns, (uint32_t)kRankSame, sub_even, [](uint32_t, int) {}, [&](uint64_t v, uint32_t) { return sub_even(v); }))
    return;
  if (c > (uint32_t)kRankFew) {
    const int x = tid & kRankSplit, half = tid / (kRankSplit + 1);  // two threads a splitter, half of the others each
    const uint64_t mine = x < kRankSplit ? list[((uint64_t)((uint32_t)(x + 1) * 0x9E3779B1u) * c) >> 32] : 0ull;
    if (half == 0) {
      L.grp[x] = mine;
      L.at[x] = 0u;
      L.hist[x] = 0u;
    }
    __syncthreads();
    uint32_t above = 0;
#pragma unroll 8
    for (int y = 0; y < (kRankSplit + 1) / 2; ++y) {
      const int o = half * ((kRankSplit + 1) / 2) + y;
      const uint64_t v = L.grp[o];
      above += v > mine || (v == mine && o < x);
    }
    atomicAdd(&L.at[x], above);
    __syncthreads();
    if (half == 0) L.split[L.at[x]] = mine;  // largest first
    __syncthreads();
    uint8_t* id = reinterpret_cast<uint8_t*>(&L.hist[kRankSplit + 2]);
    auto sub_split = [&](uint64_t v) {  // splitters above v
      int b = 0;
#pragma unroll
      for (int h = (kRankSplit + 1) / 2; h >= 1; h >>= 1)
        if (L.split[b + h - 1] > v) b += h;
      return b;
    };
    if (order(kRankSplit + 1, (uint32_t)kRankGroup, sub_split, [&](uint32_t e, int sb) { id[e] = (uint8_t)sb; },
              [&](uint64_t, uint32_t e) { return (int)id[e]; }))
      return;
  }
  for (uint32_t e0 = z * kRankT; e0 < c; e0 += parts * kRankT) {
    const uint64_t v = e0 + tid < c ? list[e0 + tid] : 0ull;
    uint32_t rank = 0;
    for (uint32_t b = 0; b < c; b += kRankGroup) {
      const uint32_t m = c - b < (uint32_t)kRankGroup ? c - b : (uint32_t)kRankGroup;
      __syncthreads();
      for (uint32_t x = tid; x < m; x += kRankT) L.grp[x] = list[b + x];
      __syncthreads();
#pragma unroll 8
      for (uint32_t x = 0; x < m; ++x) rank += L.grp[x] > v;
    }
    if (e0 + tid < c && rank < K) emit(rank, (int32_t)(~(uint32_t)v));
  }
}

fathom_status launch_topk(const float* scores, int64_t ld_s, const int64_t* n, int U, int G, int k,
                          int64_t lo, int64_t tail, int32_t* idx, float* val, void* ws, uint32_t* st,
                          hipStream_t s) {
  const int R = U * G;
  if (R == 0) return FATHOM_OK;
  const int64_t nch = topk_chunks(ld_s) > 0 ? topk_chunks(ld_s) : 1;
  const TopkWs w = carve(ws, R, k);
  hipLaunchKernelGGL(topk_init_kernel, dim3(R), dim3(1024), 0, s, w.state, reinterpret_cast<uint4*>(w.hist), k);
  // Up to 2048 workgroups in the first two passes (a merged histogram each), 256
  // in the later ones, which most rows leave at once; as many chunks to each.
  const int64_t most = std::max(2048 / R, 8), few = std::max(256 / R, 8);
  const auto even = [&](int64_t w) { return (nch + (nch + w - 1) / w - 1) / ((nch + w - 1) / w); };
  for (int pass = 0; pass <= kDigits; ++pass)
    hipLaunchKernelGGL(topk_pass_kernel, dim3((unsigned)even(std::min(nch, pass < 2 ? most : few)), (unsigned)R),
                       dim3(kTopkThreads), 0, s, scores, ld_s, n, G, lo, tail, pass, w, st);
  // Workgroups a row: 8 while three a CU hold them all, then fewer (each reads and
  // counts the whole list), but a share of at most 2048 positions each.
  int lp = 3;
  static_assert(kRankShare == 8, "8 = 2^3 workgroups a row");
  while (lp > 0 && (int64_t)R << lp > 3 * 256 && k <= 2048 << (lp - 1)) --lp;
  hipLaunchKernelGGL(topk_rank_kernel, dim3((unsigned)((R + 7) / 8 * 8) << lp), dim3(kRankT), 0, s, scores, ld_s, n, G,
                     R, lo, tail, k, lp, w, idx, val, st);
  FATHOM_LAUNCH_CHECK();
  return FATHOM_OK;
}

}  // namespace fathom
