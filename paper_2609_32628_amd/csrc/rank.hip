// Shared ranking kernels (Algorithm 1; routing appendix).
//
// Every region pair gets a unique 54-bit key: the order-preserving image of its
// float32 score in bits 53..22 and (2^22 - 1 - index) in bits 21..0, so that a
// larger key means "ranked earlier" under (score descending, index ascending).
// With the cumulative quotas cut0 = T16, cut1 = T16 + T8, cut2 = T16 + T8 + T4,
// the pairs of class 16 are exactly those with key >= key of rank cut0, class
// 8 those below it with key >= key of rank cut1, and class 4 those below that
// with key >= key of rank cut2 (1-based ranks; an empty cut matches nothing).
//
// Head scope reads the R^2 scores of a head twice:
//   sample    all workgroups: 32,768 scores of every head (8,192 of heads of up
//             to 362 blocks);
//   bracket   one workgroup per cut: order statistics of the sample bracket
//             every threshold key;
//   collect   all workgroups: counts the keys above each bracket and gathers
//             the keys inside;
//   select    one workgroup per cut: the threshold key, exactly, from the
//             gathered keys (from the scores themselves when the bracket missed
//             or the keys did not fit);
//   rows      classes, lists, counts, and the histogram of the row costs;
//   place     the attention work order from that histogram.
// Long heads count and pick the gathered keys with several workgroups per head
// before select. At R = 1,980 x 24 heads the call takes 286 us (620 with three
// histogram passes over all scores): sample 20, bracket 15, collect 100, count
// and pick 17, select 9, rows 121, place 5; the map's two reads and the results
// are 940 MB. At R = 588 x 12 heads 54 us (77).
// Heads of up to kDirectKeys scores go straight to select. Row scope is one
// launch: a wave per row selects, classifies and writes the lists (R <= 2048;
// longer rows sort their keys in LDS and are classified by a workgroup each).
#include <algorithm>
#include <cmath>
#include <mutex>

#include "common.hpp"
#include "launch.hpp"

namespace da2 {

constexpr uint64_t kNone = ~0ull;
constexpr int kIdxBits = 22;
constexpr uint32_t kIdxMask = (1u << kIdxBits) - 1u;
constexpr uint64_t kMaxKey = (1ull << 54) - 1ull;

// Order-preserving image of a score (-0 ranks like +0).
__device__ inline uint32_t score_bits(float a) {
  const uint32_t u = __float_as_uint(a + 0.0f);
  return u ^ (static_cast<uint32_t>(static_cast<int32_t>(u) >> 31) | 0x80000000u);
}
__device__ inline uint64_t rank_key(float a, uint32_t idx) {
  return (static_cast<uint64_t>(score_bits(a)) << kIdxBits) | static_cast<uint64_t>(kIdxMask - idx);
}

// Four consecutive scores; rows start at any multiple of 4 bytes.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
// Words stored over bytes and 16-bit entries, and read back over the latter.
typedef uint32_t u32u1 __attribute__((aligned(1), may_alias));
typedef uint32_t u32u2 __attribute__((aligned(2), may_alias));
typedef uint32_t u32a __attribute__((may_alias));
// Counts of a row; the lists' base is aligned to 4 bytes only.
typedef int32_t i32x4u __attribute__((ext_vector_type(4), aligned(4), may_alias));

// ---- head scope: threshold keys ------------------------------------------------
constexpr int kBins = 1024;            // bins of a key range
// Samples of a head of M scores: a power of two, and at most M/4 so that their
// scores fit the head's part of the class map (see head_scratch).
__host__ __device__ inline int sample_bits(int64_t M) { return M >= 4 * 32768 + 64 ? 15 : 13; }
constexpr int kMaxPerThread = 32;  // of the bracket's 1024 threads
// Largest head that select handles alone (32 scores per thread and pass; R = 75
// x 12 heads: 18 us for the call). R = 250 took 51 us that way and takes 38
// with a sample.
constexpr int64_t kDirectKeys = 4 * 8192 + 64;
constexpr int kOrderBins = 8192;       // bins of the work order
static_assert(4 * kOrderBins <= kCuts * kRankTailBytes, "the bins fit one head's part of the workspace");
constexpr int kFinal = 448;             // keys select ranks by counting
// A head's words in the workspace: counters 128 bytes apart (keys above each
// bracket, keys gathered, keys picked), then the bins and the picked keys of
// every cut.
constexpr int kAbove = 0, kGathered = 32 * kCuts, kPicked = kGathered + 32;
constexpr int kHeadBins = 256, kPicks = kHeadBins + kCuts * kBins;
static_assert(kPicked + 32 * kCuts <= kHeadBins, "counters fit");
constexpr int kHeadWords = kCuts * 2048;  // workspace words per head
static_assert(kPicks + kCuts * kFinal * 2 <= kHeadWords, "bins and picked keys fit");
// Heads of at least 13 x 2^17 scores (R = 1,306) count and pick their gathered
// keys with kParts workgroups: one compute unit fetches the ~130,000 keys of
// R = 1,980 in 20 us a pass (select 44 us; in parts 8 + 9 + 9). Call without and
// with parts, two thresholds / three: R = 1,448 x 1 head 71.2 / 83.4 and 63.4 /
// 66.7 us, 1,350 x 40 268 / 296.5 and 267 / 288; at R = 1,260 x 40 the two extra
// launches cost what they save (216.5 / 240.7 and 219.9 / 236.0).
constexpr int64_t kPartsKeys = 13 << 17;
constexpr int kParts = 8;

// Inclusive key range cut into kBins bins of 2^shift keys.
__device__ inline int range_shift(uint64_t lo, uint64_t hi) {
  const int bits = 64 - __builtin_clzll((hi - lo) | 1ull);
  return bits > 10 ? bits - 10 : 0;
}

__device__ inline uint32_t wave_sum_u32(uint32_t v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// One wave: narrows [lo, hi] to the bin that holds the k-th largest key of the
// range (h: its histogram), k to the rank inside that bin and cnt to the bin's
// keys; false when the range holds no such key.
__device__ inline bool narrow(const uint32_t* h, uint64_t& lo, uint64_t& hi, int64_t& k, uint32_t& cnt) {
  constexpr int per = kBins / 64;
  const int lane = threadIdx.x & 63;
  uint32_t c[per], local = 0;
#pragma unroll
  for (int q = 0; q < per; ++q) {
    c[q] = h[kBins - 1 - per * lane - q];
    local += c[q];
  }
  uint32_t x = local;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  const int64_t before = (int64_t)x - local;
  const bool mine = before < k && k <= (int64_t)x;
  const uint64_t who = __ballot(mine);
  if (who == 0) return false;
  int bin = 0;
  int64_t run = before;
  uint32_t n = 0;
  if (mine) {
#pragma unroll
    for (int q = 0; q < per; ++q) {
      if (n == 0 && k <= run + (int64_t)c[q]) {
        bin = kBins - 1 - per * lane - q;
        n = c[q];
      }
      if (n == 0) run += c[q];
    }
  }
  const int src = __builtin_ctzll(who);
  bin = __shfl(bin, src, 64);
  cnt = __shfl(n, src, 64);
  k -= __shfl(run, src, 64);
  const int sh = range_shift(lo, hi);
  const uint64_t b0 = lo + ((uint64_t)bin << sh), b1 = b0 + (1ull << sh) - 1ull;
  lo = b0;
  hi = b1 < hi ? b1 : hi;
  return true;
}

// Scratch of a head until classify writes its classes: its part of the class
// map (one byte per pair), 8-byte aligned inside. It holds the sampled scores,
// then the gathered keys.
__device__ inline uint64_t* head_scratch(const RankArgs& args, int bh, int64_t M, uint32_t* keys) {
  const uintptr_t b = reinterpret_cast<uintptr_t>(args.cls + (int64_t)bh * M), a = (b + 7u) & ~(uintptr_t)7u;
  *keys = static_cast<uint32_t>((M - (int64_t)(a - b)) / 8);
  return reinterpret_cast<uint64_t*>(a);
}

// Position of sample j of a head: a hashed place in stratum j of 2^lg equal
// strata, so that no stride of the map repeats in the sample.
__device__ inline uint32_t sample_place(uint32_t j, int64_t M, int lg) {
  const uint64_t p0 = ((uint64_t)j * (uint64_t)M) >> lg, p1 = (((uint64_t)j + 1) * (uint64_t)M) >> lg;
  uint32_t x = (j + 1u) * 0x9E3779B1u;
  x ^= x >> 15;
  x *= 0x85EBCA77u;
  x ^= x >> 13;
  return (uint32_t)(p0 + (((p1 - p0) * (uint64_t)x) >> 32));
}

// Every workgroup fetches 1,024 samples of a head (their image goes to the
// head's scratch): scattered loads of one compute unit are limited by its
// misses in flight, so one workgroup per head took 90 us for 32,768 of them at
// R = 1,980. Also clears what the later launches count into.
__global__ __launch_bounds__(256) void rank_sample_kernel(RankArgs args) {
  const int bh = blockIdx.y, tid = threadIdx.x;
  const int64_t M = (int64_t)args.R * args.R;
  const int lg = sample_bits(M);
  const float* A = args.A + (int64_t)bh * M;
  uint32_t cap;
  uint32_t* out = reinterpret_cast<uint32_t*>(head_scratch(args, bh, M, &cap));
  const uint32_t j0 = blockIdx.x * 1024u + tid;
  float v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = A[sample_place(j0 + 256 * i, M, lg)];
  if (blockIdx.x == 0)
    for (int i = tid; i < kPicks; i += 256) args.hist[(int64_t)bh * kHeadWords + i] = 0u;
  if (blockIdx.x == 0 && bh == 0)
    for (int i = tid; i < kOrderBins; i += 256) args.obins[i] = 0u;
#pragma unroll
  for (int i = 0; i < 4; ++i) out[j0 + 256 * i] = score_bits(v[i]);
}

// Bracket of one threshold key (workgroup (t, head)): a threshold of rank c lies
// between the sample's ranks c S/M -+ (sds standard deviations of a random sample
// + 4), see bracket_sds. The two bounds are narrowed by histograms: the first one is over the
// samples' scores and common to both (four copies, since neighbouring lanes
// often hit one bin); in the second a sample's first bin tells which bound it
// matters to; dense bins and ties take further ones over the keys. A bound is
// done when its bin holds at most 16 samples, and widened to the bin's edge.
__global__ __launch_bounds__(1024) void rank_bracket_kernel(RankArgs args, double sds) {
  constexpr int NB = 2;  // 0: the upper bound, 1: the lower one
  __shared__ uint32_t lh[4][kBins];
  __shared__ uint64_t s_lo[NB], s_hi[NB];
  __shared__ int64_t s_k[NB];
  __shared__ int s_open[NB], s_bin[NB];
  __shared__ uint32_t s_mn[16], s_mx[16];
  const int t = blockIdx.x, bh = blockIdx.y, tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int64_t M = (int64_t)args.R * args.R;
  if (args.cut[t] <= 0 || args.cut[t] >= M) return;
  const int lg = sample_bits(M), per = (1 << lg) / 1024;
  uint32_t cap;
  const uint32_t* in = reinterpret_cast<const uint32_t*>(head_scratch(args, bh, M, &cap));
  uint32_t s[kMaxPerThread];
#pragma unroll
  for (int i = 0; i < kMaxPerThread; ++i) s[i] = i < per ? in[tid + 1024 * i] : 0u;
  for (int i = tid; i < 4 * kBins; i += 1024) (&lh[0][0])[i] = 0u;
  uint32_t mn = 0xFFFFFFFFu, mx = 0u;
#pragma unroll
  for (int i = 0; i < kMaxPerThread; ++i)
    if (i < per) {
      mn = min(mn, s[i]);
      mx = max(mx, s[i]);
    }
  for (int o = 32; o > 0; o >>= 1) {
    mn = min(mn, (uint32_t)__shfl_xor(mn, o, 64));
    mx = max(mx, (uint32_t)__shfl_xor(mx, o, 64));
  }
  if (lane == 0) {
    s_mn[w] = mn;
    s_mx[w] = mx;
  }
  __syncthreads();
  for (int q = 0; q < 16; ++q) {
    mn = min(mn, s_mn[q]);
    mx = max(mx, s_mx[q]);
  }
  if (tid < NB) {
    const double c = (double)args.cut[t], S = (double)(1 << lg), p = c / (double)M;
    const double r = p * S, wd = sds * sqrt(S * p * (1.0 - p)) + 4.0;
    const double rr = tid == 0 ? floor(r - wd) : ceil(r + wd);
    s_open[tid] = rr >= 1.0 && rr <= S;
    s_k[tid] = (int64_t)rr;
    // a bound outside the sample's ranks is the end of the keys
    s_lo[tid] = s_open[tid] ? (uint64_t)mn << kIdxBits : 0ull;
    s_hi[tid] = s_open[tid] ? ((uint64_t)mx << kIdxBits) | kIdxMask : kMaxKey;
  }
  // wave w narrows open bound w from its histogram lh[from]
  auto narrow_bound = [&](int from) {
    uint64_t l = s_lo[w], h = s_hi[w];
    int64_t k = s_k[w];
    uint32_t cnt = 0;
    const uint64_t l0 = l;
    const int sh = range_shift(l, h);
    narrow(lh[from], l, h, k, cnt);  // 1 <= k <= the range's samples always holds
    if (lane == 0) {
      s_lo[w] = l;
      s_hi[w] = h;
      s_k[w] = k;
      s_bin[w] = (int)((l - l0) >> sh);
      if (cnt <= 16u || l == h) s_open[w] = 0;
    }
  };
  const int sh0 = range_shift((uint64_t)mn << kIdxBits, ((uint64_t)mx << kIdxBits) | kIdxMask);
  if (sh0 >= kIdxBits) {  // bins of whole scores (uniform)
    const int ss = sh0 - kIdxBits;
#pragma unroll
    for (int i = 0; i < kMaxPerThread; ++i)
      if (i < per) atomicAdd(&lh[lane & 3][(s[i] - mn) >> ss], 1u);
    __syncthreads();
    lh[0][tid] += lh[1][tid] + lh[2][tid] + lh[3][tid];
    __syncthreads();
    if (w < NB && s_open[w]) narrow_bound(0);
    __syncthreads();
    const int b0 = s_open[0] ? s_bin[0] : -1, b1 = s_open[1] ? s_bin[1] : -1;
    const uint64_t lo0 = s_lo[0], lo1 = s_lo[1];
    const int sh1 = range_shift(lo0, s_hi[0]), sh2 = range_shift(lo1, s_hi[1]);
    for (int i = tid; i < NB * kBins; i += 1024) (&lh[0][0])[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kMaxPerThread; ++i) {
      if (i >= per) continue;
      const int b = (int)((s[i] - mn) >> ss);
      if (b == b0 || b == b1) {
        const uint64_t key = ((uint64_t)s[i] << kIdxBits) | (kIdxMask - sample_place(tid + 1024 * i, M, lg));
        if (b == b0) atomicAdd(&lh[0][(key - lo0) >> sh1], 1u);
        if (b == b1) atomicAdd(&lh[1][(key - lo1) >> sh2], 1u);
      }
    }
    __syncthreads();
    if (w < NB && s_open[w]) narrow_bound(w);
  }
  __syncthreads();
  while (s_open[0] || s_open[1]) {  // uniform: every thread reads the same LDS values
    uint64_t lo[NB], hi[NB];
    int sh[NB];
    bool open[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      lo[b] = s_lo[b];
      hi[b] = s_hi[b];
      sh[b] = range_shift(lo[b], hi[b]);
      open[b] = s_open[b];
    }
    for (int i = tid; i < NB * kBins; i += 1024) (&lh[0][0])[i] = 0u;
    __syncthreads();
#pragma unroll 1
    for (int i = 0; i < per; ++i) {
      const uint32_t j = tid + 1024 * i;
      const uint64_t key = ((uint64_t)in[j] << kIdxBits) | (kIdxMask - sample_place(j, M, lg));
#pragma unroll
      for (int b = 0; b < NB; ++b)
        if (open[b] && key >= lo[b] && key <= hi[b]) atomicAdd(&lh[b][(key - lo[b]) >> sh[b]], 1u);
    }
    __syncthreads();
    if (w < NB && s_open[w]) narrow_bound(w);
    __syncthreads();
  }
  if (tid == 0) {
    args.bracket_lo[bh * kCuts + t] = s_lo[1];
    args.bracket_hi[bh * kCuts + t] = s_hi[0];
  }
}

// Every wave takes 256 scores per step (four per lane), stages the keys inside
// a bracket in its own part of LDS (its fill count is a scalar, so the loop has
// no atomics). They go to the head's list when the part is full or, for all
// waves with one reservation, at the end: thousands of reservations on one
// counter took 50 us for a single head of R = 1,980. Bound by the vector work
// of the compares beside the read of the map. (Counting the brackets'
// histograms here as well, with an atomic per gathered key, cost 110 us on
// R = 1,980 x 24 heads and saved select 16.)
__global__ __launch_bounds__(256) void rank_collect_kernel(RankArgs args, int chunk) {
  constexpr int kStage = 320;
  __shared__ uint64_t stage[4][kStage];
  __shared__ uint32_t s_above[kCuts], s_fill[4], s_base;
  const int bh = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t M = (int64_t)args.R * args.R;
  const float* A = args.A + (int64_t)bh * M;
  uint32_t* hw = args.hist + (int64_t)bh * kHeadWords;
  uint32_t cap;
  uint64_t* list = head_scratch(args, bh, M, &cap);
  if (tid < kCuts) s_above[tid] = 0u;
  uint64_t lo[kCuts], hi[kCuts];
  bool active[kCuts];
#pragma unroll
  for (int t = 0; t < kCuts; ++t) {
    active[t] = args.cut[t] > 0 && args.cut[t] < M;
    lo[t] = args.bracket_lo[bh * kCuts + t];
    hi[t] = args.bracket_hi[bh * kCuts + t];
    if (!active[t]) lo[t] = hi[t] = kNone;  // no key is inside or above
  }
  __syncthreads();
  uint32_t above[kCuts] = {0, 0, 0};
  uint32_t fill = 0;
  // writes the staged keys from list entry base on
  auto write = [&](uint32_t base) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (uint32_t i = lane; i < fill; i += 64)
      if (base + i < cap) list[base + i] = stage[w][i];
    __builtin_amdgcn_wave_barrier();
    fill = 0;
  };
  auto flush = [&]() {
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(hw + kGathered, fill);
    write(__builtin_amdgcn_readfirstlane(base));
  };
  const int64_t e0 = (int64_t)blockIdx.x * chunk, e1 = e0 + chunk < M ? e0 + chunk : M;
  // Brackets that begin and end with whole scores (all but those that split
  // equal scores) need the 32-bit images only: half the compares.
  bool split = false;
  uint32_t lo32[kCuts], hi32[kCuts];
#pragma unroll
  for (int t = 0; t < kCuts; ++t) {
    split = split || (active[t] && ((lo[t] & kIdxMask) != 0 || (hi[t] & kIdxMask) != kIdxMask));
    lo32[t] = (uint32_t)(lo[t] >> kIdxBits);
    hi32[t] = (uint32_t)(hi[t] >> kIdxBits);
  }
  auto visit = [&]<bool SPLIT, bool TAIL>(const float (&x)[4], int64_t i0) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t sb = score_bits(x[e]);
      const bool valid = !TAIL || i0 + e < e1;
      auto key = [&] { return (static_cast<uint64_t>(sb) << kIdxBits) | (kIdxMask - static_cast<uint32_t>(i0 + e)); };
      bool in = false;
#pragma unroll
      for (int t = 0; t < kCuts; ++t) {
        if (!active[t]) continue;
        const bool gt = SPLIT ? key() > hi[t] : sb > hi32[t];
        above[t] += gt && valid ? 1u : 0u;
        // inside: one unsigned compare of the distance from the lower end
        in = in || (SPLIT ? key() - lo[t] <= hi[t] - lo[t] : sb - lo32[t] <= hi32[t] - lo32[t]);
      }
      const uint64_t any = __ballot(in && valid);
      if (any == 0) continue;
      if ((any >> lane) & 1ull)
        stage[w][fill + __builtin_amdgcn_mbcnt_hi((uint32_t)(any >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)any, 0u))] =
            key();
      fill += __builtin_popcountll(any);
      if (fill > kStage - 64) flush();
    }
  };
  // two steps of loads in flight
  for (int64_t b = e0 + 256 * w; b < e1; b += 2048) {
    float x[2][4];
    const bool full = b + 1024 + 256 <= e1;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int64_t i0 = b + 1024 * u + 4 * lane;
      if (full) {
        const f32x4u f = *reinterpret_cast<const f32x4u*>(A + i0);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[u][e] = f[e];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[u][e] = A[i0 + e < M ? i0 + e : M - 1];
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int64_t i0 = b + 1024 * u + 4 * lane;
      if (split) {
        if (full)
          visit.template operator()<true, false>(x[u], i0);
        else
          visit.template operator()<true, true>(x[u], i0);
      } else {
        if (full)
          visit.template operator()<false, false>(x[u], i0);
        else
          visit.template operator()<false, true>(x[u], i0);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < kCuts; ++t) {
    const uint32_t n = wave_sum_u32(above[t]);
    if (lane == 0 && n) atomicAdd(&s_above[t], n);
  }
  if (lane == 0) s_fill[w] = fill;
  __syncthreads();
  if (tid < kCuts && s_above[tid]) atomicAdd(hw + kAbove + 32 * tid, s_above[tid]);
  if (tid == 0) {
    const uint32_t n = s_fill[0] + s_fill[1] + s_fill[2] + s_fill[3];
    s_base = n ? atomicAdd(hw + kGathered, n) : 0u;
  }
  __syncthreads();
  uint32_t base = s_base;
  for (int q = 0; q < w; ++q) base += s_fill[q];
  write(base);
}

// Share of a part in n gathered keys.
__device__ inline void part_share(uint32_t n, uint32_t* i0, uint32_t* i1) {
  *i0 = (uint32_t)((uint64_t)n * blockIdx.x / kParts);
  *i1 = (uint32_t)((uint64_t)n * (blockIdx.x + 1) / kParts);
}

// f(key) for the keys [i0, i1) of a list, all threads of the workgroup.
template <typename F>
__device__ inline void each_key(const uint64_t* list, uint32_t i0, uint32_t i1, F f) {
  constexpr int U = 16;  // loads in flight per thread
  for (uint32_t b = i0 + threadIdx.x; b < i1; b += 1024 * U) {
    uint64_t k[U];
#pragma unroll
    for (int u = 0; u < U; ++u) k[u] = list[min(b + 1024u * u, i1 - 1u)];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (b + 1024u * u < i1) f(k[u]);
  }
}

// Histogram of every bracket over a part of the gathered keys.
__global__ __launch_bounds__(1024) void rank_count_kernel(RankArgs args) {
  __shared__ uint32_t bins[kCuts][kBins];
  const int bh = blockIdx.y, tid = threadIdx.x;
  const int64_t M = (int64_t)args.R * args.R;
  uint32_t* hw = args.hist + (int64_t)bh * kHeadWords;
  uint32_t cap, i0, i1;
  const uint64_t* list = head_scratch(args, bh, M, &cap);
  const uint32_t n = hw[kGathered];
  if (n > cap) return;
  part_share(n, &i0, &i1);
  uint64_t lo[kCuts], span[kCuts];
  int sh[kCuts];
  bool active[kCuts];
#pragma unroll
  for (int t = 0; t < kCuts; ++t) {
    active[t] = args.cut[t] > 0 && args.cut[t] < M;
    lo[t] = args.bracket_lo[bh * kCuts + t];
    span[t] = args.bracket_hi[bh * kCuts + t] - lo[t];
    sh[t] = range_shift(lo[t], lo[t] + span[t]);
    bins[t][tid] = 0u;
  }
  __syncthreads();
  each_key(list, i0, i1, [&](uint64_t key) {
#pragma unroll
    for (int t = 0; t < kCuts; ++t)
      if (active[t] && key - lo[t] <= span[t]) atomicAdd(&bins[t][(key - lo[t]) >> sh[t]], 1u);
  });
  __syncthreads();
#pragma unroll
  for (int t = 0; t < kCuts; ++t)
    if (active[t] && bins[t][tid]) atomicAdd(hw + kHeadBins + t * kBins + tid, bins[t][tid]);
}

// The keys of each threshold's bin, from a part of the gathered keys.
__global__ __launch_bounds__(1024) void rank_pick_kernel(RankArgs args) {
  __shared__ uint64_t fin[kCuts][kFinal];
  __shared__ uint64_t s_lo[kCuts], s_hi[kCuts];
  __shared__ uint32_t s_n[kCuts], s_base[kCuts];
  const int bh = blockIdx.y, tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int64_t M = (int64_t)args.R * args.R;
  uint32_t* hw = args.hist + (int64_t)bh * kHeadWords;
  uint32_t cap, i0, i1;
  const uint64_t* list = head_scratch(args, bh, M, &cap);
  const uint32_t n = hw[kGathered];
  if (n > cap) return;
  part_share(n, &i0, &i1);
  if (w < kCuts) {
    uint64_t l = args.bracket_lo[bh * kCuts + w], h = args.bracket_hi[bh * kCuts + w];
    int64_t k = args.cut[w] - (int64_t)hw[kAbove + 32 * w];
    uint32_t cnt = 0;
    const bool ok = args.cut[w] > 0 && args.cut[w] < M && narrow(hw + kHeadBins + w * kBins, l, h, k, cnt);
    if (lane == 0) {
      s_lo[w] = l;
      s_hi[w] = h;
      // a missed threshold or a bin that is still too long is left to select
      s_n[w] = ok && cnt <= (uint32_t)kFinal ? 0u : ~0u;
    }
  }
  __syncthreads();
  uint64_t lo[kCuts], span[kCuts];
  bool pick[kCuts];
#pragma unroll
  for (int t = 0; t < kCuts; ++t) {
    lo[t] = s_lo[t];
    span[t] = s_hi[t] - lo[t];
    pick[t] = s_n[t] == 0u;
  }
  __syncthreads();  // every thread has read the flags before the counts start
  each_key(list, i0, i1, [&](uint64_t key) {
#pragma unroll
    for (int t = 0; t < kCuts; ++t)
      if (pick[t] && key - lo[t] <= span[t]) {
        const uint32_t pos = atomicAdd(&s_n[t], 1u);  // below kFinal: the bin's count
        if (pos < (uint32_t)kFinal) fin[t][pos] = key;
      }
  });
  __syncthreads();
  if (tid < kCuts && s_n[tid] != ~0u && s_n[tid] > 0u) s_base[tid] = atomicAdd(hw + kPicked + 32 * tid, s_n[tid]);
  __syncthreads();
#pragma unroll
  for (int t = 0; t < kCuts; ++t) {
    uint64_t* out = reinterpret_cast<uint64_t*>(hw + kPicks) + t * kFinal;
    if (pick[t] && (uint32_t)tid < min(s_n[t], (uint32_t)kFinal) && s_base[t] + tid < (uint32_t)kFinal)
      out[s_base[t] + tid] = fin[t][tid];
  }
}

// Threshold key of one cut (workgroup (t, head)). The cut's key range is
// narrowed by histograms of the keys inside it until it holds at most kFinal
// keys; those are then picked out and ranked by counting. The keys are the
// gathered ones, or the head's own scores when it was not sampled, when the
// bracket missed its threshold (which the counts show) or when the list did not
// fit. Keys are unique, so a range shrinks by the bin count with every pass and
// ties cost no more than a few. parted: the count and pick launches went before,
// and usually only the ranking of the picked keys is left.
__global__ __launch_bounds__(1024) void rank_select_kernel(RankArgs args, int sampled, int parted) {
  __shared__ uint32_t bins[kBins];
  __shared__ uint64_t fin[kFinal];
  __shared__ uint64_t s_lo, s_hi;
  __shared__ int64_t s_k;
  __shared__ uint32_t s_n;
  __shared__ int s_open, s_fail;
  __shared__ uint32_t s_mn[16], s_mx[16];
  const int t = blockIdx.x, bh = blockIdx.y, tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int64_t M = (int64_t)args.R * args.R, cut = args.cut[t];
  if (!sampled && t == 0 && bh == 0)
    for (int i = tid; i < kOrderBins; i += 1024) args.obins[i] = 0u;
  uint64_t* out = args.thr + bh * kCuts + t;
  if (cut <= 0 || cut >= M) {  // no pair, or every pair
    if (tid == 0) *out = cut <= 0 ? kNone : 0ull;
    return;
  }
  const float* A = args.A + (int64_t)bh * M;
  const uint32_t* hw = args.hist + (int64_t)bh * kHeadWords;
  uint32_t cap;
  const uint64_t* list = head_scratch(args, bh, M, &cap);
  const uint32_t gathered = sampled ? hw[kGathered] : 0u;
  bool from_list = sampled && gathered <= cap;

  // f(key) for every key of the source
  auto each = [&](auto f) {
    constexpr int U = 16;  // loads in flight per thread
    if (from_list) {
      each_key(list, 0u, gathered, f);
    } else {
      const uint32_t n = (uint32_t)M;
      for (uint32_t i0 = tid; i0 < n; i0 += 1024 * U) {
        float x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = A[min(i0 + 1024u * u, n - 1u)];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (i0 + 1024u * u < n) f(rank_key(x[u], i0 + 1024u * u));
      }
    }
  };
  // the whole key range of the scores
  auto from_scores = [&]() {
    from_list = false;
    uint32_t mn = 0xFFFFFFFFu, mx = 0u;
    each([&](uint64_t k) {
      const uint32_t s = (uint32_t)(k >> kIdxBits);
      mn = min(mn, s);
      mx = max(mx, s);
    });
    for (int o = 32; o > 0; o >>= 1) {
      mn = min(mn, (uint32_t)__shfl_xor(mn, o, 64));
      mx = max(mx, (uint32_t)__shfl_xor(mx, o, 64));
    }
    if (lane == 0) {
      s_mn[w] = mn;
      s_mx[w] = mx;
    }
    __syncthreads();
    if (tid == 0) {
      for (int q = 0; q < 16; ++q) {
        mn = min(mn, s_mn[q]);
        mx = max(mx, s_mx[q]);
      }
      s_lo = (uint64_t)mn << kIdxBits;
      s_hi = ((uint64_t)mx << kIdxBits) | kIdxMask;
      s_k = cut;
      s_open = 1;
      s_fail = 0;
    }
    __syncthreads();
  };

  if (tid == 0) s_n = 0u;
  if (from_list) {
    if (tid == 0) {
      s_lo = args.bracket_lo[bh * kCuts + t];
      s_hi = args.bracket_hi[bh * kCuts + t];
      s_k = cut - (int64_t)hw[kAbove + 32 * t];
      s_open = 1;
      s_fail = 0;
    }
    __syncthreads();
  } else {
    from_scores();
  }
  bool counted = from_list && parted;  // the bracket's histogram is in the workspace
  bool picked = false;
  while (s_open) {  // uniform: every thread reads the same LDS value
    const uint64_t lo = s_lo, span = s_hi - lo;
    const int sh = range_shift(lo, s_hi);
    bins[tid] = counted ? hw[kHeadBins + t * kBins + tid] : 0u;
    __syncthreads();
    if (!counted)
      each([&](uint64_t key) {
        if (key - lo <= span) atomicAdd(&bins[(key - lo) >> sh], 1u);
      });
    __syncthreads();
    if (w == 0) {
      uint64_t l = s_lo, h = s_hi;
      int64_t k = s_k;
      uint32_t cnt = 0;
      const bool ok = narrow(bins, l, h, k, cnt);
      if (lane == 0) {
        if (!ok && from_list) s_fail = 1;  // the bracket missed its threshold
        s_lo = l;
        s_hi = h;
        s_k = k;
        if (cnt <= (uint32_t)kFinal) s_open = 0;
      }
    }
    __syncthreads();
    picked = counted && !s_open && !s_fail;
    counted = false;
    if (s_fail) from_scores();  // (its first barrier follows every thread's read of the flag)
  }
  // the keys of the final range
  const uint64_t lo = s_lo, span = s_hi - lo;
  if (picked) {
    const uint32_t m = min(hw[kPicked + 32 * t], (uint32_t)kFinal);
    if ((uint32_t)tid < m) fin[tid] = (reinterpret_cast<const uint64_t*>(hw + kPicks) + t * kFinal)[tid];
    if (tid == 0) s_n = m;
  } else {
    each([&](uint64_t key) {
      if (key - lo <= span) {
        const uint32_t pos = atomicAdd(&s_n, 1u);  // below kFinal: the range's count
        if (pos < (uint32_t)kFinal) fin[pos] = key;
      }
    });
  }
  __syncthreads();
  const uint32_t n = min(s_n, (uint32_t)kFinal);
  if (tid < n) {
    const uint64_t mine = fin[tid];
    uint32_t g = 0;
    for (uint32_t i = 0; i < n; ++i) g += fin[i] > mine ? 1u : 0u;
    if ((int64_t)g + 1 == s_k) *out = mine;
  }
}

// ---- work order ------------------------------------------------------------------
// Rows are grouped by head and, inside a head, by row parity (two half-heads
// with near-equal cost); each group is sorted most expensive first. Workgroups
// are dispatched round-robin over the 8 XCDs, and the attention launch gives each
// XCD one contiguous segment of the order (about n/8 rows of one or two heads,
// whose K/V then share that XCD's L2), which it walks longest-first; a half-head
// that two segments share is dealt to both by cost (work_entry in attn.hip).
// Bin of row i (cost c) in the work order. 32-bit arithmetic: rows number
// fewer than 2^31 and R <= 65535 (both checked on the host), so c (n4 + n8 +
// n16 <= R blocks at most 3 each) times the bins per group (<= 4096) and the
// rescaled key (< 2^16 x 8192) stay below 2^32.
__device__ inline uint32_t order_key(const RankArgs& args, uint32_t i, int32_t c) {
  const uint32_t R = static_cast<uint32_t>(args.R), BH = static_cast<uint32_t>(args.B * args.H);
  const uint32_t cmax = 3u * R;  // cost of a row with R 4-bit or 16-bit blocks
  const uint32_t groups = 2u * BH;
  const uint32_t nbh = groups < kOrderBins ? kOrderBins / groups : 1u;  // cost bins per group
  const uint32_t bh = i / R, half = (i - bh * R) & 1u;
  const uint32_t bin = static_cast<uint32_t>(c) * (nbh - 1u) / cmax;
  uint32_t key = (2u * bh + half) * nbh + (nbh - 1u - bin);
  if (groups * nbh > kOrderBins) key = key * kOrderBins / (groups * nbh);
  return key;
}

// Attention cost of a row in units of the measured per-tile times (a 4-bit
// NVFP4 or 16-bit tile costs about 1.5 INT8 tiles).
__device__ inline int32_t row_cost(int n4, int n8, int n16) { return 3 * n4 + 2 * n8 + 3 * n16; }

// Work order from the bins that classify counted (each row's place inside its
// bin is in cost): every workgroup scans the bins for itself, so the launch
// needs no second phase, and places 1024 rows.
__global__ __launch_bounds__(1024) void rank_place_kernel(RankArgs args) {
  __shared__ uint32_t first[kOrderBins];
  __shared__ uint32_t part[16];
  constexpr int per = kOrderBins / 1024;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint32_t n = static_cast<uint32_t>(args.B * args.H) * static_cast<uint32_t>(args.R);
  uint32_t c[per], s = 0;
#pragma unroll
  for (int q = 0; q < per; ++q) {
    c[q] = args.obins[tid * per + q];
    s += c[q];
  }
  uint32_t x = s;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) part[w] = x;
  __syncthreads();
  uint32_t run = x - s;
  for (int q = 0; q < w; ++q) run += part[q];
#pragma unroll
  for (int q = 0; q < per; ++q) {
    first[tid * per + q] = run;
    run += c[q];
  }
  __syncthreads();
  const uint32_t i = blockIdx.x * 1024u + tid;
  if (i < n) {
    const i32x4u k = reinterpret_cast<const i32x4u*>(args.counts)[i];
    args.order[first[order_key(args, i, row_cost(k.x, k.y, k.z))] + (uint32_t)args.cost[i]] = (int32_t)i;
  }
}

// Work order of row scope, where every row of a group costs the same: head, row
// parity, row.
__device__ inline void place_row(const RankArgs& args, int64_t row) {
  const int R = args.R, a = (int)(row % R);
  args.order[row - a + (a & 1 ? (R + 1) / 2 : 0) + a / 2] = (int32_t)row;
}

__device__ inline void write_meta(const RankArgs& args, int64_t row) {
  if (row != 0) return;
  args.meta[0] = args.B * args.H * args.R;
  args.meta[1] = 0;  // error flags of da2_mixed_attn calls on these lists
}

// ---- classes and lists, one wave per row ------------------------------------------
// Writes row's classes, ascending lists (4-bit, 8-bit, 16-bit: the phase order
// of the attention) and counts. xs[st]: the class ranks (0 skip, 1: 4, 2: 8, 3:
// 16 bits) of the lane's four pairs 256 st + 4 lane + e, one per byte. keys_l:
// R 16-bit words of LDS of this wave.
template <int ST>
__device__ inline void write_row(const RankArgs& args, int64_t row, const uint32_t (&xs)[ST], uint16_t* keys_l) {
  const int lane = threadIdx.x & 63, R = args.R;
  uint8_t* cls = args.cls + row * R;
  uint32_t cnt[ST];
  uint32_t n4 = 0, n8 = 0, n16 = 0;
#pragma unroll
  for (int st = 0; st < ST; ++st) {
    // counts of the classes 4, 8, 16 in 10, 10 and 12 bits, from the bytes'
    // ranks of at least 1, 2 and 3
    const uint32_t one = 0x01010101u, x = xs[st], g2 = (x >> 1) & one, g1 = (x | g2) & one, g3 = x & g2;
    const uint32_t c1 = __builtin_amdgcn_udot4(g1, one, 0u, false), c2 = __builtin_amdgcn_udot4(g2, one, 0u, false),
                   c3 = __builtin_amdgcn_udot4(g3, one, 0u, false);
    cnt[st] = (c1 - c2) | ((c2 - c3) << 10) | (c3 << 20);
    const int b = 256 * st + 4 * lane;
    const uint32_t c = __builtin_amdgcn_perm(0u, 0x10080400u, xs[st]);
    if (b + 3 < R) {
      *reinterpret_cast<u32u1*>(cls + b) = c;
    } else {
      for (int e = 0; b + e < R; ++e) cls[b + e] = static_cast<uint8_t>(c >> (8 * e));
    }
  }
  // inclusive scans of the packed counts, one per step (at most 256 of a class)
  uint32_t tot[ST];
#pragma unroll
  for (int st = 0; st < ST; ++st) {
    uint32_t x = cnt[st];
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    tot[st] = __builtin_amdgcn_readlane(x, 63);
    cnt[st] = x - cnt[st];
    n4 += tot[st] & 1023u;
    n8 += (tot[st] >> 10) & 1023u;
    n16 += tot[st] >> 20;
  }
  uint32_t b4 = 0, b8 = n4, b16 = n4 + n8;
#pragma unroll
  for (int st = 0; st < ST; ++st) {
    uint32_t p4 = b4 + (cnt[st] & 1023u), p8 = b8 + ((cnt[st] >> 10) & 1023u), p16 = b16 + (cnt[st] >> 20);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t x = (xs[st] >> (8 * e)) & 3u;
      const uint32_t p = x == 1u ? p4 : (x == 2u ? p8 : p16);
      if (x) keys_l[p] = static_cast<uint16_t>(256 * st + 4 * lane + e);
      p4 += x == 1u;
      p8 += x == 2u;
      p16 += x == 3u;
    }
    b4 += tot[st] & 1023u;
    b8 += (tot[st] >> 10) & 1023u;
    b16 += tot[st] >> 20;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  uint16_t* keys = args.keys + row * R;
  const int n = (int)(n4 + n8 + n16);
  for (int i = 2 * lane; i < n; i += 128) {
    if (i + 1 < n)
      *reinterpret_cast<u32u2*>(keys + i) = *reinterpret_cast<const u32a*>(keys_l + i);
    else
      keys[i] = keys_l[i];
  }
  if (lane == 0) {
    reinterpret_cast<i32x4u*>(args.counts)[row] = i32x4u{(int)n4, (int)n8, (int)n16, 0};
    write_meta(args, row);
    if (args.scope == DA2_SCOPE_HEAD) {
      const int32_t cost = row_cost((int)n4, (int)n8, (int)n16);
      args.cost[row] = (int32_t)atomicAdd(args.obins + order_key(args, (uint32_t)row, cost), 1u);
    } else {
      place_row(args, row);
    }
  }
}

// Four scores of a row (b + e < R), or 0 beyond its end.
__device__ inline void load_scores(const float* A, int b, int R, float (&x)[4]) {
  if (b + 3 < R) {
    const f32x4u f = *reinterpret_cast<const f32x4u*>(A + b);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = f[e];
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = b + e < R ? A[b + e] : 0.0f;
  }
}

// Head scope, R <= 256 ST: a pair's class from the head's threshold keys. In a
// row other than the one that holds a threshold's index, comparing the 32-bit
// scores decides: equal scores count before that row and not after it.
template <int ST>
__global__ __launch_bounds__(256) void rank_rows_head_kernel(RankArgs args) {
  __shared__ __align__(8) uint16_t keys_l[4][256 * ST];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, R = args.R;
  const int64_t row = (int64_t)blockIdx.x * 4 + w;
  if (row >= (int64_t)args.B * args.H * R) return;
  const int bh = (int)(row / R), a = (int)(row - (int64_t)bh * R);
  const float* A = args.A + row * R;
  float x[ST][4];
#pragma unroll
  for (int st = 0; st < ST; ++st) load_scores(A, 256 * st + 4 * lane, R, x[st]);
  // scores at or above from[t] are in; in the threshold's own row, of the
  // scores equal to it those at columns up to last[t] (so, too, where no image
  // lies above the threshold's, that of a NaN of all ones)
  uint32_t from[kCuts], t32[kCuts];
  int last[kCuts], empty = 0;
  bool own = false;
#pragma unroll
  for (int t = 0; t < kCuts; ++t) {
    const uint64_t thr = args.thr[bh * kCuts + t];
    empty += thr == kNone;
    t32[t] = (uint32_t)(thr >> kIdxBits);
    const int64_t c = (int64_t)(kIdxMask - ((uint32_t)thr & kIdxMask)) - (int64_t)a * R;
    last[t] = (int)(c < -1 ? -1 : (c > R ? R : c));
    own = own || (thr != kNone && last[t] < R - 1 && (last[t] >= 0 || t32[t] == 0xFFFFFFFFu));
    from[t] = last[t] < 0 ? t32[t] + 1u : t32[t];
  }
  uint32_t xs[ST];
  // E: empty cuts (the first ones, since the cuts are cumulative)
  auto ranks = [&]<int E, bool OWN>() {
#pragma unroll
    for (int st = 0; st < ST; ++st) {
      xs[st] = 0;
      const int b = 256 * st + 4 * lane;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t s = score_bits(x[st][e]);
        uint32_t r = 0;
#pragma unroll
        for (int t = E; t < kCuts; ++t)
          r += (OWN ? s > t32[t] || (s == t32[t] && b + e <= last[t]) : s >= from[t]) ? 1u : 0u;
        xs[st] |= r << (8 * e);
      }
      if (256 * st + 256 > R) {  // the row's last step: no class beyond its end
        const int n = R - b;
        xs[st] = n >= 4 ? xs[st] : (n <= 0 ? 0u : xs[st] & ((1u << (8 * n)) - 1u));
      }
    }
  };
  auto ranks_e = [&]<int E>() {
    if (own)
      ranks.template operator()<E, true>();
    else
      ranks.template operator()<E, false>();
  };
  if (empty == 0)
    ranks_e.template operator()<0>();
  else if (empty == 1)
    ranks_e.template operator()<1>();
  else if (empty == 2)
    ranks_e.template operator()<2>();
  else
    ranks_e.template operator()<3>();
  write_row<ST>(args, row, xs, keys_l[w]);
}

// Row scope, R <= 256 ST: the wave finds each cut's threshold score by bisecting
// the bits of the scores' images (counts over the wave, stopping as soon as a
// bound splits off exactly the quota), takes equal scores in index order, and
// writes the row. Nothing leaves the registers but the results. Against a
// bitonic sort of every row's keys in LDS: R = 588 x 12 heads 210 -> 21 us,
// R = 1,980 x 24 heads 2,970 -> 284 us for the call.
template <int ST>
__global__ __launch_bounds__(256) void rank_rows_row_kernel(RankArgs args) {
  __shared__ __align__(8) uint16_t keys_l[4][256 * ST];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, R = args.R;
  const int64_t row = (int64_t)blockIdx.x * 4 + w;
  if (row >= (int64_t)args.B * args.H * R) return;
  const float* A = args.A + row * R;
  float x[ST][4];
#pragma unroll
  for (int st = 0; st < ST; ++st) load_scores(A, 256 * st + 4 * lane, R, x[st]);
  uint32_t s[ST][4];
  uint32_t mn = 0xFFFFFFFFu, mx = 0u;
#pragma unroll
  for (int st = 0; st < ST; ++st)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s[st][e] = score_bits(x[st][e]);
      if (256 * st + 4 * lane + e < R) {
        mn = min(mn, s[st][e]);
        mx = max(mx, s[st][e]);
      } else {
        s[st][e] = 0u;  // below every bound that is tried (a set bit each)
      }
    }
  for (int o = 32; o > 0; o >>= 1) {
    mn = min(mn, (uint32_t)__shfl_xor(mn, o, 64));
    mx = max(mx, (uint32_t)__shfl_xor(mx, o, 64));
  }
  mn = __builtin_amdgcn_readfirstlane(mn);
  mx = __builtin_amdgcn_readfirstlane(mx);
  uint32_t xs[ST];
#pragma unroll
  for (int st = 0; st < ST; ++st) xs[st] = 0;
#pragma unroll 1
  for (int t = 0; t < kCuts; ++t) {
    const int c = (int)args.cut[t];
    if (c <= 0) continue;
    // v: largest score image with at least c scores at or above it
    const int top = mn == mx ? -1 : 31 - __builtin_clz(mn ^ mx);
    uint32_t v = top < 0 ? mn : (mn >> top >> 1) << top << 1;
    int ge = R;  // scores at or above v (all of them, from the common prefix)
    for (int bit = top; bit >= 0 && ge != c; --bit) {
      const uint32_t tv = v | (1u << bit);
      int n = 0;
#pragma unroll
      for (int st = 0; st < ST; ++st)
#pragma unroll
        for (int e = 0; e < 4; ++e) n += __builtin_popcountll(__ballot(s[st][e] >= tv));
      if (n >= c) {
        v = tv;
        ge = n;
      }
    }
    if (ge == c) {  // everything at or above v
#pragma unroll
      for (int st = 0; st < ST; ++st)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          xs[st] += (s[st][e] >= v && 256 * st + 4 * lane + e < R ? 1u : 0u) << (8 * e);
    } else {  // ties at v: the first (c - those above) of them in index order
      int above = 0;
#pragma unroll
      for (int st = 0; st < ST; ++st)
#pragma unroll
        for (int e = 0; e < 4; ++e) above += __builtin_popcountll(__ballot(s[st][e] > v));
      int left = c - above;
#pragma unroll
      for (int st = 0; st < ST; ++st) {
        bool eq[4];
        uint32_t mine = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          eq[e] = s[st][e] == v && 256 * st + 4 * lane + e < R;
          mine += eq[e];
        }
        uint32_t y = mine;
        for (int o = 1; o < 64; o <<= 1) {
          const uint32_t z = __shfl_up(y, o, 64);
          if (lane >= o) y += z;
        }
        int rank = (int)(y - mine);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          xs[st] += (s[st][e] > v || (eq[e] && rank < left) ? 1u : 0u) << (8 * e);
          rank += eq[e];
        }
        left -= (int)__builtin_amdgcn_readlane(y, 63);
      }
    }
  }
  write_row<ST>(args, row, xs, keys_l[w]);
}

// ---- long rows (row scope, R > 2048) ------------------------------------------------
// Row scope: sort each row's keys descending in LDS, read the threshold keys.
__global__ __launch_bounds__(256) void rank_row_select_kernel(RankArgs args, int P) {
  extern __shared__ uint64_t sk[];
  const int a = blockIdx.x, bh = blockIdx.y, R = args.R;
  const float* A = args.A + ((int64_t)bh * R + a) * R;
  for (int i = threadIdx.x; i < P; i += 256) sk[i] = i < R ? rank_key(A[i], i) : 0ull;
  __syncthreads();
  for (int k = 2; k <= P; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = threadIdx.x; i < P; i += 256) {
        const int l = i ^ j;
        if (l > i) {
          const bool desc = (i & k) == 0;
          const uint64_t x = sk[i], y = sk[l];
          if (desc ? (x < y) : (x > y)) {
            sk[i] = y;
            sk[l] = x;
          }
        }
      }
      __syncthreads();
    }
  }
  if (threadIdx.x < kCuts) {
    const int t = threadIdx.x;
    const int64_t want = args.cut[t];
    args.thr[((int64_t)bh * R + a) * kCuts + t] = want > 0 ? sk[want - 1] : kNone;
  }
}

// Exclusive prefix sum of 64-bit values over a 256-thread block.
__device__ inline uint64_t block_exscan_u64(uint64_t v, uint64_t* sh, uint64_t* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint64_t x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh[w] = x;
  __syncthreads();
  uint64_t base = 0;
  for (int q = 0; q < w; ++q) base += sh[q];
  *total = sh[0] + sh[1] + sh[2] + sh[3];
  __syncthreads();
  return base + x - v;
}

// Classes, ascending per-row lists (4-bit, then 8-bit, then 16-bit: the phase
// order of the attention), counts and work order; one workgroup per row. The
// row's scores are staged in LDS (R floats, dynamic) with coalesced loads;
// thread i then owns the contiguous run of key blocks [i E, (i + 1) E),
// E = ceil(R / 256): it classifies its run, a block-wide scan of the packed
// per-class counts (21 bits each) gives every class's write offset, and a second
// walk over the run writes the lists.
__global__ __launch_bounds__(256) void rank_classify_kernel(RankArgs args) {
  extern __shared__ float srow[];
  __shared__ uint64_t sh[4];
  const int a = blockIdx.x, bh = blockIdx.y, R = args.R, tid = threadIdx.x;
  const int64_t row = (int64_t)bh * R + a;
  const float* A = args.A + row * R;
  // eight loads in flight per thread (indices past the row read its last entry)
  for (int b0 = tid; b0 < R; b0 += 256 * 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = A[min(b0 + 256 * u, R - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (b0 + 256 * u < R) srow[b0 + 256 * u] = v[u];
  }
  __syncthreads();
  const uint64_t* thr = args.thr + row * kCuts;
  const uint64_t t16 = thr[0], t8 = thr[1], t4 = thr[2];
  uint8_t* cls = args.cls + row * R;
  uint16_t* keys = args.keys + row * R;
  auto class_of = [&](int b) -> int {
    const uint64_t key = rank_key(srow[b], static_cast<uint32_t>(b));
    return key >= t16 ? 16 : (key >= t8 ? 8 : (key >= t4 ? 4 : 0));
  };
  constexpr int kF = 21;
  constexpr uint64_t kM = (1ull << kF) - 1ull;
  auto field = [](int c) -> uint64_t {
    return c == 4 ? 1ull : (c == 8 ? (1ull << kF) : (c == 16 ? (1ull << (2 * kF)) : 0ull));
  };
  const int E = (R + 255) / 256;
  const int b0 = min(R, tid * E), b1 = min(R, b0 + E);
  uint64_t cnt = 0;
  for (int b = b0; b < b1; ++b) {
    const int c = class_of(b);
    cls[b] = static_cast<uint8_t>(c);
    cnt += field(c);
  }
  uint64_t tot;
  const uint64_t before = block_exscan_u64(cnt, sh, &tot);
  const uint32_t n4 = static_cast<uint32_t>(tot & kM), n8 = static_cast<uint32_t>((tot >> kF) & kM),
                 n16 = static_cast<uint32_t>((tot >> (2 * kF)) & kM);
  uint32_t p4 = static_cast<uint32_t>(before & kM);
  uint32_t p8 = n4 + static_cast<uint32_t>((before >> kF) & kM);
  uint32_t p16 = n4 + n8 + static_cast<uint32_t>((before >> (2 * kF)) & kM);
  for (int b = b0; b < b1; ++b) {
    const int c = class_of(b);
    if (c == 4)
      keys[p4++] = static_cast<uint16_t>(b);
    else if (c == 8)
      keys[p8++] = static_cast<uint16_t>(b);
    else if (c == 16)
      keys[p16++] = static_cast<uint16_t>(b);
  }
  if (tid == 0) {
    args.counts[row * 4 + 0] = n4;
    args.counts[row * 4 + 1] = n8;
    args.counts[row * 4 + 2] = n16;
    args.counts[row * 4 + 3] = 0;
    write_meta(args, row);
    place_row(args, row);
  }
}

// Fixed device scratch for callers that cannot allocate (da2_rank_assign_noalloc):
// every workspace array of the ranking lives here instead of in a caller
// buffer. Each device holds its own copy for the life of the process; calls
// on one device share it, so such calls must not overlap on that device. The
// kernels clear what must start at zero (the first launch of head scope), so no state from
// an earlier call is read.
static __device__ __align__(256) uint8_t scratch[kRankScratchBytes];

// Device address of this device's copy of the scratch array, looked up once
// per device with that device current and then reused. In host code the
// array's name is only a stand-in for the symbol, never a device address.
hipError_t rank_scratch_address(void** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (addr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *out = addr[dev];
  return hipSuccess;
}

// Half-width of the brackets in standard deviations of a sample's rank: 4 (a
// bracket misses one threshold in 16,000), or what lets the gathered keys fill
// 0.88 of the list, M/8 keys, if the brackets of all cuts are expected to hold
// more (a bracket holds 23 samples on top: 4 and half a bin of 16 at either end).
// That concerns small heads with three cuts in the middle of the ranks: 8,192
// samples, 30/20/20% of the pairs, 3.2. With 4 their lists overflowed and select
// read the scores: R = 362 x 12 heads 92 us, now 43; 0.88 leaves four
// standard deviations of the number gathered.
double bracket_sds(const RankArgs& args, int64_t M) {
  const double S = (double)(1 << sample_bits(M));
  double sd = 0.0, room = 0.88 * S / 8.0;
  for (int t = 0; t < kCuts; ++t)
    if (args.cut[t] > 0 && args.cut[t] < M) {
      const double p = (double)args.cut[t] / (double)M;
      sd += std::sqrt(S * p * (1.0 - p));
      room -= 23.0;
    }
  return sd > 0.0 ? std::min(4.0, room / (2.0 * sd)) : 4.0;
}

template <int ST>
void launch_rows(const RankArgs& args, hipStream_t stream) {
  const dim3 grid((unsigned)(((int64_t)args.B * args.H * args.R + 3) / 4));
  if (args.scope == DA2_SCOPE_HEAD)
    hipLaunchKernelGGL(rank_rows_head_kernel<ST>, grid, dim3(256), 0, stream, args);
  else
    hipLaunchKernelGGL(rank_rows_row_kernel<ST>, grid, dim3(256), 0, stream, args);
}

hipError_t launch_rank(const RankArgs& args, hipStream_t stream) {
  const int BH = args.B * args.H, R = args.R;
  const int64_t rows = (int64_t)BH * R;
  if (args.scope == DA2_SCOPE_ROW && R > 2048) {
    int P = 1;
    while (P < R) P <<= 1;
    hipLaunchKernelGGL(rank_row_select_kernel, dim3(R, BH), dim3(256), P * sizeof(uint64_t), stream, args, P);
    hipLaunchKernelGGL(rank_classify_kernel, dim3(R, BH), dim3(256), R * sizeof(float), stream, args);
    return hipGetLastError();
  }
  if (args.scope == DA2_SCOPE_HEAD) {
    const int64_t M = (int64_t)R * R;
    const bool sampled = M > kDirectKeys;
    if (sampled) {
      hipLaunchKernelGGL(rank_sample_kernel, dim3((1 << sample_bits(M)) / 1024, BH), dim3(256), 0, stream, args);
      hipLaunchKernelGGL(rank_bracket_kernel, dim3(kCuts, BH), dim3(1024), 0, stream, args, bracket_sds(args, M));
      // 4,096 keys per workgroup, more where that makes over 4,096 workgroups
      const int64_t per = (BH * M / 4096 + 2047) / 2048 * 2048;
      const int chunk = (int)(per < 4096 ? 4096 : per);
      hipLaunchKernelGGL(rank_collect_kernel, dim3((unsigned)((M + chunk - 1) / chunk), BH), dim3(256), 0, stream, args,
                         chunk);
    }
    const bool parted = M >= kPartsKeys;
    if (parted) {
      hipLaunchKernelGGL(rank_count_kernel, dim3(kParts, BH), dim3(1024), 0, stream, args);
      hipLaunchKernelGGL(rank_pick_kernel, dim3(kParts, BH), dim3(1024), 0, stream, args);
    }
    hipLaunchKernelGGL(rank_select_kernel, dim3(kCuts, BH), dim3(1024), 0, stream, args, (int)sampled, (int)parted);
  }
  // steps of 256 pairs a wave holds; a row with 4, 6 or 7 steps takes the next
  // larger form (forms of their own, 12 heads: R = 1,024 head scope 97.3 -> 95.8,
  // row scope 62.5 -> 53.3 us; 1,536 133.7 -> 129.2, 144.9 -> 110.3; each adds
  // 48 KB of code)
  const int st = (R + 255) / 256;
  if (st <= 1)
    launch_rows<1>(args, stream);
  else if (st <= 2)
    launch_rows<2>(args, stream);
  else if (st <= 3)
    launch_rows<3>(args, stream);
  else if (st <= 5)
    launch_rows<5>(args, stream);
  else
    launch_rows<8>(args, stream);
  if (args.scope == DA2_SCOPE_HEAD)
    hipLaunchKernelGGL(rank_place_kernel, dim3((unsigned)((rows + 1023) / 1024)), dim3(1024), 0, stream, args);
  return hipGetLastError();
}

}  // namespace da2
