// Ordering inside the applications in one launch (Alg. 1 "requests in g sorted by priority"; Sec. 5.3.2 with subgroups), for
// windows of up to kRankMax requests.
//
// A workgroup owns kRanks consecutive places of an application's service order.  From a sample of the application's keys (all of
// them, where they are few) it finds the range of keys that holds its places for all but certain, reads all keys, counts those before the
// range and collects those inside it in LDS, and puts these in order.  No workgroup waits for another or reads what another has
// written.  A key with the request's position behind it is unique, so the order is stable.
//
// Both the range and the order inside it come from counting in bins of equal width (a monotone map of the key: any such map
// gives the right order, how even the bins are decides the time alone).  A request's place among those collected is its bin's
// first one and the number of smaller ones in that bin.  Where that does not do:
//   * bins that hold too much (keys that are equal, or close beside some that are far off): every bin is divided into as many as it has
//     requests, between its least and greatest key, or by position where all its keys are equal;
//   * bins that are crowded all the same: a sorting network;
//   * a range that misses a place, or holds more than LDS does: the keys at its ends are found exactly by counting digits of eleven bits
//     (places among equal keys by position).
// Bound by dependent trips to memory (descriptor, keys, records; of longer applications one for the positions collected) and by the counting and
// comparing, of which every workgroup of an application does all.  Kernel, us, where runs and merges took as many launches as given before:
// 65,536 requests of eight applications 9.3 (three: 18.2), 4,096 of three 5.7 (two: 12.7).  A workgroup of 8,192 keys of its application: sample
// in registers 1.4, counted 1.9, all keys tested and the range collected 2.0, counted again 1.1, in place 1.2; each 8,192 more 1.35 (1.5 when every
// turn asked for its own places in LDS: one application of 65,536 requests 38.0 -> 36.8 us per call, three of 100,000 38.7 -> 38.2).
#pragma once
#include "sp_sort.h"

namespace sp {

constexpr int kRankThreads = 1024;
constexpr int kRankWaves = kRankThreads / kWave;
constexpr int kRanks = 512;                     // places per workgroup
constexpr int kRankBins = 4096;                 // (four per thread)
constexpr int kRankItems = 8;                   // keys a thread holds at a time
constexpr int kRankHeld = kRankItems * kRankThreads;      // ... all of an application's, or the sample
constexpr int kRankAll = 4096;                  // applications of up to this many are collected whole
constexpr int kRankCap = 7168;                  // requests collected in LDS
constexpr int kRankOwn = kRankCap / kRankThreads;
constexpr int kRankMates = 64;                  // fullest bin whose requests are compared one by one ...
constexpr int kRankMatesLast = 512;             // ... after a division (few are as full: places next to another key's)
constexpr int kRankMax = 106496;                // longest window (see one_launch_order)
constexpr int kRankMaxFew = 65536;              // ... of one or two applications
constexpr int kRankPosBits = 17;                // label, key and position inside the application are one word
constexpr int kRankLabels = 1 << (32 - kRankPosBits);     // subgroup labels
static_assert(kRankBins == 4 * kRankThreads && kRankCap <= 2 * kRankBins && kRankHeld <= 2 * kRankBins, "shares of a thread; bins of a division");
static_assert(kRankMax < 1 << kRankPosBits, "positions, and the one behind the last");

// A request as one word: label (with subgroups), key, position in the application.
typedef unsigned long long Ranked;
__device__ __forceinline__ Ranked ranked(uint32_t label, uint32_t key, int pos) {
  return ((Ranked)label << (32 + kRankPosBits)) | ((Ranked)key << kRankPosBits) | (Ranked)(uint32_t)pos;
}
__device__ __forceinline__ uint32_t ranked_key(Ranked e) { return (uint32_t)(e >> kRankPosBits); }
__device__ __forceinline__ int ranked_pos(Ranked e) { return (int)((uint32_t)e & ((1u << kRankPosBits) - 1u)); }
__device__ __forceinline__ uint32_t ranked_label(Ranked e) { return (uint32_t)(e >> (32 + kRankPosBits)); }

// What a key is counted under: a number of bins in floating point, rounded on the way, which keeps the order; what lies outside goes to
// the ends.  With subgroups the labels, and inside each the keys; while there are bins for all labels, none has requests of two.  The
// labels are the sample's.  Requests of greater ones, which it may have missed, have bins behind all of its labels' (at least the last one, and
// there whatever their labels are).
template <bool SPLIT>
struct RankBins {
  uint32_t least, label_high;
  float scale, per_label, first, finer;         // (then bins from `first` on, `finer` of them for one)
  __device__ __forceinline__ void over(uint32_t low, uint32_t high, uint32_t top_label) {
    least = low;
    label_high = top_label;
    constexpr float kMost = (float)(kRankBins - 1);
    const float labels = (float)(top_label + 1u);
    per_label = labels > kMost ? kMost / labels : floorf(kMost / labels);
    scale = (SPLIT ? per_label : (float)kRankBins) / ((float)(high - low) + 1.0f);
    first = 0.f;
    finer = 1.f;
  }
  __device__ __forceinline__ float at(uint32_t label, uint32_t key) const {
    const float v = (float)(max(key, least) - least) * scale;
    // (a label's last bins end a thousandth early: the sum is never rounded to the next label's first)
    if constexpr (SPLIT) return fmaf((float)label, per_label, fminf(v, fmaxf(per_label - 0.001f, 0.f)));
    else return v;
  }
  __device__ __forceinline__ bool beyond(uint32_t label) const { return SPLIT && label > label_high; }
  __device__ __forceinline__ uint32_t operator()(uint32_t label, uint32_t key) const { return whole(at(label, key)); }
  // (ends first: a number outside of what an integer holds has no integer)
  static __device__ __forceinline__ uint32_t whole(float v) { return (uint32_t)__builtin_amdgcn_fmed3f(v, 0.f, (float)(kRankBins - 1)); }
  __device__ __forceinline__ uint32_t fine(Ranked e) const {
    return whole((at(ranked_label(e), ranked_key(e)) - first) * finer);
  }
};

// Exclusive prefix sums of the bins, in place; the caller's barrier stands before, one stands behind.  cnt and beg: this thread's four.
__device__ __forceinline__ void rank_scan(uint32_t* bins, uint32_t* wave_sum, uint32_t (&cnt)[4], uint32_t (&beg)[4]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint4* const mine = reinterpret_cast<uint4*>(bins) + tid;
  const uint4 c = *mine;
  cnt[0] = c.x; cnt[1] = c.y; cnt[2] = c.z; cnt[3] = c.w;
  const uint32_t sum = c.x + c.y + c.z + c.w, incl = wave_scan_incl(sum);
  if (lane == kWave - 1) wave_sum[wave] = incl;
  __syncthreads();
  const uint32_t w = lane < kRankWaves ? wave_sum[lane] : 0u, wi = wave_scan_incl<true>(w);    // (sixteen: one row)
  const uint32_t before = __builtin_amdgcn_readlane((int)(wi - w), __builtin_amdgcn_readfirstlane(wave));
  beg[0] = before + incl - sum;
  beg[1] = beg[0] + c.x;
  beg[2] = beg[1] + c.y;
  beg[3] = beg[2] + c.z;
  *mine = make_uint4(beg[0], beg[1], beg[2], beg[3]);
  __syncthreads();
}

// Sorts the first n words of s by Batcher's odd-even merging network, which takes any n: all of its comparisons put the smaller one first.
__device__ __forceinline__ void rank_network(Ranked* s, int n) {
  __syncthreads();
  for (int p = 1; p < n; p *= 2)
    for (int k = p; k >= 1; k /= 2) {
      const int skip = k % p;
      for (int t = threadIdx.x; 2 * t < n + 2 * k; t += kRankThreads) {
        const int i = skip + 2 * k * (t / k) + t % k, j = i + k;
        if (j < n && i / (2 * p) == j / (2 * p)) {
          const Ranked a = s[i], b = s[j];
          if (a > b) { s[i] = b; s[j] = a; }
        }
      }
      __syncthreads();
    }
}

// The bins divided: where a request of bin b lies in the bins of a second counting.  start: the first counting's prefix sums, and its total
// behind them; low, high: the bins' least and greatest keys.  Keys that the first counting has not seen keep their order too.
struct RankDivision {
  const uint32_t *start, *low, *high;
  float per_pos;                // 1 / size of the application
  int half;                     // 1: two places to a bin (of more than kRankBins)
  __device__ __forceinline__ uint32_t operator()(uint32_t b, uint32_t key, int pos) const {
    const uint32_t first = start[b], n = start[b + 1] - first, lo = low[b], hi = high[b];
    if (n == 0u || key < lo) return first >> half;
    const float part = lo == hi ? (float)pos * per_pos : (float)(key - lo) * __builtin_amdgcn_rcpf((float)(hi - lo) + 1.0f);
    return (first + (key > hi ? n - 1u : min((uint32_t)(part * (float)n), n - 1u))) >> half;
  }
};

template <bool SPLIT>
__global__ __launch_bounds__(kRankThreads) void k_order(SortPlan sp, const uint32_t* __restrict__ keys, const int32_t* __restrict__ labels,
                                                        uint32_t* __restrict__ label_out, int n, Window w) {
  __shared__ __align__(16) uint32_t bins[kRankBins + 4];
  __shared__ uint32_t bin_low[kRankBins], bin_high[kRankBins];
  __shared__ __align__(16) Ranked held[kRankCap];
  __shared__ uint32_t wave_sum[kRankWaves], wave_low[kRankWaves], wave_high[kRankWaves], wave_label[kRankWaves];
  __shared__ uint32_t bin_s[2], beg_s[2], cnt_s[2], n_held, n_before, crowded[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // units of the same application on the same die
  const int unit = (blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds;
  const int4 desc = sp.desc[unit];                              // (the array covers the launch)
  const int units = sp.unit_start[sp.nseg], nv = sp.seg[sp.nseg];
  loaded_here(desc.x); loaded_here(desc.y); loaded_here(desc.z); loaded_here(units); loaded_here(nv);
  const auto clear_bins = [&](uint32_t* b) { reinterpret_cast<uint4*>(b)[tid] = make_uint4(0u, 0u, 0u, 0u); };
  clear_bins(bins);
  if (tid == 0) n_held = n_before = crowded[0] = crowded[1] = 0u;
  // the per-request outputs (by request id) and what lies behind the valid requests: nobody waits for these
  const auto rest = [&] {
    const int i = blockIdx.x * kRanks + (tid & (kRanks - 1));
    if (i >= n) return;
    if (tid < kRanks) {
      w.model[i] = -1;
      w.round_of[i] = -1;
    } else {
      w.order_of[i] = 0;
      w.util[i] = 0.f;
      if (i >= nv) w.alive_s[i] = 0;
    }
  };
  if (unit >= units) {
    rest();
    return;
  }
  const int s0 = __builtin_amdgcn_readfirstlane(desc.x), size = __builtin_amdgcn_readfirstlane(desc.z) - s0;
  const uint32_t r0 = (uint32_t)(__builtin_amdgcn_readfirstlane(desc.y) - s0), r1 = min(r0 + (uint32_t)kRanks, (uint32_t)size);
  keys += s0;
  if (SPLIT) labels += s0;
  // Keys are read in pieces of 256, four neighbours a lane; positions past the end give the last request again.
  typedef uint32_t quad __attribute__((ext_vector_type(4), aligned(4)));
  struct Keys { uint32_t key[kRankItems], label[SPLIT ? kRankItems : 1]; };
  const auto load = [&](Keys& v, int q, int i) {
    if (i + 4 <= size) {
      const quad k4 = *reinterpret_cast<const quad*>(keys + i);
#pragma unroll
      for (int j = 0; j < 4; ++j) v.key[4 * q + j] = k4[j];
      if constexpr (SPLIT) {
        const quad l4 = *reinterpret_cast<const quad*>(labels + i);
#pragma unroll
        for (int j = 0; j < 4; ++j) v.label[4 * q + j] = l4[j];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int e = min(i + j, size - 1);
        v.key[4 * q + j] = keys[e];
        if constexpr (SPLIT) v.label[4 * q + j] = (uint32_t)labels[e];
      }
    }
  };
  const auto label_of = [](const Keys& v, int j) { return SPLIT ? v.label[SPLIT ? j : 0] : 0u; };
  constexpr int kPiece = 4 * kWave, kQuads = kRankItems / 4;
  static_assert(kQuads == 2, "a wavefront's pieces");
  // pieces of a wavefront's share of kRankHeld requests, or of all where there are fewer: neighbouring ones
  const bool all_held = size <= kRankHeld;
  const int mine = size <= kPiece * kRankWaves ? 1 : kQuads;
  const auto piece_at = [&](int base, int q) { return base + kPiece * (mine * wave + q) + 4 * lane; };
  // the sample's: all where all are held, else 512 pieces of 16 evenly spaced over the application
  constexpr int kSpots = kRankHeld / 16;
  const auto sampled_at = [&](int q) {
    const uint32_t spot = (uint32_t)((kQuads * wave + q) * (kWave / 4) + (lane >> 2));
    return all_held ? piece_at(0, q) : (int)((uint32_t)(size - 16) * spot / (uint32_t)(kSpots - 1)) + 4 * (lane & 3);
  };
  static_assert((int64_t)kRankMax * kSpots < (int64_t)1 << 32, "a spot's place in 32 bits");
  Keys v;
#pragma unroll
  for (int q = 0; q < kQuads; ++q)
    if (q < mine) load(v, q, sampled_at(q));                    // (uniform)
  // f(label, key, position, inside) for the sample; every lane calls it
  const auto each_sampled = [&](auto f) {
#pragma unroll
    for (int q = 0; q < kQuads; ++q)
      if (q < mine) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int pos = sampled_at(q) + j;
          f(label_of(v, 4 * q + j), v.key[4 * q + j], pos, pos < size);
        }
      }
  };
  rest();
  uint32_t key_low, key_high, label_high = 0u;                  // the sample's
  {
    uint32_t lo = 0u, hi = 0u, top = 0u;                        // lo: of the inverted keys
    each_sampled([&](uint32_t lb, uint32_t k, int, bool) {
      lo = max(lo, ~k);
      hi = max(hi, k);
      top = max(top, lb);
    });
    lo = wave_max_u32(lo);
    hi = wave_max_u32(hi);
    if (SPLIT) top = wave_max_u32(top);
    if (lane == 0) {
      wave_low[wave] = lo;
      wave_high[wave] = hi;
      if (SPLIT) wave_label[wave] = top;
    }
    __syncthreads();                                            // (also covers the cleared bins)
    key_low = ~wave_max_u32(lane < kRankWaves ? wave_low[lane] : 0u);
    key_high = wave_max_u32(lane < kRankWaves ? wave_high[lane] : 0u);
    if (SPLIT) label_high = wave_max_u32(lane < kRankWaves ? wave_label[lane] : 0u);
  }
  RankBins<SPLIT> bin_of;
  bin_of.over(key_low, key_high, label_high);
  uint32_t b0 = 0u, b1 = kRankBins - 1u;                        // the range in bins, and
  uint32_t d0 = 0u, d1 = ~0u;                                   // (divided) in those of the second counting
  bool divided = false;
  const bool divisible = !SPLIT || label_high + 1u < (uint32_t)kRankBins;     // (a bin has requests of one label, or of none of the sample's)
  uint32_t cnt[4], beg[4];
  RankDivision div{bins, bin_low, bin_high, 1.0f / (float)size, 0};
  const auto prepare_division = [&] {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      bin_low[4 * tid + j] = ~0u;
      bin_high[4 * tid + j] = 0u;
    }
  };
  const auto to_division = [&](uint32_t b, uint32_t key) {
    if (key < bin_low[b]) atomicMin(&bin_low[b], key);          // (most find that another has been there)
    if (key > bin_high[b]) atomicMax(&bin_high[b], key);
  };
  if (size > kRankAll) {
    each_sampled([&](uint32_t lb, uint32_t k, int, bool in) { if (in) atomicAdd(&bins[bin_of(lb, k)], 1u); });
    __syncthreads();
    rank_scan(bins, wave_sum, cnt, beg);
    // An estimated place is off by half the application's size over the square root of the sample: four times that on either side, and
    // one piece (places among equal keys go by position).
    const int m = all_held ? size : kRankHeld;
    const float ratio = (float)m / (float)size, t0 = (float)r0 * ratio, t1 = (float)r1 * ratio;
    const auto margin = [&](float u) { return 4.25f * sqrtf(fmaxf(u * (1.0f - u / (float)m), 0.f)) + 18.0f; };
    const int u0 = all_held ? (int)r0 : max((int)(t0 - margin(t0)), 0), u1 = all_held ? (int)r1 : min((int)(t1 + margin(t1)) + 1, m);
    const auto find = [&](int e, uint32_t u) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (beg[j] <= u && u < beg[j] + cnt[j]) {
          bin_s[e] = 4 * tid + j;
          beg_s[e] = beg[j];
          cnt_s[e] = cnt[j];
        }
    };
    // (beyond the sample's ends everything belongs to the range)
    const auto range = [&](uint32_t& first, uint32_t& last) {
      find(0, (uint32_t)u0);
      find(1, (uint32_t)u1 - 1u);
      __syncthreads();
      if (u0 > 0) first = (uint32_t)__builtin_amdgcn_readfirstlane((int)bin_s[0]);
      if (u1 < m) last = (uint32_t)__builtin_amdgcn_readfirstlane((int)bin_s[1]);
    };
    range(b0, b1);
    const uint32_t in_range = __builtin_amdgcn_readfirstlane((int)(beg_s[1] + cnt_s[1] - beg_s[0]));
    divided = divisible && in_range > 2u * (uint32_t)(u1 - u0) + 256u;     // (uniform)
    if (divided) {
      uint32_t* const second = reinterpret_cast<uint32_t*>(held);
      static_assert(sizeof(held) >= sizeof(bins), "room for a second counting");
      div.half = m > kRankBins ? 1 : 0;
      prepare_division();
      clear_bins(second);
      if (tid == 0) bins[kRankBins] = (uint32_t)m;
      __syncthreads();
      each_sampled([&](uint32_t lb, uint32_t k, int, bool in) { if (in) to_division(bin_of(lb, k), k); });
      __syncthreads();
      each_sampled([&](uint32_t lb, uint32_t k, int pos, bool in) { if (in) atomicAdd(&second[div(bin_of(lb, k), k, pos)], 1u); });
      __syncthreads();
      rank_scan(second, wave_sum, cnt, beg);
      range(d0, d1);
    } else {
      clear_bins(bins);                                         // (whoever counts in them next has passed a barrier)
    }
  }

  // ---- all keys: those before the range are counted, those inside it collected (of longer applications the positions alone) ----
  {
    // the first number for which a condition that stays true once it is holds, sixty-four ways at a time; there has to be one
    const auto first_true = [&](int top_shift, auto holds) {
      uint32_t base = 0u;
      for (int shift = top_shift;; shift = max(shift - 6, 0)) {
        const uint32_t k = base + ((uint32_t)lane << shift);
        const int n_false = __popcll(__ballot(k >= base && !holds(k)));        // (a prefix of the lanes; of the last ones k may start over)
        if (shift == 0) return base + (uint32_t)n_false;
        if (n_false > 0) base += (uint32_t)(n_false - 1) << shift;
      }
    };
    const auto first_key = [&](uint32_t b) { return first_true(26, [&](uint32_t k) { return bin_of(0u, k) >= b; }); };
    // Where the keys of one label are all there are, the range's ends as keys, or (divided) as requests: cheaper to compare with.
    uint32_t k0 = 0u, k_width = ~0u;
    Ranked low = 0ull, high = ~0ull;                            // (the first one behind it)
    if (!SPLIT && divided) {
      // the first request of bin b with at least d in the second counting; behind all keys, or all of bin b's one key, where there is none
      const auto end_of = [&](uint32_t b, uint32_t d) {
        if (bin_low[b] != bin_high[b]) {
          const auto holds = [&](uint32_t k) {
            const uint32_t at = bin_of(0u, k);
            return at > b || (at == b && div(b, k, 0) >= d);
          };
          return holds(~0u) ? ranked(0u, first_true(26, holds), 0) : ~0ull;
        }
        return ranked(0u, bin_low[b], (int)first_true(12, [&](uint32_t p) { return p >= (uint32_t)size || div(b, bin_low[b], (int)p) >= d; }));
      };
      if (d0 > 0u) low = end_of(b0, d0);
      if (d1 != ~0u) high = end_of(b1, d1 + 1u);
    } else if (!SPLIT && !all_held) {
      k0 = b0 > 0u ? first_key(b0) : 0u;
      // (of bins of few keys the last one's may be the greatest there is)
      k_width = (b1 < kRankBins - 1u && bin_of(0u, ~0u) > b1 ? first_key(b1 + 1u) - 1u : ~0u) - k0;
    }
    uint32_t before = 0u;
    const auto test = [&](const Keys& k, int base, uint32_t& in, auto where) {       // (-1: before the range, 0: inside)
      const bool full = base + kRankHeld <= size;               // (uniform)
#pragma unroll
      for (int q = 0; q < kQuads; ++q)
        if (q < mine) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int pos = piece_at(base, q) + j;
            const int d = where(label_of(k, 4 * q + j), k.key[4 * q + j], pos);
            const bool there = full || pos < size;
            before += there && d < 0 ? 1u : 0u;
            in |= there && d == 0 ? 1u << (4 * q + j) : 0u;
          }
        }
    };
    const auto test_any = [&](const Keys& k, int base, uint32_t& in) {
      if (!SPLIT && divided)
        test(k, base, in, [&](uint32_t, uint32_t key, int pos) {
          const Ranked x = ranked(0u, key, pos);
          return x < low ? -1 : x < high ? 0 : 1;
        });
      else if (divided)
        test(k, base, in, [&](uint32_t lb, uint32_t key, int pos) {
          const uint32_t b = bin_of(lb, key);
          if (b != b0 && b != b1) return b < b0 ? -1 : b < b1 ? 0 : 1;
          const uint32_t d = div(b, key, pos);
          return d < d0 ? -1 : d <= d1 ? 0 : 1;
        });
      else if (SPLIT || all_held)
        test(k, base, in, [&](uint32_t lb, uint32_t key, int) {
          const uint32_t b = bin_of(lb, key);
          return b < b0 ? -1 : b <= b1 ? 0 : 1;
        });
      else
        test(k, base, in, [&](uint32_t, uint32_t key, int) { return key < k0 ? -1 : key - k0 <= k_width ? 0 : 1; });
    };
    const auto room_for = [&](uint32_t in) {                    // this lane's first place in `held`
      const uint32_t c = (uint32_t)__popc(in), incl = wave_scan_incl(c);
      uint32_t at = 0u;
      if (lane == kWave - 1) at = atomicAdd(&n_held, incl);
      return (uint32_t)__builtin_amdgcn_readlane((int)at, kWave - 1) + incl - c;
    };
    if (all_held) {
      uint32_t in = 0u;
      test_any(v, 0, in);
      uint32_t at = room_for(in);
#pragma unroll
      for (int e = 0; e < kRankItems; ++e)
        if (in >> e & 1u) {
          if (at < (uint32_t)kRankCap) held[at] = ranked(label_of(v, e), v.key[e], piece_at(0, e >> 2) + (e & 3));
          ++at;
        }
    } else {
      // (places in LDS are asked for four turns at a time, a bit for each key: every wavefront waits for its answer)
      uint32_t in = 0u;
      int turns = 0;
      const auto take = [&](const Keys& k, int base) {
        uint32_t bits = 0u;
        test_any(k, base, bits);
        in |= bits << (kRankItems * turns);
        ++turns;
      };
      const auto put = [&](int first) {                          // first: of the turns' keys
        uint32_t at = room_for(in);
        while (in != 0u) {
          const int e = __ffs((int)in) - 1, turn = e / kRankItems;
          in &= in - 1u;
          if (at < (uint32_t)kRankCap) held[at] = (Ranked)(uint32_t)(piece_at(first + turn * kRankHeld, (e % kRankItems) >> 2) + (e & 3));
          ++at;
        }
        turns = 0;
      };
      static_assert(4 * kRankItems == 32, "four turns' keys in a word");
      Keys u;
      const auto fetch = [&](Keys& k, int base) {
#pragma unroll
        for (int q = 0; q < kQuads; ++q)
          if (base + kPiece * (kQuads * wave + q) < size) load(k, q, piece_at(base, q));       // (uniform)
      };
      fetch(v, 0);
      for (int base = 0; base < size; base += 2 * kRankHeld) {  // one turn ahead
        fetch(u, base + kRankHeld);
        take(v, base);
        fetch(v, base + 2 * kRankHeld);
        if (base + kRankHeld < size) take(u, base + kRankHeld);
        if (turns >= 3 || base + 2 * kRankHeld >= size) put(base + (turns > 2 ? -2 * kRankHeld : 0));
      }
    }
    before = wave_scan_incl(before);
    if (lane == kWave - 1 && before != 0u) atomicAdd(&n_before, before);
  }
  __syncthreads();
  uint32_t from = __builtin_amdgcn_readfirstlane((int)n_before);
  int count = __builtin_amdgcn_readfirstlane((int)n_held);
  const auto place = [&](uint32_t rank, Ranked e) {
    if (rank < r0 || rank >= r1) return;
    const int at = s0 + (int)rank;
    if constexpr (SPLIT) label_out[at] = ranked_label(e);
    finish_position(w, at, ranked_key(e), s0 + ranked_pos(e), SPLIT ? 1 : 0);
  };
  if (count <= kRankCap && from <= r0 && r1 <= from + (uint32_t)count) {
    // ---- in finer bins over the range: counted, then put bin by bin, a bin's start counting up to its end ----
    if (divided) {
      clear_bins(bins);
      __syncthreads();
    }
    bin_of.first = (float)b0;
    bin_of.finer = floorf((float)kRankBins / (float)(b1 - b0 + 1u));
    Ranked own[kRankOwn];
#pragma unroll
    for (int h = 0; h < kRankOwn; ++h)
      if (h * kRankThreads < count) own[h] = held[min(tid + h * kRankThreads, count - 1)];           // (uniform)
    if (!all_held) {
#pragma unroll
      for (int h = 0; h < kRankOwn; ++h)
        if (h * kRankThreads < count) {
          const int pos = (int)(uint32_t)own[h];
          own[h] = ranked(SPLIT ? (uint32_t)labels[pos] : 0u, keys[pos], pos);
        }
    }
#pragma unroll
    for (int h = 0; h < kRankOwn; ++h)
      if (tid + h * kRankThreads < count) atomicAdd(&bins[bin_of.fine(own[h])], 1u);
    __syncthreads();
    rank_scan(bins, wave_sum, cnt, beg);
    const auto any_crowded = [&](int level) {
      if (max(max(cnt[0], cnt[1]), max(cnt[2], cnt[3])) > (uint32_t)(level == 0 ? kRankMates : kRankMatesLast)) crowded[level] = 1u;
      __syncthreads();
      return crowded[level] != 0u;
    };
    if (!any_crowded(0)) {
#pragma unroll
      for (int h = 0; h < kRankOwn; ++h)
        if (tid + h * kRankThreads < count) held[atomicAdd(&bins[bin_of.fine(own[h])], 1u)] = own[h];
      __syncthreads();
      for (int i = tid; i < count; i += kRankThreads) {
        const Ranked e = held[i];
        const uint32_t b = bin_of.fine(e);
        const int first = b == 0u ? 0 : (int)bins[b - 1], last = (int)bins[b];
        uint32_t rank = from + (uint32_t)first;
        for (int m = first; m < last; ++m) rank += held[m] < e ? 1u : 0u;
        place(rank, e);
      }
      return;
    }
    if (divisible) {
      prepare_division();
      if (tid == 0) bins[kRankBins] = (uint32_t)count;
      __syncthreads();
#pragma unroll
      for (int h = 0; h < kRankOwn; ++h)
        if (tid + h * kRankThreads < count) to_division(bin_of.fine(own[h]), ranked_key(own[h]));
      __syncthreads();
      div.half = count > kRankBins ? 1 : 0;
      uint32_t sub[kRankOwn] = {};
#pragma unroll
      for (int h = 0; h < kRankOwn; ++h)
        if (tid + h * kRankThreads < count) {
          const uint32_t b = bin_of.fine(own[h]);
          // (a bin of labels beyond the sample's may have several of them, and is not divided by keys)
          sub[h] = bin_of.beyond(ranked_label(own[h])) ? bins[b] >> div.half : div(b, ranked_key(own[h]), ranked_pos(own[h]));
        }
      __syncthreads();
      clear_bins(bins);
      __syncthreads();
#pragma unroll
      for (int h = 0; h < kRankOwn; ++h)
        if (tid + h * kRankThreads < count) atomicAdd(&bins[sub[h]], 1u);
      __syncthreads();
      rank_scan(bins, wave_sum, cnt, beg);
      if (!any_crowded(1)) {
#pragma unroll
        for (int h = 0; h < kRankOwn; ++h)
          if (tid + h * kRankThreads < count) held[atomicAdd(&bins[sub[h]], 1u)] = own[h];
        __syncthreads();
#pragma unroll
        for (int h = 0; h < kRankOwn; ++h)
          if (tid + h * kRankThreads < count) {
            const int first = sub[h] == 0u ? 0 : (int)bins[sub[h] - 1], last = (int)bins[sub[h]];
            uint32_t rank = from + (uint32_t)first;
            for (int m = first; m < last; ++m) rank += held[m] < own[h] ? 1u : 0u;
            place(rank, own[h]);
          }
        return;
      }
    }
    if (!all_held) {                                            // (positions alone so far)
#pragma unroll
      for (int h = 0; h < kRankOwn; ++h)
        if (tid + h * kRankThreads < count) held[tid + h * kRankThreads] = own[h];
    }
  } else {
    // ---- the keys of the first and the last place exactly, and how many keys lie before those ----
    constexpr int kDigit = 11, kHalf = 1 << kDigit;
    static_assert(2 * kHalf == kRankBins, "digits of either place");
    constexpr int kTop = ((SPLIT ? 48 : 32) + kDigit - 1) / kDigit * kDigit - kDigit;
    Ranked at0 = 0ull, at1 = 0ull;                              // digits of (label and) key found so far
    uint32_t less0 = 0u, less1 = 0u;                            // keys before those
    const auto whole = [&](int i) { return (SPLIT ? (Ranked)(uint32_t)labels[i] << 32 : 0ull) | (Ranked)keys[i]; };
    for (int shift = kTop; shift >= 0; shift -= kDigit) {
      __syncthreads();
      clear_bins(bins);
      __syncthreads();
      for (int base = 0; base < size; base += 4 * kRankThreads) {
        Ranked k[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) k[q] = whole(min(base + q * kRankThreads + tid, size - 1)) >> shift;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const bool in = base + q * kRankThreads + tid < size;
          if (in && k[q] >> kDigit == at0) atomicAdd(&bins[(uint32_t)k[q] & (kHalf - 1)], 1u);
          if (in && k[q] >> kDigit == at1) atomicAdd(&bins[kHalf + ((uint32_t)k[q] & (kHalf - 1))], 1u);
        }
      }
      __syncthreads();
      rank_scan(bins, wave_sum, cnt, beg);
      const uint32_t half = tid < kRankThreads / 2 ? 0u : bins[kHalf];         // (the second half counts on from the first)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t b = beg[j] - half;
        if (tid < kRankThreads / 2) {
          if (less0 + b <= r0 && r0 < less0 + b + cnt[j]) { bin_s[0] = 4 * tid + j; beg_s[0] = b; }
        } else {                                                // (the last place is r1 - 1)
          if (less1 + b < r1 && r1 <= less1 + b + cnt[j]) { bin_s[1] = 4 * tid + j - kHalf; beg_s[1] = b; }
        }
      }
      __syncthreads();
      at0 = at0 << kDigit | bin_s[0];
      at1 = at1 << kDigit | bin_s[1];
      less0 += beg_s[0];
      less1 += beg_s[1];
    }
    // in the order of positions: of the first key what lies behind r0 - less0 others of it, of the last what lies before r1 - less1
    const uint32_t skip = r0 - less0, take = r1 - less1;
    uint32_t same0 = 0u, same1 = 0u;
    __syncthreads();
    if (tid == 0) n_held = 0u;
    for (int base = 0; base < size; base += kRankThreads) {
      const int i = base + tid;
      const Ranked k = whole(min(i, size - 1));
      const bool is0 = i < size && k == at0, is1 = i < size && k == at1;
      const unsigned long long m0 = __ballot(is0), m1 = __ballot(is1), lower = (1ull << lane) - 1ull;
      __syncthreads();
      if (lane == 0) wave_sum[wave] = (uint32_t)__popcll(m0) | (uint32_t)__popcll(m1) << 16;
      __syncthreads();
      const uint32_t ws = lane < kRankWaves ? wave_sum[lane] : 0u, wi = wave_scan_incl<true>(ws);       // (up to 1,024 of either)
      const uint32_t before = __builtin_amdgcn_readlane((int)(wi - ws), wave), all = __builtin_amdgcn_readlane((int)wi, kRankWaves - 1);
      const bool in = i < size && k >= at0 && k <= at1 && (!is0 || same0 + (before & 0xffffu) + (uint32_t)__popcll(m0 & lower) >= skip) &&
                      (!is1 || same1 + (before >> 16) + (uint32_t)__popcll(m1 & lower) < take);
      if (in) held[atomicAdd(&n_held, 1u)] = ranked((uint32_t)(k >> 32), (uint32_t)k, i);
      same0 += all & 0xffffu;
      same1 += all >> 16;
    }
    from = r0;
    count = (int)(r1 - r0);
  }
  rank_network(held, count);
  for (int i = tid; i < count; i += kRankThreads) place(from + (uint32_t)i, held[i]);
}

}  // namespace sp
