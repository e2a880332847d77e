// Grouping and ordering of a window's requests (Alg. 1 "HashMap<app : request list>" and "requests in g sorted by
// priority"; eq. (12); Sec. 5.3.2 with subgroups).
//
// Grouping by application.  Short windows of up to seven applications: one kernel, in which every workgroup counts the whole
// window.  Else windows of up to 262,144 requests of up to 31 applications: one kernel too, whose tiles hand each other their counts, and
// count for themselves what does not come (GroupWords).  Else up to 255 applications: one kernel counts the applications of every tile of
// the queue (k_group_count), a second one places the requests (k_group_place): a tile reads the counts of all tiles, which are few
// (tiles times applications words), so no tile waits for another.  More applications: two or three stable radix passes
// over the ids (k_digit_totals, k_radix_pass), whose tiles learn the digit counts of the tiles before them by looking back
// through published words.
//
// Ordering inside each application by the inverted bits of the priority key (or the deadline bits, or (subgroup, key)).
// Windows of some length by priority keys: one launch (sp_order.h).  Else up to kMergeMax requests: runs of kRun consecutive requests are sorted by one workgroup each in LDS (k_sort_runs); runs are
// then merged several at a time (k_merge_runs): a workgroup takes consecutive elements of one run and finds the place of each
// by counting, with binary searches in LDS, what precedes it in the sibling runs.  No workgroup waits for another, the number
// of launches follows from the window's size alone (one for up to 1,024 requests, two for up to 16,384, three beyond), and
// the last one writes the service order's arrays itself.  Longer windows: four radix passes inside the applications'
// ranges and a gather, which read and write every element five times but do no searching.  Ordering took, merges against
// passes: 20 us against 45 for 65,536 requests of 8 applications, 35 against 66 for 200,003 of 12; 58 against 70 for 300,000
// of 12 but 97 against 79 for 300,000 of one, 133 against 82 for 600,000 of 8.
#pragma once
#include <type_traits>
#include "sp_common.h"
#include "sp_wave.h"

namespace sp {

constexpr int kSortThreads = 512;
constexpr int kSortWaves = kSortThreads / kWave;
constexpr int kSortItems = 8;                         // elements per thread
constexpr int kSortTile = kSortThreads * kSortItems;  // elements per tile
constexpr int kSortSpinLimit = 1 << 20;               // polls before a look-back is given up
constexpr int kMaxSortPasses = 6;                     // four key passes and up to two over subgroup labels
constexpr uint32_t kSortCountMask = 0x3FFFFFFFu;      // a published word: generation << 32 | status << 30 | count
constexpr int kLookBack = 8;                          // tiles whose published words are requested together

struct SortPlan {
  const int32_t* seg;          // [nseg+1] segment starts
  const int32_t* unit_start;   // [nseg+1] prefix of runs per segment
  int32_t nseg;
  const int4* desc;            // per run or tile: (start of the segment, first element, end of the segment, 0); null = one segment
};

// mask of lanes whose 8-bit digit equals mine
__device__ __forceinline__ unsigned long long match_digit(uint32_t digit, bool valid) {
  unsigned long long m = __ballot(valid);
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const bool bit = (digit >> b) & 1u;
    const unsigned long long vote = __ballot(bit);
    m &= bit ? vote : ~vote;
  }
  return m;
}

// This workgroup's tile of a pass: elements [beg, end) of a segment that starts at s0 with tile `first`.  One segment
// (desc == null), or the applications' ranges.  False for a workgroup without a tile.
__device__ __forceinline__ bool sort_tile(const SortPlan& sp, int tile, int& s0, int& beg, int& end, int& first) {
  if (sp.desc == nullptr) {
    const int n = sp.seg[1];
    s0 = 0; first = 0;
    beg = tile * kSortTile;
    end = min(beg + kSortTile, n);
    return beg < n;
  }
  if (tile >= sp.unit_start[sp.nseg]) return false;
  const int4 d = sp.desc[tile];
  s0 = d.x; beg = d.y;
  end = min(beg + kSortTile, d.z);
  first = tile - (beg - s0) / kSortTile;
  return true;
}

// The key of element i: as stored, or (clamp_a > 0) an application id clamped into [0, A] with A = "invalid".
__device__ __forceinline__ uint32_t sort_key_at(const uint32_t* __restrict__ keys, int i, int clamp_a, bool& bad) {
  const uint32_t k = keys[i];
  if (clamp_a <= 0) return k;
  const int a = (int)k;
  const bool ok = a >= 0 && a < clamp_a;
  bad |= !ok;
  return ok ? k : (uint32_t)clamp_a;
}

constexpr int kSegTable = 1024;                        // applications whose tile prefixes k_segments keeps in LDS

// Start of every digit of a segment, given its 256 digit totals: lane l returns the starts of digits
// 4l .. 4l+3.
__device__ __forceinline__ uint4 wave_digit_bases(const uint32_t* __restrict__ tot_s, uint32_t seg_start, int lane) {
  const uint4 t = *reinterpret_cast<const uint4*>(tot_s + 4 * lane);
  const uint32_t mine = t.x + t.y + t.z + t.w;
  const uint32_t incl = wave_scan_incl(mine);
  uint4 b;
  b.x = seg_start + incl - mine;
  b.y = b.x + t.x;
  b.z = b.y + t.y;
  b.w = b.z + t.z;
  return b;
}

// Where the applications' ranges start, the prefixes of scoring tiles and sort runs, and a descriptor for each of either, so that
// a workgroup finds its place with a single load.  Scoring tiles are numbered application by application, in the order of
// by_cost where they are dealt in turn (see tile_of), sort runs in ascending order.
struct SegArgs {
  int32_t n, A;
  const uint32_t* sorted_app;   // application-sorted keys (not used where the counts of the ids are given)
  int32_t tile, unit;           // requests per scoring tile and per sort run
  const int32_t* by_cost;       // [A] applications, costly tiles first
  const int32_t* cost;          // [A] what a scoring tile of each costs; null where that is the same (tiles in contiguous eighths)
  int32_t grid;                 // workgroups that the tiles are dealt to
  int32_t* seg;
  int32_t* unit_start;
  int4* tile_desc;
  int4* sort_desc;
};

// Until (and unless) the requests are split into subgroups, group g is application g.
__device__ __forceinline__ void plain_group(const Window& w, int a, int beg, int end) {
  w.head[a] = beg;
  w.head[w.gcap + a] = beg;
  w.grp_app[a] = a;
  w.grp_end[a] = end;
}

// Last k < n with start[k] <= i (empty ranges share a start; start[0] = 0).
__device__ __forceinline__ int range_of(const int* start, int n, int i) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (start[mid] <= i) lo = mid; else hi = mid;
  }
  return lo;
}

// What the dies' contiguous eighths of a window's tiles cost: an application's tiles [first, first + count) added to them.
__device__ __forceinline__ void add_to_dies(unsigned long long* dies, int first, int count, int cost, int n_tiles) {
  const int per = (n_tiles + kXcds - 1) / kXcds, end = first + count;
  if (count <= 0) return;                              // (else there are tiles)
  for (int d = first / per; d * per < end; ++d) atomicAdd(&dies[d], (unsigned long long)(min(end, (d + 1) * per) - max(first, d * per)) * (unsigned)cost);
}
// Tiles are dealt in turn where the costliest eighth holds over 1/32 more than its share: as much as contiguous eighths gain
// where they are even (weights in one L2).  us of the scoring kernel, contiguous / in turn, a million requests of 256 floats: 31 applications of
// 1,000 classes and one of 10 1,531 / 1,546 (100,000 requests 189 / 193), 1,000 and 600 classes by turns (64 floats) 630 / 645; 16 of 1,000
// and then 16 of 850 1,540 / 1,460, of 680 1,535 / 1,350 (100,000 requests 188 / 171), of 500 1,484 / 1,248, 32 from 1,000 down to 318
// 1,366 / 1,143; half a million, half of them of the one with 10: 801 / 516.
__device__ __forceinline__ bool dies_uneven(const unsigned long long* dies) {
  unsigned long long most = 0ull, sum = 0ull;
  for (int d = 0; d < kXcds; ++d) {
    most = dies[d] > most ? dies[d] : most;
    sum += dies[d];
  }
  return 32ull * kXcds * most > 33ull * sum;
}

// The descriptors of all tiles and runs from the tables in LDS, by `threads` threads.
__device__ __forceinline__ void write_descriptors(const SegArgs& g, bool in_turn, const int* s_tile, const int* s_unit, const int* s_seg, const int* s_app,
                                                  int tid, int threads) {
  const int n_tiles = s_tile[g.A];
  for (int wg = tid; wg < g.grid; wg += threads) {                  // (application, first request, end of its range, 0)
    const int t = tile_of(in_turn, wg, n_tiles);
    int4 d = make_int4(-1, 0, 0, 0);
    if (t >= 0) {
      const int k = range_of(s_tile, g.A, t), a = s_app[k];
      d = make_int4(a, s_seg[a] + (t - s_tile[k]) * g.tile, s_seg[a + 1], 0);
    }
    g.tile_desc[wg] = d;
  }
  for (int u = tid; u < s_unit[g.A]; u += threads) {                // (start of the application, first element, end, 0)
    const int a = range_of(s_unit, g.A, u);
    g.sort_desc[u] = make_int4(s_seg[a], s_seg[a] + (u - s_unit[a]) * g.unit, s_seg[a + 1], 0);
  }
}

// From the sorted ids (values in [0, A], A = invalid): seg[a] = first position with an id >= a.  One workgroup.
__global__ __launch_bounds__(256) void k_segments(SegArgs g, Window w) {
  // A look-back that ran out has left holes in the sorted ids: the window will be refused, and until then it has no
  // requests, so that nothing reads what was never written.
  const int n = (w.st->err & kErrSortSync) ? 0 : g.n;
  const int A = g.A, tile = g.tile, unit = g.unit, tid = threadIdx.x;
  const uint32_t* __restrict__ sorted_app = g.sorted_app;
  int32_t* seg = g.seg;
  for (int a = tid; a <= A + 1; a += 256) {
    int lo = 0, hi = n;                     // lower_bound(sorted_app, a)
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (sorted_app[mid] < (uint32_t)a) lo = mid + 1; else hi = mid;
    }
    seg[a] = lo;                            // seg[A] = number of valid requests, seg[A+1] = n
  }
  __syncthreads();
  for (int a = tid; a < A; a += 256) plain_group(w, a, seg[a], seg[a + 1]);
  if (tid == 0) {
    w.grp_n[0] = A;
    w.grp_n[1] = 1;
  }
  // prefixes of tiles and units over the applications: every thread takes a run of consecutive
  // applications, the runs' totals are scanned across the workgroup
  __shared__ int run_t[256], run_u[256];
  __shared__ unsigned long long dies[kXcds];
  __shared__ int s_tile[kSegTable + 1], s_seg[kSegTable + 1], s_unit[kSegTable + 1], s_app[kSegTable];   // used when A <= kSegTable
  const int per = (A + 255) / 256;
  const int a_lo = min(A, tid * per), a_hi = min(A, a_lo + per);
  const auto tiles_of = [&](int c) { return (seg[c + 1] - seg[c] + tile - 1) / tile; };
  const auto scan_runs = [&] {
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
      const int t_up = tid >= o ? run_t[tid - o] : 0;
      const int u_up = tid >= o ? run_u[tid - o] : 0;
      __syncthreads();
      run_t[tid] += t_up;
      run_u[tid] += u_up;
      __syncthreads();
    }
  };
  int ts = 0, us = 0;
  bool in_turn = false;
  if (g.cost != nullptr) {                             // (uniform)
    if (tid < kXcds) dies[tid] = 0ull;
    for (int k = a_lo; k < a_hi; ++k) ts += tiles_of(k);
    run_t[tid] = ts;
    run_u[tid] = 0;
    scan_runs();
    int first = run_t[tid] - ts;
    for (int k = a_lo; k < a_hi; ++k) {
      const int nt = tiles_of(k);
      add_to_dies(dies, first, nt, g.cost[k], run_t[255]);
      first += nt;
    }
    __syncthreads();
    in_turn = dies_uneven(dies);
    ts = 0;
  }
  const auto app_at = [&](int k) { return in_turn ? g.by_cost[k] : k; };
  for (int k = a_lo; k < a_hi; ++k) {
    ts += tiles_of(app_at(k));
    us += (seg[k + 1] - seg[k] + unit - 1) / unit;
  }
  run_t[tid] = ts;                                     // (read by others before the last barrier only)
  run_u[tid] = us;
  scan_runs();
  const int ts0 = run_t[tid] - ts, us0 = run_u[tid] - us;   // exclusive prefixes of this thread's run
  const bool table = A <= kSegTable;
  ts = ts0;
  us = us0;
  for (int k = a_lo; k < a_hi; ++k) {
    const int c = app_at(k);
    g.unit_start[k] = us;
    if (table) {
      s_tile[k] = ts;
      s_app[k] = c;
      s_unit[k] = us;
      s_seg[k] = seg[k];
    }
    ts += tiles_of(c);
    us += (seg[k + 1] - seg[k] + unit - 1) / unit;
  }
  if (tid == 255) {
    g.unit_start[A] = run_u[255];
    if (table) {
      s_tile[A] = run_t[255];
      s_unit[A] = run_u[255];
      s_seg[A] = seg[A];
    }
  }
  __syncthreads();
  if (table) {
    write_descriptors(g, in_turn, s_tile, s_unit, s_seg, s_app, tid, 256);
  } else {
    ts = ts0;
    us = us0;
    for (int k = a_lo; k < a_hi; ++k) {
      const int c = app_at(k), cb = seg[c], ce = seg[c + 1], nt = tiles_of(c);
      const int sb = seg[k], se = seg[k + 1], nu = (se - sb + unit - 1) / unit;
      for (int t = 0; t < nt; ++t) g.tile_desc[workgroup_of(in_turn, ts + t, run_t[255])] = make_int4(c, cb + t * tile, ce, 0);
      for (int u = 0; u < nu; ++u) g.sort_desc[us + u] = make_int4(sb, sb + u * unit, se, 0);
      ts += nt;
      us += nu;
    }
    for (int wg = tid; wg < g.grid; wg += 256)
      if (tile_of(in_turn, wg, run_t[255]) < 0) g.tile_desc[wg] = make_int4(-1, 0, 0, 0);
  }
}

__device__ __forceinline__ void clear_words(uint32_t* __restrict__ p, int64_t words) {
  if (p == nullptr) return;
  for (int64_t i = (int64_t)blockIdx.x * kSortThreads + threadIdx.x; i < words; i += (int64_t)gridDim.x * kSortThreads) p[i] = 0u;
}

// Digit totals of every segment for n_pass consecutive passes (digits at shift0, shift0 + 8, ...):
// dtot[(p * tiles_cap + first tile of the segment) * 256 + digit], which must be zero beforehand.  Also
// clears zero_words words of the next sort's totals.
__global__ __launch_bounds__(kSortThreads) void k_digit_totals(SortPlan sp, const uint32_t* __restrict__ keys,
                                                               int clamp_a, int shift0, int n_pass, int64_t tiles_cap,
                                                               uint32_t* __restrict__ dtot, uint32_t* __restrict__ zero_ptr,
                                                               int64_t zero_words, State* st) {
  __shared__ uint32_t h[4][256];
  const int tid = threadIdx.x;
  clear_words(zero_ptr, zero_words);
  int s0, beg, end, first;
  if (!sort_tile(sp, blockIdx.x, s0, beg, end, first)) return;
  for (int i = tid; i < 4 * 256; i += kSortThreads) h[0][i] = 0u;
  __syncthreads();
  bool bad = false;
#pragma unroll
  for (int c = 0; c < kSortItems; ++c) {
    const int i = beg + c * kSortThreads + tid;
    if (i < end) {
      const uint32_t k = sort_key_at(keys, i, clamp_a, bad);
      for (int p = 0; p < n_pass; ++p) atomicAdd(&h[p][(k >> (shift0 + 8 * p)) & 255u], 1u);
    }
  }
  if (bad) atomicOr(&st->err, kErrApp);
  __syncthreads();
  for (int i = tid; i < n_pass * 256; i += kSortThreads) {
    const uint32_t c = h[0][i];
    if (c) atomicAdd(&dtot[((int64_t)(i >> 8) * tiles_cap + first) * 256 + (i & 255)], c);
  }
}

// Exclusive prefix sums of one value per thread over the first 256 threads of the workgroup (all of its
// threads call it; those beyond 255 pass 0 and get the total).
template <int WAVES = kSortWaves>
__device__ __forceinline__ uint32_t scan256_excl(uint32_t v, uint32_t* wave_tot /*[WAVES]*/) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t incl = wave_scan_incl(v);
  __syncthreads();
  if (lane == 63) wave_tot[wave] = incl;
  __syncthreads();
  uint32_t before = 0;
  for (int i = 0; i < WAVES; ++i) before += i < wave ? wave_tot[i] : 0u;
  return before + incl - v;
}

// Two floats that travel with an element through a pass (the grouping pass brings every request's deadline
// and weight to its grouped position, so that the scoring kernel reads them in order instead of gathering
// them by request id, 4 useful bytes per 64-byte line): read from two arrays or from one array of pairs,
// indexed by element, written as pairs.
struct SortCarry {
  const float* in0;            // [n], with in1; or null
  const float* in1;
  const float2* in01;          // [n] pairs (a second pass); or null
  float2* out;                 // [n] pairs at the elements' new positions
};

// One stable pass: (keys_in, vals_in) -> (keys_out, vals_out) by the digit at `shift`.  vals_in == nullptr
// means the identity (value = element index).  dtot_pass: this pass's slab of digit totals.  state:
// [tiles][256] published words; gen: this launch's generation (never reused while the array lives).
template <bool CARRY>
__global__ __launch_bounds__(kSortThreads) void k_radix_pass(
    SortPlan sp, const uint32_t* __restrict__ keys_in, const int32_t* __restrict__ vals_in, int shift, int clamp_a,
    const uint32_t* __restrict__ dtot_pass, unsigned long long* __restrict__ state, uint32_t gen, int spin_limit,
    uint32_t* __restrict__ keys_out, int32_t* __restrict__ vals_out, State* st, SortCarry cy) {
  __shared__ uint32_t cnt[kSortWaves][256];      // digit counts per wavefront, then their exclusive prefix over the wavefronts
  __shared__ uint32_t lstart[256];               // where each digit starts inside the sorted tile
  __shared__ uint32_t dbase[256];                // global position of the digit's first element of this tile, minus lstart
  __shared__ uint32_t wave_tot[kSortWaves];
  __shared__ uint32_t skey[kSortTile];
  __shared__ int32_t sval[kSortTile];
  __shared__ float2 spay[CARRY ? kSortTile : 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // (an earlier pass whose look-back ran out has left holes: what is in them would not match the totals)
  if ((vals_in != nullptr || sp.desc != nullptr) && (st->err & kErrSortSync)) return;
  int s0, beg, end, first;
  if (!sort_tile(sp, blockIdx.x, s0, beg, end, first)) return;
  const int tile = blockIdx.x;
  for (int i = tid; i < kSortWaves * 256; i += kSortThreads) cnt[0][i] = 0u;
  // a wavefront takes kSortItems chunks of 64 consecutive elements: all loads go out before the first is used
  uint32_t key[kSortItems];
  int32_t val[kSortItems];
  bool bad = false;
#pragma unroll
  for (int c = 0; c < kSortItems; ++c) {
    const int i = beg + (wave * kSortItems + c) * 64 + lane;
    key[c] = i < end ? sort_key_at(keys_in, i, clamp_a, bad) : 0u;
    val[c] = i < end ? (vals_in ? vals_in[i] : i) : 0;
  }
  float2 pay[CARRY ? kSortItems : 1];
#pragma unroll
  for (int c = 0; c < (CARRY ? kSortItems : 0); ++c) {
    const int i = beg + (wave * kSortItems + c) * 64 + lane;
    pay[c] = make_float2(0.f, 0.f);
    if (i < end) pay[c] = cy.in01 ? cy.in01[i] : make_float2(cy.in0[i], cy.in1[i]);
  }
  if (bad) atomicOr(&st->err, kErrApp);
  __syncthreads();
  // rank inside the wavefront: lanes with my digit ahead of me in this chunk, plus the wavefront's earlier chunks
  const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint32_t rank[kSortItems];
#pragma unroll
  for (int c = 0; c < kSortItems; ++c) {
    const int i = beg + (wave * kSortItems + c) * 64 + lane;
    const bool valid = i < end;
    const uint32_t dg = (key[c] >> shift) & 255u;
    const unsigned long long same = match_digit(dg, valid);
    const int leader = valid ? (__ffsll((long long)same) - 1) : lane;
    uint32_t before = 0;
    if (valid && lane == leader) before = atomicAdd(&cnt[wave][dg], (uint32_t)__popcll(same));
    before = __shfl(before, leader);
    rank[c] = before + (uint32_t)__popcll(same & lt);
  }
  __syncthreads();
  // digit counts of the tile; cnt becomes the exclusive prefix over the wavefronts
  uint32_t mine = 0;
  if (tid < 256) {
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
      const uint32_t c = cnt[w][tid];
      cnt[w][tid] = mine;
      mine += c;
    }
  }
  // tiles before this one in the segment: publish, look back, publish the running prefix
  uint32_t excl = 0;
  if (tid < 256) {
    unsigned long long* slot = state + (size_t)tile * 256 + tid;
    const unsigned long long tag = (unsigned long long)gen << 32;
    if (tile == first) {
      __hip_atomic_store(slot, tag | (2ull << 30) | mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      __hip_atomic_store(slot, tag | (1ull << 30) | mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      // Look back a window of tiles at a time: all of the window's words are requested together (one trip
      // to memory for up to kLookBack tiles), then taken nearest first until one carries a running prefix.
      bool lost = false, found = false;
      for (int t2 = tile - 1; t2 >= first && !found && !lost; t2 -= kLookBack) {
        unsigned long long v[kLookBack];
#pragma unroll
        for (int q = 0; q < kLookBack; ++q) {
          const int t3 = max(t2 - q, first);
          v[q] = __hip_atomic_load(state + (size_t)t3 * 256 + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int q = 0; q < kLookBack; ++q) {
          if (t2 - q < first || found || lost) continue;
          unsigned long long w = v[q];
          if (spin_limit < 0) lost = true;                             // a test's way into the failure path: give up unseen
          for (int k = 0; !lost && (uint32_t)(w >> 32) != gen; ++k) {  // not published yet: poll this one
            if (k >= spin_limit) { lost = true; break; }
            __builtin_amdgcn_s_sleep(1);
            w = __hip_atomic_load(state + (size_t)(t2 - q) * 256 + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          if (lost) continue;
          excl += (uint32_t)w & kSortCountMask;
          found = ((uint32_t)w >> 30) == 2u;
        }
      }
      if (lost) atomicOr(&st->err, kErrSortSync);     // the counts seen so far keep every write inside the segment
      __hip_atomic_store(slot, tag | (2ull << 30) | ((excl + mine) & kSortCountMask), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  // where the digits start: inside the tile, and in the segment
  const uint32_t tot = tid < 256 ? dtot_pass[(size_t)first * 256 + tid] : 0u;
  const uint32_t ls = scan256_excl(mine, wave_tot);
  const uint32_t gs = scan256_excl(tot, wave_tot);
  if (tid < 256) {
    lstart[tid] = ls;
    dbase[tid] = (uint32_t)s0 + gs + excl - ls;
  }
  __syncthreads();
  // into LDS in sorted order
#pragma unroll
  for (int c = 0; c < kSortItems; ++c) {
    const int i = beg + (wave * kSortItems + c) * 64 + lane;
    if (i < end) {
      const uint32_t dg = (key[c] >> shift) & 255u;
      const uint32_t p = lstart[dg] + cnt[wave][dg] + rank[c];
      skey[p] = key[c];
      sval[p] = val[c];
      if (CARRY) spay[p] = pay[c];
    }
  }
  __syncthreads();
  // and out: neighbouring threads hold neighbouring elements of a digit's run
  const int n_tile = end - beg;
  for (int j = tid; j < n_tile; j += kSortThreads) {
    const uint32_t k = skey[j];
    const uint32_t dst = dbase[(k >> shift) & 255u] + (uint32_t)j;
    keys_out[dst] = k;
    vals_out[dst] = sval[j];
    if (CARRY) cy.out[dst] = spay[j];
  }
}

// ---- grouping by application, up to 255 of them ----

constexpr int kGroupThreads = 512;
constexpr int kGroupWaves = kGroupThreads / kWave;
constexpr int kMaxGroupApps = 255;
// Requests per tile: small tiles spread a short queue over the chip; from kGroupSmall requests on, larger ones keep the
// table of counts that every tile reads short.
constexpr int kGroupSmall = 131072;
constexpr int group_tile(int64_t n) { return n <= kGroupSmall ? 1024 : 2048; }

// mask of lanes whose digit of nbits bits equals mine
__device__ __forceinline__ unsigned long long match_bits(uint32_t digit, bool valid, int nbits) {
  unsigned long long m = __ballot(valid);
  for (int b = 0; b < nbits; ++b) {
    const bool bit = (digit >> b) & 1u;
    const unsigned long long vote = __ballot(bit);
    m &= bit ? vote : ~vote;
  }
  return m;
}

// Requests of every application in every tile: counts[tile][a], a = A for ids outside [0, A).  The first kernel of a
// window: its first workgroup also resets the window's state.
template <int ITEMS>
__global__ __launch_bounds__(kGroupThreads) void k_group_count(int n, int A, int nbits, const int32_t* __restrict__ app,
                                                               uint32_t* __restrict__ counts, State* st,
                                                               uint32_t* __restrict__ zero_ptr, int64_t zero_words) {
  __shared__ uint32_t h[256];
  clear_words(zero_ptr, zero_words);                   // the digit totals of a long window's ordering
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (blockIdx.x == 0 && tid == 0) reset_state(st);
  if (tid < 256) h[tid] = 0u;
  const int beg = blockIdx.x * (kGroupThreads * ITEMS);
  uint32_t key[ITEMS];
  bool bad = false;
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const int i = beg + (wave * ITEMS + c) * 64 + lane;
    key[c] = i < n ? sort_key_at((const uint32_t*)app, i, A, bad) : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const bool valid = beg + (wave * ITEMS + c) * 64 + lane < n;
    const unsigned long long same = match_bits(key[c], valid, nbits);
    if (valid && lane == __ffsll((long long)same) - 1) atomicAdd(&h[key[c]], (uint32_t)__popcll(same));
  }
  __syncthreads();
  if (tid <= A) counts[(size_t)blockIdx.x * 256 + tid] = h[tid];
}

// Long windows: exclusive prefixes of every application's counts over the tiles, in place, and the totals (row n_tiles).  One
// workgroup per application (and one for the invalid ids).  Up to kGroupDirect tiles, each tile adds the counts up itself.
constexpr int kGroupDirect = 128;
__global__ __launch_bounds__(1024) void k_group_scan(uint32_t* __restrict__ counts, int n_tiles) {
  __shared__ uint32_t wave_tot[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, a = blockIdx.x;
  uint32_t carry = 0;
  for (int t0 = 0; t0 < n_tiles; t0 += 1024) {
    const int t = t0 + tid;
    const uint32_t c = t < n_tiles ? counts[(size_t)t * 256 + a] : 0u;
    const uint32_t incl = wave_scan_incl(c);
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    uint32_t before = carry, all = carry;
    for (int v = 0; v < 16; ++v) {
      before += v < wave ? wave_tot[v] : 0u;
      all += wave_tot[v];
    }
    if (t < n_tiles) counts[(size_t)t * 256 + a] = before + incl - c;
    carry = all;
    __syncthreads();
  }
  if (tid == 0) counts[(size_t)n_tiles * 256 + a] = carry;
}

// Sums of the tiles' counts per application, over all tiles and over those before `tile`, into LDS (256 words each, zero
// beyond A).  The whole workgroup takes part: the rows are dealt to as many groups of threads as there are.
__device__ __forceinline__ void group_sums(const uint32_t* __restrict__ counts, int n_tiles, int tile, int A, int nbits,
                                           uint32_t* before, uint32_t* total, uint32_t (*red)[2][64]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (n_tiles > kGroupDirect) {                                  // (uniform) k_group_scan has done it
    if (tid < 256) {
      before[tid] = tid <= A ? counts[(size_t)tile * 256 + tid] : 0u;
      total[tid] = tid <= A ? counts[(size_t)n_tiles * 256 + tid] : 0u;
    }
    __syncthreads();
    return;
  }
  const int nd = 1 << nbits, parts = kGroupThreads >> nbits;     // nd > A, at most 256
  const int dg = tid & (nd - 1);
  uint32_t b = 0, t = 0;
  if (dg <= A) {
#pragma unroll 8
    for (int q = tid >> nbits; q < n_tiles; q += parts) {
      const uint32_t c = counts[(size_t)q * 256 + dg];
      t += c;
      b += q < tile ? c : 0u;
    }
  }
  for (int o = nd; o < 64; o <<= 1) {
    b += __shfl_xor(b, o);
    t += __shfl_xor(t, o);
  }
  red[wave][0][lane] = b;
  red[wave][1][lane] = t;
  __syncthreads();
  if (tid < 256) {
    uint32_t sb = 0, stt = 0;
    if (tid <= A) {
      const int per = nd > 64 ? nd >> 6 : 1;                     // wavefronts that hold the digits once between them
      for (int v = tid >> 6; v < kGroupWaves; v += per) {
        sb += red[v][0][tid & 63];
        stt += red[v][1][tid & 63];
      }
    }
    before[tid] = sb;
    total[tid] = stt;
  }
  __syncthreads();
}

// Short windows of few applications: a workgroup counts the whole window itself, in one trip to memory, which spares the launch
// before it: 3.6 us for 256 requests where two launches take 1.7 + 4.2, 5.1 for 4,096 (2.4 + 5.0), 5.8 for 16,384 (2.8 + 5.1), 7.2 for
// 32,768 (3.9 + 5.5), and the gap between them.  The ids that every workgroup reads are 128 KB at the end of this range; at twice the ids
// per thread it is the slower way: us per scoring call of three applications, one launch / two, 44.2 / 45.6 (32,768 requests), 46.3 / 45.7
// (32,769), 47.1 / 46.2 (40,000), 49.9 / 48.7 (65,535); with one application and with seven the same.  Eight bits per application and
// thread, up to kGroupSelfApps applications and the invalid ids.
constexpr int kGroupSelf = 32768, kGroupSelfApps = 7;

// What group_sums gives, from the ids themselves; n <= 2,048 QUADS.
template <int QUADS>
__device__ __forceinline__ void group_sums_self(const int32_t* __restrict__ app, int n, int tile, int tile_size, int A, uint32_t* before,
                                                uint32_t* total, uint32_t (*red)[2][64]) {
  static_assert(4 * QUADS <= 255, "a thread's counts take eight bits each");
  static_assert(kGroupSelfApps < 8, "and a quad's four");
  static_assert(kGroupSelf <= 0xffff, "the workgroup's sixteen");
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  u32x4 id[QUADS];
  if (n >= 4) {                                        // (uniform)
#pragma unroll
    for (int q = 0; q < QUADS; ++q) id[q] = *(const u32x4*)(app + min(4 * (q * kGroupThreads + tid), n - 4));
  } else {
    for (int q = 0; q < QUADS; ++q)
      for (int e = 0; e < 4; ++e) id[q][e] = (uint32_t)app[min(e, n - 1)];
  }
  uint32_t all[2] = {0u, 0u}, ahead[2] = {0u, 0u};     // a byte per application: even ones, odd ones
#pragma unroll
  for (int q = 0; q < QUADS; ++q) {
    const int i = 4 * (q * kGroupThreads + tid);
    uint32_t mine = 0u;                                // four bits each
    if (i + 3 < n) {
#pragma unroll
      for (int e = 0; e < 4; ++e) mine += 1u << (4u * min(id[q][e], (uint32_t)A));
    } else if (i < n) {                                // the last quad of the window, which was loaded from n - 4 on
      const int at = n >= 4 ? n - 4 : 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) mine += (uint32_t)(at + e >= i && at + e < n) << (4u * min(id[q][e], (uint32_t)A));
    }
    const bool before_tile = i < tile * tile_size;     // (tiles are whole quads)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t m = (mine >> (4 * h)) & 0x0f0f0f0fu;
      all[h] += m;
      ahead[h] += before_tile ? m : 0u;
    }
  }
  // sums over the wavefront in sixteen bits
#pragma unroll
  for (int v = 0; v < 2; ++v) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t sum = wave_scan_incl(((v ? all : ahead)[j >> 1] >> (8 * (j & 1))) & 0x00ff00ffu);
      if (lane == 63) red[wave][v][j] = sum;
    }
  }
  __syncthreads();
  if (tid < 256) {
    uint32_t sb = 0, stt = 0;
    if (tid <= A) {
      const int j = (tid & 1) * 2 + ((tid >> 1) & 1), shift = 16 * (tid >> 2);
#pragma unroll
      for (int v = 0; v < kGroupWaves; ++v) {
        sb += (red[v][0][j] >> shift) & 0xffffu;
        stt += (red[v][1][j] >> shift) & 0xffffu;
      }
    }
    before[tid] = sb;
    total[tid] = stt;
  }
  __syncthreads();
}

// Windows of up to kGroupDirect tiles that are not counted in that way: every workgroup counts its tile, hands the counts to the others and
// waits for theirs, which spares a launch.  A word carries two counts and the number of the launch, which the launch before has left in
// memory (not an argument: a recorded launch may be played again), and is valid exactly when that number is the launch's.  A wait that
// runs out (the grid did not fit on the device beside other work) is no error: what has not come is counted from the ids.  Kernels, 65,536
// requests: 3.4 to 4.6 + 5.1 to 6.2 us -> 7.4 to 8.9.  us per scoring call (16 features, both ways in turn), two launches / one: eight applications
// of 64 requests 16.0 / 15.8, 500 16.9 / 16.4, 2,000 21.7 / 20.2, 8,000 24.4 / 23.1, 33,000 31.2 / 30.0, 65,536 35.6 / 34.2, 131,072 49.0 /
// 48.1, 262,144 75.7 / 74.1; thirty-one of 500 17.0 / 16.7, 4,000 21.8 / 21.0, 65,536 36.0 / 34.1, 262,144 67.6 / 66.0; one of 33,000 37.0 /
// 35.7, 262,144 88.6 / 87.4; seven of 131,072 (128 tiles, where the polls are most) 48.6 / 48.4.  Where no count comes at all, behind some 30
// us of polls: of 65,536 40 to 49, 262,144 127 to 167.
constexpr int kGroupOneApps = 31;                      // (sixteen words a tile; a workgroup reads all tiles' words)
constexpr int kGroupWords = (kGroupOneApps + 2) / 2;
constexpr int kGroupSpins = 64;                        // polls of about half a microsecond
struct GroupWords {
  unsigned long long* words;                           // [kGroupDirect][kGroupWords]
  uint32_t* launch;                                    // workgroups that have their sums; launches so far
  int32_t spins;
  int32_t silent;                                      // tiles whose number has these bits hand out nothing (0 but in a test)
};

// A tile's counts (of up to 2,048 requests) to the other workgroups.
__device__ __forceinline__ void publish_counts(const GroupWords& gw, uint32_t launch, int tile, int A, const uint32_t* count) {
  const int tid = threadIdx.x;
  if (2 * tid > A || (tile & gw.silent) != 0) return;
  const uint32_t two = count[2 * tid] | (2 * tid + 1 <= A ? count[2 * tid + 1] << 16 : 0u);
  __hip_atomic_store(gw.words + tile * kGroupWords + tid, ((unsigned long long)(launch + 1u) << 32) | two, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What group_sums gives, from the words of all tiles.
__device__ __forceinline__ void group_sums_handed(const GroupWords& gw, uint32_t launch, const int32_t* __restrict__ app, int n, int n_tiles, int tile,
                                                  int tile_size, int A, uint32_t* before, uint32_t* total, uint32_t (*red)[2][64]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_words = A / 2 + 1;
  int bits = 0;
  while ((1 << bits) < n_words) ++bits;
  const int nw = 1 << bits, parts = kGroupThreads >> bits, word = tid & (nw - 1);
  constexpr int kMost = kGroupDirect * kGroupWords / kGroupThreads;
  static_assert((kGroupWords & (kGroupWords - 1)) == 0 && kGroupWords <= 16 && kGroupDirect * kGroupWords % kGroupThreads == 0, "shares of a thread");
  __shared__ uint32_t lost[kGroupDirect];              // the words of a tile that have not come, a bit each
  __shared__ int any_lost;
  if (tid < kGroupDirect) lost[tid] = 0u;
  if (tid == 0) any_lost = 0;
  unsigned long long v[kMost];
  uint32_t wanted = 0u;                                // of this thread's words, a bit each
  for (int spin = 0; spin < gw.spins; ++spin) {
    wanted = 0u;
#pragma unroll
    for (int k = 0; k < kMost; ++k) {
      const int q = (tid >> bits) + k * parts;
      if (q < n_tiles && word < n_words) v[k] = __hip_atomic_load(gw.words + q * kGroupWords + word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int k = 0; k < kMost; ++k) {
      const int q = (tid >> bits) + k * parts;
      if (q < n_tiles && word < n_words && (uint32_t)(v[k] >> 32) != launch + 1u) wanted |= 1u << k;
    }
    if (wanted == 0u) break;
  }
  if (gw.spins == 0) wanted = ~0u;                     // (a test's: nothing has been read)
  uint32_t sum[2][2] = {{0u, 0u}, {0u, 0u}};           // before, total; even and odd application
#pragma unroll
  for (int k = 0; k < kMost; ++k) {
    const int q = (tid >> bits) + k * parts;
    if (q >= n_tiles || word >= n_words || (wanted >> k & 1u) != 0u) continue;
    const uint32_t c[2] = {(uint32_t)v[k] & 0xffffu, (uint32_t)(v[k] >> 16) & 0xffffu};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      sum[1][h] += c[h];
      sum[0][h] += q < tile ? c[h] : 0u;
    }
  }
  for (int o = nw; o < kWave; o <<= 1)
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int h = 0; h < 2; ++h) sum[e][h] += __shfl_xor(sum[e][h], o);
  if (lane < nw) {
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int h = 0; h < 2; ++h) red[wave][e][2 * lane + h] = sum[e][h];
  }
  __syncthreads();
  if (tid < 256) {
    uint32_t sb = 0, stt = 0;
    if (tid <= A) {
#pragma unroll
      for (int u = 0; u < kGroupWaves; ++u) {
        sb += red[u][0][tid];
        stt += red[u][1][tid];
      }
    }
    before[tid] = sb;
    total[tid] = stt;
  }
  if (wanted != 0u) {
#pragma unroll
    for (int k = 0; k < kMost; ++k) {
      const int q = (tid >> bits) + k * parts;
      if (q < n_tiles && word < n_words && (wanted >> k & 1u) != 0u) {
        atomicOr(&lost[q], 1u << word);
        any_lost = 1;
      }
    }
  }
  // (all words read: the last workgroup to come here makes the launch's number the next one's)
  if (tid == 0 && atomicAdd(gw.launch, 1u) == (uint32_t)n_tiles) {
    __hip_atomic_store(gw.launch, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(gw.launch + 1, launch + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (any_lost == 0) return;
  // what has not come, from the ids: a wavefront takes every kGroupWaves-th tile, sixteen ids a lane at a time
  constexpr int kAtATime = 16;
  for (int q = wave; q < n_tiles; q += kGroupWaves) {
    const uint32_t words = lost[q];
    if (words == 0u) continue;                         // (uniform in the wavefront)
    const int end = min((q + 1) * tile_size, n);
    for (int i0 = q * tile_size + lane; i0 - lane < end; i0 += kAtATime * kWave) {
      uint32_t id[kAtATime];
#pragma unroll
      for (int e = 0; e < kAtATime; ++e) id[e] = (uint32_t)app[min(i0 + e * kWave, n - 1)];
#pragma unroll
      for (int e = 0; e < kAtATime; ++e) {
        const uint32_t key = min(id[e], (uint32_t)A);
        // (those of the first lane's application at once: with few applications most are)
        const bool in = i0 + e * kWave < end && (words >> (key >> 1) & 1u) != 0u, with_first = key == (uint32_t)__builtin_amdgcn_readfirstlane((int)key);
        const uint32_t firsts = (uint32_t)__popcll(__ballot(in && with_first)), add = !with_first ? (in ? 1u : 0u) : lane == 0 ? firsts : 0u;
        if (add == 0u) continue;
        atomicAdd(&total[key], add);
        if (q < tile) atomicAdd(&before[key], add);
      }
    }
  }
  __syncthreads();
}

// The segments from the number of requests of every application (and of invalid ids, total[A]), at most 255 of them: one thread
// per application, tables in LDS, three barriers (k_group_place takes 4.0 us for 256 requests where tables in memory took 4.8), two
// more where tiles differ in cost.
__device__ __forceinline__ void segments_from_totals(const SegArgs& g, const Window& w, const uint32_t* total, int costly /*by_cost[tid]*/,
                                                     int cost /*cost[tid], or 0*/) {
  __shared__ int s_seg[257], s_tile[257], s_unit[257], s_app[256];
  __shared__ int wave_t[4], wave_u[4], wave_i[4];
  __shared__ unsigned long long dies[kXcds];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, A = g.A;
  if (wave == 0) {
    const uint4 b = wave_digit_bases(total, 0u, lane);
    s_seg[4 * lane] = (int)b.x;
    s_seg[4 * lane + 1] = (int)b.y;
    s_seg[4 * lane + 2] = (int)b.z;
    s_seg[4 * lane + 3] = (int)b.w;
    if (lane == 0) s_seg[256] = g.n;
    if (lane < kXcds) dies[lane] = 0ull;
  }
  __syncthreads();
  if (tid <= A + 1) g.seg[tid] = s_seg[tid];                        // seg[A] = number of valid requests, seg[A+1] = n
  bool in_turn = false;
  if (g.cost != nullptr) {                                          // (uniform)
    const int nt = tid < A ? (s_seg[tid + 1] - s_seg[tid] + g.tile - 1) / g.tile : 0;
    int first = (int)wave_scan_incl((uint32_t)nt) - nt;
    if (lane == 63 && wave < 4) wave_i[wave] = first + nt;
    __syncthreads();
    for (int v = 0; v < min(wave, 4); ++v) first += wave_i[v];
    if (tid < A) add_to_dies(dies, first, nt, cost, wave_i[0] + wave_i[1] + wave_i[2] + wave_i[3]);
    __syncthreads();
    in_turn = dies_uneven(dies);
  }
  int ts = 0, us = 0, ti = 0, ui = 0;
  if (tid < 256) {
    if (tid < A) {
      const int c = in_turn ? costly : tid;
      plain_group(w, tid, s_seg[tid], s_seg[tid + 1]);
      s_app[tid] = c;
      ts = (s_seg[c + 1] - s_seg[c] + g.tile - 1) / g.tile;
      us = (s_seg[tid + 1] - s_seg[tid] + g.unit - 1) / g.unit;
    }
    ti = (int)wave_scan_incl((uint32_t)ts);
    ui = (int)wave_scan_incl((uint32_t)us);
    if (lane == 63) {
      wave_t[wave] = ti;
      wave_u[wave] = ui;
    }
  }
  if (tid == 0) {
    w.grp_n[0] = A;
    w.grp_n[1] = 1;
  }
  __syncthreads();
  if (tid < 256) {
    for (int v = 0; v < wave; ++v) {
      ti += wave_t[v];
      ui += wave_u[v];
    }
    if (tid <= A) {
      s_tile[tid] = ti - ts;
      s_unit[tid] = ui - us;
      g.unit_start[tid] = ui - us;
    }
  }
  __syncthreads();
  write_descriptors(g, in_turn, s_tile, s_unit, s_seg, s_app, tid, kGroupThreads);
}

// Every request to its grouped position (applications in ascending order, request ids ascending inside), with its deadline
// and weight (the scoring kernel then reads them in order instead of gathering by request id, 4 useful bytes per 64-byte
// line).  One extra workgroup turns the counts into segment starts and descriptors.  Bound by three or four dependent
// trips to memory (2 us each), not by its 28 bytes per request.
// SELF > 0: the first kernel of a short window; it counts 2,048 SELF ids itself and resets the window's state.  SELF < 0: the first kernel
// too; its workgroups hand each other their counts (GroupWords).
template <int ITEMS, int SELF = 0>
__global__ __launch_bounds__(kGroupThreads) void k_group_place(int n, int A, int nbits, const int32_t* __restrict__ app,
                                                               const float* __restrict__ D, const float* __restrict__ weight,
                                                               const uint32_t* __restrict__ counts, int n_tiles,
                                                               int32_t* __restrict__ ids_out, float2* __restrict__ dw_out,
                                                               SegArgs sg, Window sw, State* st, GroupWords gw) {
  constexpr int kTile = kGroupThreads * ITEMS;
  __shared__ uint32_t before[256];
  __shared__ __align__(16) uint32_t total[256];        // (read four words at a time: wave_digit_bases)
  __shared__ uint32_t red[kGroupWaves][2][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (blockIdx.x == 0) {              // (the first: as the last it would wait for a place on a full chip)
    const int costly = sg.by_cost[min(tid, A - 1)], cost = sg.cost != nullptr ? sg.cost[min(tid, A - 1)] : 0;
    loaded_here(costly); loaded_here(cost);
    if constexpr (SELF > 0) {
      if (tid == 0) reset_state(st);
      group_sums_self<SELF>(app, n, 0, kTile, A, before, total, red);
    } else if constexpr (SELF < 0) {
      if (tid == 0) reset_state(st);
      group_sums_handed(gw, gw.launch[1], app, n, n_tiles, 0, kTile, A, before, total, red);
    } else {
      group_sums(counts, n_tiles, 0, A, nbits, before, total, red);
    }
    if (tid == 0 && total[A] != 0u) atomicOr(&st->err, kErrApp);
    segments_from_totals(sg, sw, total, costly, cost);
    return;
  }
  // neighbouring tiles write neighbouring runs of every application: on one die, so that the lines they meet in are whole
  // when they leave its L2
  const int tile = xcd_tile(blockIdx.x - 1, n_tiles);
  if (tile < 0) return;
  __shared__ uint32_t cnt[kGroupWaves][256];
  __shared__ uint32_t lstart[256], dbase[256];
  __shared__ uint32_t wave_tot[kGroupWaves];
  __shared__ int32_t sval[kTile];
  __shared__ float2 spay[kTile];
  __shared__ uint8_t skey[kTile];
  for (int i = tid; i < kGroupWaves * 256; i += kGroupThreads) cnt[0][i] = 0u;
  const int beg = tile * kTile;
  const uint32_t launch = SELF < 0 ? gw.launch[1] : 0u;
  uint32_t key[ITEMS];
  float2 pay[ITEMS];
  bool bad = false;
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const int i = beg + (wave * ITEMS + c) * 64 + lane;
    key[c] = i < n ? sort_key_at((const uint32_t*)app, i, A, bad) : 0u;
    pay[c] = i < n ? make_float2(D[i], weight[i]) : make_float2(0.f, 0.f);
  }
  // (the barriers in here cover the cleared counts)
  if constexpr (SELF > 0) group_sums_self<SELF>(app, n, tile, kTile, A, before, total, red);
  else if constexpr (SELF == 0) group_sums(counts, n_tiles, tile, A, nbits, before, total, red);
  else __syncthreads();
  // rank inside the wavefront: lanes with my application ahead of me in this chunk, plus the wavefront's earlier chunks
  const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint32_t rank[ITEMS];
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const bool valid = beg + (wave * ITEMS + c) * 64 + lane < n;
    const unsigned long long same = match_bits(key[c], valid, nbits);
    const int leader = valid ? (__ffsll((long long)same) - 1) : lane;
    uint32_t ahead = 0;
    if (valid && lane == leader) ahead = atomicAdd(&cnt[wave][key[c]], (uint32_t)__popcll(same));
    ahead = __shfl(ahead, leader);
    rank[c] = ahead + (uint32_t)__popcll(same & lt);
  }
  __syncthreads();
  uint32_t mine = 0;
  if (tid <= A) {
#pragma unroll
    for (int v = 0; v < kGroupWaves; ++v) {
      const uint32_t c = cnt[v][tid];
      cnt[v][tid] = mine;
      mine += c;
    }
  }
  if constexpr (SELF < 0) {
    if (tid < 256) lstart[tid] = mine;
    __syncthreads();
    publish_counts(gw, launch, tile, A, lstart);
    group_sums_handed(gw, launch, app, n, n_tiles, tile, kTile, A, before, total, red);
  }
  const uint32_t ls = scan256_excl<kGroupWaves>(tid < 256 ? mine : 0u, wave_tot);
  const uint32_t gs = scan256_excl<kGroupWaves>(tid < 256 ? total[tid] : 0u, wave_tot);
  if (tid < 256) {
    lstart[tid] = ls;
    dbase[tid] = gs + before[tid] - ls;
  }
  __syncthreads();
  // through LDS in sorted order, so that neighbouring threads write neighbouring elements
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const int i = beg + (wave * ITEMS + c) * 64 + lane;
    if (i < n) {
      const uint32_t p = lstart[key[c]] + cnt[wave][key[c]] + rank[c];
      skey[p] = (uint8_t)key[c];
      sval[p] = i;
      spay[p] = pay[c];
    }
  }
  __syncthreads();
  const int n_tile = min(kTile, n - beg);
  for (int j = tid; j < n_tile; j += kGroupThreads) {
    const uint32_t dst = dbase[skey[j]] + (uint32_t)j;
    ids_out[dst] = sval[j];
    dw_out[dst] = spay[j];
  }
}

// ---- ordering inside the applications ----

// Requests per run.  Short runs spread even a small window over the chip: with 4,096 a run took 19 us to sort (by radix passes) and
// the first merge of two runs 10; with 1,024 sorting takes 7 and a merge of up to sixteen runs 6 to 8.
constexpr int kRun = 1024;
constexpr int kRunThreads = 256;                       // (of a merge: four workgroups for a run's length)
constexpr int kRunItems = kRun / kRunThreads;
constexpr int kMergeWays = 16;                         // most runs merged at a time
constexpr int kMergeMax = 262144;                      // longest window that is ordered this way (see the top of this file)

// How many merge launches a window of n requests takes and how many runs each merges: the largest application may hold
// every run.
inline void merge_plan(int64_t n, int& levels, int& ways) {
  const int64_t runs = (n + kRun - 1) / kRun;
  levels = 0;
  ways = 1;
  if (runs <= 1) return;
  for (int64_t c = 1; c < runs; c *= kMergeWays) ++levels;
  for (ways = 2;; ++ways) {
    int64_t c = 1;
    for (int l = 0; l < levels; ++l) c *= ways;
    if (c >= runs) return;
  }
}

// This workgroup's run, or its share of one that PARTS workgroups take: elements [beg, end) of the segment [s0, se).  Runs are
// dealt to the dies in contiguous eighths of the launch (see xcd_tile; the launch holds a multiple of 8 PARTS workgroups).
template <int PARTS>
__device__ __forceinline__ bool my_run(const SortPlan& sp, int& s0, int& beg, int& end, int& se) {
  const int at = (blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds, unit = at / PARTS;
  const int4 d = sp.desc[unit];                       // (the array covers the launch)
  if (unit >= sp.unit_start[sp.nseg]) return false;
  s0 = __builtin_amdgcn_readfirstlane(d.x);
  beg = __builtin_amdgcn_readfirstlane(d.y) + at % PARTS * (kRun / PARTS);
  se = __builtin_amdgcn_readfirstlane(d.z);
  end = min(beg + kRun / PARTS, se);
  return beg < end;
}

// What a launch of the ordering reads and writes: sort keys, positions of the application-grouped array, subgroup labels
// (with subgroups).
struct SortedRun {
  uint32_t* key;
  int32_t* pos;
  uint32_t* label;
};

// A request at its final service position: id, deadline and weight come with one gather of the record the scoring kernel
// left at the grouped position, the key straight from the sorted key bits.
__device__ __forceinline__ void finish_position(const Window& w, int at, uint32_t key, int gpos, int edf) {
  const float4 rc = w.rec_g[gpos];
  const int id = __float_as_int(rc.x);
  w.id_s[at] = id;
  w.D_s[at] = rc.y;
  w.w_s[at] = rc.z;
  // sorted were the inverted key bits, or (earliest deadline first) the deadline bits
  w.key_s[at] = edf ? w.key[id] : __uint_as_float(~key);
  w.alive_s[at] = 1;
}

// The last launch also resets the per-request outputs (by request id) and what lies behind the valid requests.
template <int THREADS>
__device__ __forceinline__ void finish_rest(const Window& w, int n, int n_valid_at, const int32_t* __restrict__ seg) {
  const int nv = seg[n_valid_at], i = blockIdx.x * THREADS + threadIdx.x;
  if (i >= n) return;
  if (i >= nv) w.alive_s[i] = 0;
  w.model[i] = -1;
  w.round_of[i] = -1;
  w.order_of[i] = 0;
  w.util[i] = 0.f;
}

// The value of lane ^ J, without LDS: quad permutes, a mirrored half row and a reversed quad, a row turned by eight, swapped rows
// and halves.
template <int J>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v, int lane) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  if (J == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, false);
  if (J == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, false);
  if (J == 4) return (uint32_t)__builtin_amdgcn_update_dpp(0, __builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, false), 0x1B, 0xf, 0xf, false);
  if (J == 8) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false);
  const u32x2 sw = J == 16 ? __builtin_amdgcn_permlane16_swap(v, v, false, false) : __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return (lane & J) ? sw[0] : sw[1];
}
// The steps of a bitonic stage inside a wavefront, from distance J down: ascending where `up`.
template <int J>
__device__ __forceinline__ void bitonic_steps(unsigned long long& v, bool up, int lane) {
  const unsigned long long p = ((unsigned long long)lane_xor<J>((uint32_t)(v >> 32), lane) << 32) | (unsigned long long)lane_xor<J>((uint32_t)v, lane);
  v = (p < v) == (((lane & J) == 0) == up) ? p : v;
  if constexpr (J > 1) bitonic_steps<J / 2>(v, up, lane);
}

// Sorts one run by one element per thread: a bitonic network over (label, key, place in the run) packed into 58 bits, so that
// no two are equal and the order is stable.  The 45 steps between lanes of a wavefront (of 55 for a full run) take no LDS and no barrier, the
// others one of each; runs of fewer elements take the stages they need.  Bound by about eight vector instructions a step with four
// wavefronts per SIMD: 6.8 us for full runs, 4.0 for 256 elements, 7.2 with subgroups; 8.0, 8.2 and 10.2 with stable passes of 8 bits
// through LDS (four barriers each); 8.4, 6.3 and 8.9 with four elements per thread in four wavefronts, one to a SIMD.
template <bool SPLIT, bool FINISH>
__global__ __launch_bounds__(kRun) void k_sort_runs(SortPlan sp, SortedRun in, SortedRun out, const int32_t* __restrict__ sub_g, int n,
                                                    Window w, int edf) {
  static_assert(kRun == 1024, "ten bits of place, one element per thread");
  __shared__ unsigned long long exchange[2][kRun];
  const int tid = threadIdx.x, lane = tid & 63;
  if (FINISH) finish_rest<kRun>(w, n, sp.nseg, sp.seg);
  int s0, beg, end, se;
  if (!my_run<1>(sp, s0, beg, end, se)) return;
  const int len = end - beg;
  unsigned long long v = ~0ull;                                // behind everything (labels have 16 bits: 65,536 slots)
  if (tid < len) {
    v = ((unsigned long long)in.key[beg + tid] << 10) | (unsigned long long)tid;
    if (SPLIT) v |= (unsigned long long)(uint32_t)sub_g[beg + tid] << 42;
  }
  bitonic_steps<1>(v, (tid & 2) == 0, lane);
  bitonic_steps<2>(v, (tid & 4) == 0, lane);
  bitonic_steps<4>(v, (tid & 8) == 0, lane);
  bitonic_steps<8>(v, (tid & 16) == 0, lane);
  bitonic_steps<16>(v, (tid & 32) == 0, lane);
  bitonic_steps<32>(v, (tid & 64) == 0, lane);
  int turn = 0;
  for (int k = 128; k / 2 < len; k *= 2) {                     // (uniform)
    const bool up = (tid & k) == 0;
    for (int j = k / 2; j >= 64; j /= 2) {
      exchange[turn][tid] = v;
      __syncthreads();
      const unsigned long long p = exchange[turn][tid ^ j];
      v = (p < v) == (((tid & j) == 0) == up) ? p : v;
      turn ^= 1;                                               // (read until the next step's barrier)
    }
    bitonic_steps<32>(v, up, lane);
  }
  if (tid >= len) return;
  const uint32_t key = (uint32_t)(v >> 10);
  const int32_t pos = beg + (int)(v & 1023u);
  if (SPLIT) out.label[beg + tid] = (uint32_t)(v >> 42);
  if (FINISH) {
    finish_position(w, beg + tid, key, pos, edf);
  } else {
    out.key[beg + tid] = key;
    out.pos[beg + tid] = pos;
  }
}

// Merges up to `ways` sorted runs of run_chunks * kRun elements of the same application.  A workgroup owns a quarter of a
// chunk of one run, one element per thread; the place of an element is its place in its own run plus, for every sibling run, the
// number of elements there that precede it (equal keys: the earlier run first, so the order is stable).  A sibling is looked
// at in chunks of kRun: the chunks that lie wholly before or wholly behind the workgroup's own elements are settled by their
// first and last key, the others (one to three per sibling, for keys in no particular order) are brought into LDS, kBatch of
// them in one trip to memory, and searched.  Bound by three dependent
// trips to memory and by the searches (four instructions for each of eleven steps, element and chunk), which a quarter of a
// chunk per workgroup spreads over the chip: 15 us with whole chunks, 6.7 with quarters (65,536 requests of 8 applications).
template <bool SPLIT, bool FINISH>
__global__ __launch_bounds__(kRunThreads) void k_merge_runs(SortPlan sp, SortedRun in, SortedRun out, int run_chunks, int ways,
                                                            int n, Window w, int edf) {
  typedef typename std::conditional<SPLIT, unsigned long long, uint32_t>::type K;     // label << 32 | key, or the key
  constexpr int kBatch = 8;                                    // chunks brought into LDS together
  __shared__ K chunk[kBatch][kRun];
  __shared__ int32_t active[kRunThreads];
  __shared__ int n_active;
  __shared__ uint32_t whole;                                   // elements of chunks that lie wholly before
  const int tid = threadIdx.x;
  if (FINISH) finish_rest<kRunThreads>(w, n, sp.nseg, sp.seg);
  int s0, beg, end, se;
  if (!my_run<kRunItems>(sp, s0, beg, end, se)) return;
  const int na = se - s0, len = end - beg, o = beg - s0;
  // chunk numbers inside the application (a run starts at a multiple of kRun): the runs merged here are the chunks
  // [c0, c1), this workgroup's own run the chunks [m0, m1)
  const int n_chunks = (na + kRun - 1) / kRun, mine = o / kRun;
  const int c0 = mine / (run_chunks * ways) * (run_chunks * ways), c1 = min(c0 + run_chunks * ways, n_chunks);
  const int m0 = mine / run_chunks * run_chunks, m1 = min(m0 + run_chunks, n_chunks);
  auto load_key = [&](int e) -> K {                            // e: element of the application
    if constexpr (SPLIT) return ((unsigned long long)in.label[s0 + e] << 32) | in.key[s0 + e];
    else return in.key[s0 + e];
  };
  const K key = tid < len ? load_key(o + tid) : ~K(0);
  const int32_t val = tid < len ? in.pos[beg + tid] : 0;
  uint32_t rank = (uint32_t)(o - m0 * kRun) + tid;
  if (c1 - c0 > m1 - m0) {                                     // (uniform) there are siblings
    const K first_key = load_key(o), last_key = load_key(o + len - 1);
    for (int cb = c0; cb < c1; cb += kRunThreads) {
      // (these keys travel with the elements' own: one trip to memory for both)
      const int ch = cb + tid;
      const bool sibling = ch < c1 && !(ch >= m0 && ch < m1);
      K kf = 0, kl = 0;
      if (sibling) {
        kf = load_key(ch * kRun);
        kl = load_key(min(ch * kRun + kRun, na) - 1);
      }
      if (tid == 0) {
        n_active = 0;
        whole = 0u;
      }
      __syncthreads();
      if (sibling) {
        const bool earlier = ch < m0;                          // an earlier run goes first among equal keys
        if (earlier ? kl <= first_key : kl < first_key) atomicAdd(&whole, (uint32_t)(min(ch * kRun + kRun, na) - ch * kRun));
        else if (earlier ? kf <= last_key : kf < last_key) active[atomicAdd(&n_active, 1)] = ch;
      }
      __syncthreads();
      const int n_act = n_active;
      const uint32_t n_whole = whole;
      rank += n_whole;
      for (int q0 = 0; q0 < n_act; q0 += kBatch) {
        // all loads of the batch go out before the first is stored; what lies behind the last element or the last chunk
        // sorts last and is not counted
        K in_flight[kBatch][kRunItems];
        int id_q[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) id_q[q] = q0 + q < n_act ? __builtin_amdgcn_readfirstlane(active[q0 + q]) : n_chunks;
#pragma unroll
        for (int q = 0; q < kBatch; ++q)
#pragma unroll
          for (int c = 0; c < kRunItems; ++c) {
            const int e = id_q[q] * kRun + c * kRunThreads + tid;
            in_flight[q][c] = ~K(0);
            if (e < na) in_flight[q][c] = load_key(e);
          }
#pragma unroll
        for (int q = 0; q < kBatch; ++q)
#pragma unroll
          for (int c = 0; c < kRunItems; ++c) chunk[q][c * kRunThreads + tid] = in_flight[q][c];
        __syncthreads();
#pragma unroll
        for (int h = 0; h < kBatch; h += 4) {                  // the searches of four chunks side by side
          if (q0 + h >= n_act) break;
          uint32_t at[4];
          K less[4];                                           // counted is what is less than this
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            at[q] = 0;
            less[q] = id_q[h + q] < m0 ? key + 1 : key;
          }
#pragma unroll
          for (int step = kRun / 2; step > 0; step >>= 1)
#pragma unroll
            for (int q = 0; q < 4; ++q) at[q] += chunk[h + q][at[q] + step - 1] < less[q] ? step : 0;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const uint32_t clen = (uint32_t)max(0, min(kRun, na - id_q[h + q] * kRun));
            at[q] += chunk[h + q][at[q]] < less[q] ? 1 : 0;
            // (the largest key of all, in an earlier run: everything there goes first)
            if (id_q[h + q] < m0 && key == ~K(0)) at[q] = clen;
            rank += min(at[q], clen);
          }
        }
        __syncthreads();
      }
      __syncthreads();                                         // n_active and whole are cleared for the next chunks
    }
  }
  if (tid >= len) return;
  const int at = s0 + c0 * kRun + (int)rank;
  if constexpr (SPLIT) out.label[at] = (uint32_t)(key >> 32);
  if (FINISH) {
    finish_position(w, at, (uint32_t)key, val, edf);
  } else {
    out.key[at] = (uint32_t)key;
    out.pos[at] = val;
  }
}

// ---- the same for long windows: radix passes, then a gather ----

// Subgroup codes as sort keys, in the current order of the passes' values (grouped positions).
__global__ void k_gather_sub_keys(int n_valid_at, const int32_t* __restrict__ seg, const int32_t* __restrict__ grouped_pos,
                                  const int32_t* __restrict__ sub_g, uint32_t* __restrict__ keys, const State* st) {
  if (st->err & kErrSortSync) return;                  // (the passes have left positions unwritten)
  const int pos = blockIdx.x * blockDim.x + threadIdx.x;
  if (pos < seg[n_valid_at]) keys[pos] = (uint32_t)sub_g[grouped_pos[pos]];
}

// After the last pass: positions of the application-grouped array travelled as values.
__global__ void k_finish_order(int n, int n_valid_at, const int32_t* __restrict__ seg, const int32_t* __restrict__ grouped_pos,
                               const uint32_t* __restrict__ sorted_keys, Window w, int edf) {
  finish_rest<kRunThreads>(w, n, n_valid_at, seg);
  if (w.st->err & kErrSortSync) return;                // (the passes have left positions unwritten)
  const int pos = blockIdx.x * kRunThreads + threadIdx.x;
  if (pos < seg[n_valid_at]) finish_position(w, pos, sorted_keys[pos], grouped_pos[pos], edf);
}

// Range of every possible (application, subgroup code) pair in the service order: two binary searches on
// the sorted codes inside the application's range.  Slot s belongs to application slot_app[s] and code
// s - slot_base[application].
__global__ void k_slot_ranges(int n_slots, const int32_t* __restrict__ slot_app, const int32_t* __restrict__ slot_base,
                              const int32_t* __restrict__ seg, const uint32_t* __restrict__ sub_sorted,
                              int32_t* __restrict__ slot_beg, int32_t* __restrict__ slot_end) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n_slots) return;
  const int a = slot_app[s];
  const uint32_t code = (uint32_t)(s - slot_base[a]);
  const int b0 = seg[a], e0 = seg[a + 1];
  int lo = b0, hi = e0;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (sub_sorted[mid] < code) lo = mid + 1; else hi = mid;
  }
  const int beg = lo;
  hi = e0;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (sub_sorted[mid] <= code) lo = mid + 1; else hi = mid;
  }
  slot_beg[s] = beg;
  slot_end[s] = lo;
}

// The non-empty slots, in slot order, become the groups of the rounds.  One workgroup.
__global__ __launch_bounds__(1024) void k_groups_compact(int n_slots, const int32_t* __restrict__ slot_app,
                                                         const int32_t* __restrict__ slot_beg,
                                                         const int32_t* __restrict__ slot_end, Window w,
                                                         int32_t* __restrict__ grp_n_host /*pinned [2]*/) {
  __shared__ int wave_cnt[16];
  __shared__ int base_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) base_s = 0;
  __syncthreads();
  for (int s0 = 0; s0 < n_slots; s0 += 1024) {
    const int s = s0 + tid;
    const bool full = s < n_slots && slot_end[s] > slot_beg[s];
    const unsigned long long bal = __ballot(full);
    if (lane == 0) wave_cnt[wave] = __popcll(bal);
    __syncthreads();
    int before = base_s, total = 0;
    for (int i = 0; i < 16; ++i) {
      if (i < wave) before += wave_cnt[i];
      total += wave_cnt[i];
    }
    if (full) {
      const int j = before + __popcll(bal & ((1ull << lane) - 1ull));
      if (j < w.gcap) {
        w.grp_app[j] = slot_app[s];
        w.grp_end[j] = slot_end[s];
        w.head[j] = slot_beg[s];
        w.head[w.gcap + j] = slot_beg[s];
      }
    }
    __syncthreads();
    if (tid == 0) base_s += total;
    __syncthreads();
  }
  const int G = min(base_s, w.gcap);
  // the most groups any application has (the groups of an application are consecutive): it decides whether
  // the resident rounds kernel, whose workgroups each serve all groups of one application, can take the window
  __shared__ int max_run;
  if (tid == 0) max_run = 0;
  __threadfence();
  __syncthreads();
  for (int j = tid; j < G; j += 1024) {
    const int a = w.grp_app[j];
    if (j == 0 || w.grp_app[j - 1] != a) {
      int lo = j, hi = G;                                 // first index past j whose application is not a
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (w.grp_app[mid] == a) lo = mid; else hi = mid;
      }
      atomicMax(&max_run, hi - j);
    }
  }
  __syncthreads();
  if (tid == 0) {
    w.grp_n[0] = G;
    w.grp_n[1] = max_run;
    grp_n_host[0] = G;
    grp_n_host[1] = max_run;
  }
}

// Both in one workgroup, for up to kFewSlots slots: a slot ends where the next one begins, so one search is enough, four ways at a time
// (both kernels wait for one dependent trip to memory after the other).  Eight applications of 101 slots, 65,536 requests: 6.5 + 7.2 us
// -> 7.6.
constexpr int kFewSlots = 1024;
__global__ __launch_bounds__(kFewSlots) void k_groups_few(int n_slots, const int32_t* __restrict__ slot_app, const int32_t* __restrict__ slot_base,
                                                          const int32_t* __restrict__ seg, const uint32_t* __restrict__ sub_sorted, Window w,
                                                          int32_t* __restrict__ grp_n_host /*pinned [2]*/) {
  __shared__ int wave_cnt[kFewSlots / kWave], beg_s[kFewSlots], of_app[kFewSlots];
  __shared__ int max_run;
  const int s = threadIdx.x, lane = s & 63, wave = s >> 6;
  of_app[s] = 0;
  if (s == 0) max_run = 0;
  const int a = slot_app[min(s, n_slots - 1)];
  const int base = slot_base[a], b0 = seg[a], e0 = seg[a + 1];
  const bool last = s + 1 >= n_slots || slot_app[s + 1] != a;    // (of its application)
  const uint32_t code = (uint32_t)(s - base);
  int lo = b0, hi = s < n_slots ? e0 : b0;                        // first position with at least this code
  while (lo < hi) {
    const int step = (hi - lo) / 4, p0 = lo + step, p1 = p0 + step, p2 = p1 + step;    // lo <= p0 <= p1 <= p2 < hi
    const uint32_t c0 = sub_sorted[p0], c1 = sub_sorted[p1], c2 = sub_sorted[p2];
    if (c2 < code) lo = p2 + 1;
    else if (c1 < code) { lo = p1 + 1; hi = p2; }
    else if (c0 < code) { lo = p0 + 1; hi = p1; }
    else hi = p0;
  }
  beg_s[s] = lo;
  __syncthreads();
  const int end = last ? e0 : beg_s[s + 1];
  const bool full = s < n_slots && end > lo;
  const unsigned long long bal = __ballot(full);
  if (lane == 0) wave_cnt[wave] = __popcll(bal);
  if (full) atomicAdd(&of_app[a], 1);                             // (every application has a slot, so there are no more of them than slots)
  __syncthreads();
  int before = 0, total = 0;
  for (int i = 0; i < kFewSlots / kWave; ++i) {
    before += i < wave ? wave_cnt[i] : 0;
    total += wave_cnt[i];
  }
  if (of_app[s] > 0) atomicMax(&max_run, of_app[s]);
  if (full) {
    const int j = before + __popcll(bal & ((1ull << lane) - 1ull));
    if (j < w.gcap) {
      w.grp_app[j] = a;
      w.grp_end[j] = end;
      w.head[j] = lo;
      w.head[w.gcap + j] = lo;
    }
  }
  __syncthreads();
  if (s == 0) {
    grp_n_host[0] = w.grp_n[0] = min(total, w.gcap);
    grp_n_host[1] = w.grp_n[1] = max_run;
  }
}

// The same two numbers of an empty window for the host, in the order of the stream: an earlier window's k_groups_compact may
// still be on its way there.
__global__ void k_groups_publish(Window w, int32_t* __restrict__ grp_n_host /*pinned [2]*/) {
  if (threadIdx.x < 2) grp_n_host[threadIdx.x] = w.grp_n[threadIdx.x];
}

}  // namespace sp
