// One greedy round in one launch of one workgroup (Alg. 1 generalised to batch-capped rounds; eq. (2), eq. (13), eq. (1) as in
// sp_rounds.h, decision for decision), for profiles small enough that one compute unit evaluates a round's candidates in the time
// that a second kernel would cost.
//
// One wavefront per application brings the application's window into LDS; the triangles of all (application, variant) pairs
// are dealt to sixteen wavefronts, four lanes per pair of batch sizes; every wavefront takes the maximum over the wavefronts'
// candidates; one of them writes the batch out.  Bound by its dependent trips to memory (state; records; accuracies; about 0.8 us
// each) and by about 1.5 us of triangles: 5.6 us for one application of three variants and batches of 16 (13.8 in a launch of
// resident workgroups), 7.9 for three of four and batches of 32 (9.0 + 6.0 as two kernels, and the gap between them).
#pragma once
#include "sp_rounds.h"

namespace sp {

typedef float ea_quad __attribute__((ext_vector_type(4)));

constexpr int kSingleThreads = 1024;
constexpr int kSingleWaves = kSingleThreads / kWave;
constexpr int kSingleApps = kSingleWaves - 1;        // one wavefront brings each window, the others clear outputs
constexpr int kSingleBatch = kWave;                  // largest batch: one lane per member
// Entries per application: a window that lacks one, and 64 more (whole groups of sixteen are read).
__host__ __device__ inline int single_cap(int Bcap) { return (Bcap - 1 + kWave + 15) / 16 * 16; }
constexpr int kSingleScan = 16;                      // service positions per lane of a walk over dead requests, in each ...
constexpr int kSingleBlocks = 2;                     // ... of the blocks of a step
// Up to what this kernel is used: a round's utility evaluations (with the group-first rule one application's: the others are not
// evaluated), and kSingleSlot for each pair of batch sizes of each (application, variant), which four lanes take together.  us per call
// of sp_greedy_round, two kernels against this one, and evaluations + 14 pairs of sizes: 23.5 / 17.2 (1,472: one application of 16
// variants, batches of 8), 24.1 / 18.9 (11,136: six of 8, 15), 24.0 / 21.4 (24,064: two of 16, 32), 24.3 / 22.8 (29,952: eight of 8, 24),
// 24.8 / 24.5 (33,600: six of 16, 20), 24.0 / 22.5 (40,448: one of 16, 64), 24.4 / 25.5 (41,184: eleven of 8, 24), 24.7 / 26.9 (42,000:
// fifteen of 8, 20), 25.0 / 27.9 (40,832: eleven of 16, 15), 24.2 / 25.3 (45,360: fifteen of 2, 48).  Group first: 27.3 / 20.5 (18,560:
// eight of 8, 32), 27.3 / 22.3 (30,912: eight of 8, 48), 27.8 / 24.5 (37,120: eight of 16, 32), 27.2 / 26.2 (54,784: three of 16, 64),
// 27.6 / 27.7 (56,064: eleven of 8, 64), 27.3 / 27.6 (61,952: four of 16, 64).
constexpr int64_t kSingleSlot = 14, kSingleCost = 40500, kSingleCostGroupFirst = 55000;
// Dynamic LDS.  A workgroup that asks for more waits for a compute unit that is next to empty: beside two streams of matrix products and
// one of elementwise kernels one call in ten took 0.4 to 0.7 ms with 122 to 146 KB, 0.07 as with two kernels up to 120.
constexpr size_t kSingleLds = 110 * 1024;
// Requests up to which it fills the caller's outputs (while it reads the windows).
constexpr int kSingleOutputs = 16384;

struct Single {
  Outputs out;                  // the caller's arrays, when this round starts a window and fills them (else null)
  int32_t* ids_out;             // members of the batch for the caller, or null
  Decision* log_host;           // pinned: the decision, or null
  long long* ticks;             // constant-rate timestamps, launch start and decision, or null
};

// Groups of four variants whose accuracies an entry holds.
constexpr int single_quads(int Mmax) { return Mmax <= 4 ? 1 : Mmax <= 8 ? 2 : 4; }
// Dynamic LDS: entries, latencies.
inline size_t single_lds_bytes(int A, int Mmax, int B, int Bcap) {
  return (size_t)A * single_cap(Bcap) * (2 + single_quads(Mmax)) * 16 + (size_t)A * Mmax * B * 4;
}

// Candidate ids inside this kernel: fields instead of a product, the same order.
__device__ __forceinline__ uint32_t single_cid(int a, int m) { return ((uint32_t)a << 12) | ((uint32_t)m << 8); }
static_assert(kMaxModels <= 16 && kMaxBatch <= 256, "fields of a candidate id");

// Scores of the batch sizes p + 1 and Bw - p over a window of nw requests by four lanes: the sums of triangle_best, term for term
// and in its order (a lane holds 4 of its 16 partial sums).  Entries up to the next multiple of 16 behind the window are read
// but not counted.  About 13 instructions per evaluation and 60 around them.
template <int KIND>
__device__ __forceinline__ unsigned long long single_pair(const float4* e4, const float* ea_m, const float* lat, int p, int nw, int Bw,
                                                         double t0, uint32_t cid0, int only_b, int q /* lane of the four */) {
  const int b1 = p + 1, b2 = Bw - p;
  const int n1 = (only_b == 0 || b1 == only_b) ? b1 : 0;       // (p < nw)
  const int n2 = (b2 <= nw && b2 != b1 && (only_b == 0 || b2 == only_b)) ? b2 : 0;
  const double E1 = t0 + (double)lat[b1 - 1], E2 = t0 + (double)lat[b2 - 1];
  const float e1h = (float)E1, e1l = (float)(E1 - (double)e1h);
  const float e2h = (float)E2, e2l = (float)(E2 - (double)e2h);
  float s1[4] = {0.f, 0.f, 0.f, 0.f}, s2[4] = {0.f, 0.f, 0.f, 0.f};
  const int n = max(n1, n2) - 4 * q, m1 = n1 - 4 * q, m2 = n2 - 4 * q;
  e4 += 4 * q;
  ea_m += 16 * q;
  for (int j0 = 0; j0 < n; j0 += 16) {
    float4 e[4];
    float x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      e[i] = e4[j0 + i];
      x[i] = ea_m[4 * (j0 + i)];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[i] *= e[i].x;
      const float v = fmaf(x[i], one_minus_penalty_f32<KIND>(e[i].y, e[i].w, e[i].z, e2h, e2l), s2[i]);
      s2[i] = j0 + i < m2 ? v : s2[i];
    }
    if (j0 < m1) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = fmaf(x[i], one_minus_penalty_f32<KIND>(e[i].y, e[i].w, e[i].z, e1h, e1l), s1[i]);
        s1[i] = j0 + i < m1 ? v : s1[i];
      }
    }
  }
  const float r1 = sum4((s1[0] + s1[1]) + (s1[2] + s1[3]));
  const float r2 = sum4((s2[0] + s2[1]) + (s2[2] + s2[3]));
  // (the order of packed candidates: by the scores' bits, where a NaN is above every number, then the smaller size)
  const bool second = n2 > 0 && (n1 == 0 || __float_as_uint(r2) > __float_as_uint(r1));
  return (n1 | n2) > 0 ? pack_candidate(second ? r2 : r1, cid0 + (uint32_t)((second ? b2 : b1) - 1)) : 0ull;
}

// The smallest deadline that is_dead leaves alive at E0 >= 0: a comparison in 32 bits then says the same as its own in 64, for every
// deadline (E0 > D, or E0 >= 2 D; halving is exact).
__device__ __forceinline__ float least_live(int kind, double E0) {
  const double bound = kind == 0 ? E0 : 0.5 * E0;
  const float f = (float)bound;
  const bool above = kind == 0 ? (double)f >= bound : (double)f > bound;
  return above ? f : __uint_as_float(__float_as_uint(f) + 1u);         // (f >= 0: the next float)
}

// One step of a wavefront's walk over service positions that are mostly dead: the live ones among the next kSingleBlocks * 1,024 go to
// `found` behind the n that are there, up to kWave in all.  All loads go out before the first is used, from addresses that stay
// inside the application's range, so that no branch parts them.  About 0.9 us for 2,048 positions; 1,024 a step with comparisons in
// 64 bits took 1.5 us.  us per call of sp_greedy_round, two kernels / those steps / these (one application; most die at once, or in the
// course of the window): 16,384 requests 33 / 27 / 23 and 28 / 20.5 / 19, 65,536 35 / 35 / 25 and 28 / 21 / 19, 262,144 48 / 84 / 37 and 29
// / 26 / 20, 1,048,576 102 / 272 / 91 and 35 / 42 / 25.  Four blocks take more than 64 registers: 5.5 -> 6.0 us for the smallest windows.
__device__ __forceinline__ void walk_dead(const Window& w, float least, int& scan, int end, int32_t* found, int& n, int lane) {
  typedef uint32_t words __attribute__((ext_vector_type(4), aligned(4)));
  constexpr int kBlock = kSingleScan * kWave;
  const int base = scan & ~3, p0 = base + kSingleScan * lane, last = (end - 1) & ~3;     // (both arrays are padded by 16)
  float4 d[kSingleBlocks][kSingleScan / 4];
  words alive[kSingleBlocks];
#pragma unroll
  for (int u = 0; u < kSingleBlocks; ++u) {
    const int at = min(p0 + u * kBlock, last);
#pragma unroll
    for (int q = 0; q < kSingleScan / 4; ++q) d[u][q] = *reinterpret_cast<const float4*>(w.D_s + at + 4 * q);
    alive[u] = *reinterpret_cast<const words*>(w.alive_s + at);
  }
#pragma unroll
  for (int u = 0; u < kSingleBlocks; ++u) {
    if (n >= kWave) break;                             // (uniform)
    const int pu = p0 + u * kBlock;
    uint32_t mask = 0;
#pragma unroll
    for (int q = 0; q < kSingleScan / 4; ++q) {
      const uint32_t due = (d[u][q].x >= least ? 1u : 0u) | (d[u][q].y >= least ? 2u : 0u) | (d[u][q].z >= least ? 4u : 0u) |
                           (d[u][q].w >= least ? 8u : 0u);
      // (four bytes of 0 or 1 to four bits, others above them; what lies behind the window's end may be anything)
      const uint32_t pending = ((alive[u][q] & 0x01010101u) * 0x01020408u) >> 24;
      mask |= (due & pending) << (4 * q);
    }
    // inside [scan, end)
    mask &= ~0u << min(max(scan - pu, 0), kSingleScan);
    mask &= (1u << min(max(end - pu, 0), kSingleScan)) - 1u;
    const int cnt = __popc(mask), incl = (int)wave_scan_incl((uint32_t)cnt);
    int rank = n + incl - cnt;
    n = min(n + __builtin_amdgcn_readlane(incl, kWave - 1), kWave);
    while (mask != 0 && rank < kWave) {
      const int j = __ffs((int)mask) - 1;
      mask &= mask - 1;
      found[rank++] = pu + j;
    }
  }
  wave_sync();
  scan = n == kWave ? __builtin_amdgcn_readfirstlane(found[kWave - 1]) + 1 : min(base + kSingleBlocks * kBlock, end);
}

// QUADS: groups of four variants.
template <int QUADS>
__global__ __launch_bounds__(kSingleThreads) void k_round_single(Tables tb, Window w, Single sg) {
  extern __shared__ __align__(16) unsigned char single_lds[];
  __shared__ int32_t held_s[kSingleApps], scan_s[kSingleApps];      // entries in LDS; first service position behind them
  __shared__ int32_t kind_s[kSingleApps];
  __shared__ float swap_s[kSingleApps][kMaxModels], prio_s[kSingleApps];
  __shared__ uint8_t pair_s[kSingleApps * kMaxModels];              // application << 4 | variant of each pair
  __shared__ int32_t found_s[kSingleApps][kWave];                   // positions a walk has found
  __shared__ unsigned long long best_s[kSingleWaves];
  State* st = w.st;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int A = tb.A, B = tb.B, Bw = tb.Bcap, Mmax = tb.Mmax, cap = single_cap(Bw);
  float4* const dd = reinterpret_cast<float4*>(single_lds);                              // [A][cap] weight in a batch's sum, D, 1/D, 2D
  int4* const meta = reinterpret_cast<int4*>(dd + A * cap);                       // [A][cap] service position, request id, weight, ordering value
  ea_quad* const eas = reinterpret_cast<ea_quad*>(meta + A * cap);                // [A][QUADS][cap] expected accuracies
  float* const lat_s = reinterpret_cast<float*>(eas + A * QUADS * cap);           // [A][Mmax][B]
  const bool owner = wave < A;

  // ---- what the launch starts from: one trip to memory ----
  const double t = st->t, twu = st->total_wu, tu = st->total_u, tv = st->total_viol;
  const int round0 = st->round, last_a = st->last.app, last_m = st->last.model, next_order = st->next_order;
  const bool stopped = st->done || st->err;
  const int my_a = min(wave, A - 1);
  const int a_kind = tb.penalty[my_a], a_end = w.grp_end[my_a], head_even = w.head[my_a], head_odd = w.head[w.gcap + my_a];
  const float a_lmin = tb.lmin[my_a], a_swap = tb.swap[my_a * Mmax + min(lane, Mmax - 1)];
  const float lat0 = tb.lat[min(tid, A * Mmax * B - 1)];
  const int models = tb.n_models[min(lane, A - 1)];
  loaded_here(a_kind); loaded_here(a_end); loaded_here(head_even); loaded_here(head_odd); loaded_here(a_lmin); loaded_here(a_swap);
  loaded_here(lat0); loaded_here(models); loaded_here(twu); loaded_here(tu); loaded_here(tv); loaded_here(next_order); loaded_here(last_m);
  if (stopped) {
    if (tid == 0) {
      mirror_state(w);
      tell_host_ended(w);
    }
    return;
  }
  const int r = __builtin_amdgcn_readfirstlane(round0);
  if (tid == 0 && sg.ticks) sg.ticks[0] = wall_clock64();
  if (tid < A * Mmax * B) lat_s[tid] = lat0;
  for (int i = tid + kSingleThreads; i < A * Mmax * B; i += kSingleThreads) lat_s[i] = tb.lat[i];
  // the pairs, application-major
  const int pairs_incl = (int)wave_scan_incl((uint32_t)(lane < A ? models : 0));
  const int n_pairs = __builtin_amdgcn_readlane(pairs_incl, kWave - 1);
  if (wave == kSingleWaves - 1 && lane < A)
    for (int m = 0; m < models; ++m) pair_s[pairs_incl - models + m] = (uint8_t)(lane << 4 | m);

  if (owner) {
    // ---- the application's window: its first live requests ----
    const int kind = __builtin_amdgcn_readfirstlane(a_kind), end = __builtin_amdgcn_readfirstlane(a_end);
    int scan = __builtin_amdgcn_readfirstlane((r & 1) ? head_odd : head_even);
    const double E0 = t + (double)a_lmin;
    int held = 0;
    // 64 at a time: two dependent trips to memory where half of the next 64 positions are live, else one for every 2,048
    // positions and two more
    while (held < Bw && scan < end) {
      int pos = min(scan + lane, end - 1);
      int id = w.id_s[pos];
      float D = w.D_s[pos], key = w.key_s[pos], wt = w.w_s[pos];
      bool live = scan + lane < end && w.alive_s[pos] != 0 && !is_dead(kind, D, E0);
      if (__popcll(__ballot(live)) >= kWave / 2 || scan + kWave >= end) {
        scan = min(scan + kWave, end);
      } else {
        int n = 0;
        const float least = least_live(kind, E0);
        do walk_dead(w, least, scan, end, found_s[wave], n, lane); while (n < Bw && scan < end);
        live = lane < n;
        pos = n > 0 ? found_s[wave][min(lane, n - 1)] : end - 1;
        id = w.id_s[pos];
        D = w.D_s[pos];
        key = w.key_s[pos];
        wt = w.w_s[pos];
        wave_sync();
      }
      const float* row = w.ea + (int64_t)id * Mmax;
      ea_quad ea[QUADS];
#pragma unroll
      for (int q = 0; q < QUADS; ++q)
#pragma unroll
        for (int j = 0; j < 4; ++j) ea[q][j] = row[min(4 * q + j, Mmax - 1)];
      const unsigned long long bal = __ballot(live);
      if (live) {
        const int at = held + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
        dd[wave * cap + at] = make_float4(tb.pol_unit_weight ? 1.0f : key, D, 1.0f / D, 2.0f * D);
        meta[wave * cap + at] = make_int4(pos, id, __float_as_int(wt), __float_as_int(tb.pol_edf ? -D : key));
#pragma unroll
        for (int q = 0; q < QUADS; ++q) eas[(wave * QUADS + q) * cap + at] = ea[q];
      }
      held += __popcll(bal);
    }
    if (lane < Mmax) swap_s[wave][lane] = a_swap;
    if (tb.pol_group_first) {
      // eq. (14) over the window, in the order of block_sum_f64
      wave_sync();
      const int nw = min(held, Bw);
      double s = lane < nw ? (double)__int_as_float(meta[wave * cap + lane].w) : 0.0;
#pragma unroll
      for (int o = kWave / 2; o > 0; o >>= 1) s += __shfl_down(s, o);
      if (lane == 0) prio_s[wave] = nw > 0 ? (float)(s / (double)nw) : 0.f;
    }
    if (lane == 0) {
      held_s[wave] = held;
      scan_s[wave] = scan;
      kind_s[wave] = kind;
    }
  } else {
    // the caller's arrays as a window without rounds leaves them
    const int first = (wave - A) * kWave + lane, step = (kSingleWaves - A) * kWave;
    fill_output(sg.out.model, w.n, -1, first, step);
    fill_output(sg.out.round_of, w.n, -1, first, step);
    fill_output(sg.out.order_of, w.n, 0, first, step);
    fill_output(reinterpret_cast<int32_t*>(sg.out.util), w.n, 0, first, step);
  }
  __syncthreads();

  // ---- triangles ----
  // group first: the application with the highest priority among those with a window (ties: the smallest) alone competes
  int only_a = -1;
  if (tb.pol_group_first) {
    unsigned long long top = 0ull;
    if (lane < A && held_s[lane] > 0) top = ((unsigned long long)ordered_bits(prio_s[lane]) << 32) | (unsigned long long)(0xFFFFFFFFu - (uint32_t)lane);
    top = wave_max_u64(top);
    if (top != 0ull) only_a = (int)(0xFFFFFFFFu - (uint32_t)(top & 0xFFFFFFFFull));
  }
  unsigned long long best = 0ull;
  // pairs of batch sizes of all pairs, sixteen per wavefront and step: four lanes each
  const int sizes = (Bw + 1) / 2, n_slots = n_pairs * sizes;
  for (int slot = wave * (kWave / 4) + (lane >> 2); __builtin_amdgcn_ballot_w64(slot < n_slots) != 0ull; slot += kSingleWaves * (kWave / 4)) {
    const int pair = min(slot, n_slots - 1) / sizes, p = slot - pair * sizes;
    const int am = pair_s[pair], a = am >> 4, m = am & 15, nw = min(held_s[a], Bw);
    const bool on = slot < n_slots && p < nw && (only_a < 0 || a == only_a);     // (past nw neither size is a candidate)
    const int kind = scoring_penalty(tb, kind_s[a]);
    const double t0 = (last_a == a && last_m == m) ? t : t + (double)swap_s[a][m];
    const float4* e4 = dd + a * cap;
    const float* ea_m = reinterpret_cast<const float*>(eas + (a * QUADS + (m >> 2)) * cap) + (m & 3);
    const float* lat = lat_s + (a * Mmax + m) * B;
    const int only_b = tb.pol_whole ? nw : 0;
    unsigned long long c = 0ull;
    if (on && kind == 0) c = single_pair<0>(e4, ea_m, lat, p, nw, Bw, t0, single_cid(a, m), only_b, lane & 3);
    if (on && kind == 1) c = single_pair<1>(e4, ea_m, lat, p, nw, Bw, t0, single_cid(a, m), only_b, lane & 3);
    if (on && kind == 2) c = single_pair<2>(e4, ea_m, lat, p, nw, Bw, t0, single_cid(a, m), only_b, lane & 3);
    best = c > best ? c : best;
  }
  best = wave_max_packed(best);
  if (lane == 0) best_s[wave] = best;
  __syncthreads();
  best = wave_max_packed(lane < kSingleWaves ? best_s[lane] : 0ull);
  const uint32_t cid = 0xFFFFFFFFu - (uint32_t)best;
  const int a = best != 0ull ? (int)(cid >> 12) : -1, m = (int)(cid >> 8) & 15, b = (int)(cid & 0xffu) + 1;

  if (owner && lane == 0) {
    // first position that may still be live, for the next round
    const int skip = wave == a ? b : 0, held = held_s[wave];
    w.head[((r + (a >= 0 ? 1 : 0)) & 1) * w.gcap + wave] = skip < held ? meta[wave * cap + skip].x : scan_s[wave];
    atomicAdd(&st->n_evals, triangle_evals(min(held, Bw), tb.pol_whole) * (unsigned long long)tb.n_models[wave]);   // (as every route counts)
  }
  if (wave != kSingleWaves - 1) {
    stores_arrived();
    __syncthreads();                                   // (the last wavefront tells the host)
    return;
  }
  // ---- the batch: outputs, pending flags, the three sums (one member per lane, in the order of commit_members), the state ----
  if (best == 0ull) {                                  // nothing live anywhere
    if (lane == 0) {
      st->done = 1;
      mirror_state(w);
    }
    stores_arrived();
    __syncthreads();
    if (lane == 0) tell_host_ended(w);
    return;
  }
  const double E = ((last_a == a && last_m == m) ? t : t + (double)swap_s[a][m]) + (double)lat_s[(a * Mmax + m) * B + b - 1];
  double wu = 0.0, su = 0.0, viol = 0.0;
  if (lane < b) {
    const int at = a * cap + lane;
    const int4 mt = meta[at];
    const float4 e = dd[at];
    const float acc = reinterpret_cast<const float*>(eas + (a * QUADS + (m >> 2)) * cap + lane)[m & 3];
    const int pos = mt.x, id = mt.y;
    const float u = acc * one_minus_penalty(kind_s[a], e.y, e.z, E);
    w.model[id] = m;
    w.round_of[id] = r;
    w.order_of[id] = next_order + lane;
    w.util[id] = u;
    if (sg.out.model) sg.out.model[id] = m;
    if (sg.out.round_of) sg.out.round_of[id] = r;
    if (sg.out.order_of) sg.out.order_of[id] = next_order + lane;
    if (sg.out.util) sg.out.util[id] = u;
    w.alive_s[pos] = 0;
    w.last_ids[lane] = id;
    if (sg.ids_out) sg.ids_out[lane] = id;
    wu = (double)__int_as_float(mt.z) * (double)u;
    su = (double)u;
    viol = fmax(0.0, E - (double)e.y);
  }
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    wu += __shfl_down(wu, o);
    su += __shfl_down(su, o);
    viol += __shfl_down(viol, o);
  }
  const Decision dc{a, m, b, r, t, E, __uint_as_float((uint32_t)(best >> 32)), (float)wu};
  if (lane == 0) {
    if (r < w.log_cap) w.log[r] = dc;
    if (sg.log_host) sg.log_host[0] = dc;
    if (sg.ticks) sg.ticks[1] = wall_clock64();
    // (the host's copy is written alongside, not read back from this one)
    for (State* s : {st, w.st_host}) {
      s->last = dc;
      s->t = E;
      s->total_wu = twu + wu;
      s->total_u = tu + su;
      s->total_viol = tv + viol;
      s->round = r + 1;
      s->next_order = next_order + b;
      s->n_sched = next_order + b - 1;                   // (orders count from one)
      s->done = 0;                                       // (or this launch would have left at once)
      s->err = 0u;
    }
  }
  stores_arrived();
  __syncthreads();
  if (lane == 0) tell_host_ended(w);
}

}  // namespace sp
