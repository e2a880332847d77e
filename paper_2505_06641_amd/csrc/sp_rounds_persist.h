// All greedy rounds of a chunk in one launch (Alg. 1 generalised to batch-capped rounds; eq. (2),
// eq. (13), eq. (1) as in sp_rounds.h, which this kernel reproduces decision for decision).
//
// One workgroup per (application, variant) pair stays resident for the whole chunk; two more take the
// maximum over the pairs and do the commits.  What a round costs on the two-kernel path is mostly latency: two kernel
// boundaries, the walk over the service order and the gathers behind it.  Here
//   * each pair keeps its application's candidate window in LDS between rounds, with look-ahead entries
//     behind it (kWinCap in all).  A round removes the entries the previous decision consumed (always a
//     prefix: the greedy takes the first b live requests) and those whose penalty has reached 1 at the
//     new clock (they never come back: the clock only advances).  The walk over the service order that
//     refills the look-ahead runs one step per round while the candidates are being exchanged; a round
//     waits for it only when fewer than B entries remain while the application still has unvisited
//     requests.  Every position of the service order is visited once per launch, not once per round;
//   * between a decision and the candidates of the next round lies no barrier: every wavefront finds the live entries of the
//     window by itself, the list is put in order while the candidates are exchanged.  A round of 12 pairs takes 2.9 to
//     3.3 us (4.2 with the list put in order first and looping triangles), of 64 pairs 4.5 in the mean (5.1), of 512 pairs 7.1
//     to 8.2 (8.6 to 8.9); one that has to wait for the walk 3 to 4 more, which the means hold;
//   * the arg max over all pairs goes through one slot per pair and a reducing workgroup: every pair
//     publishes its best candidate, the reducer polls the slots (one per thread), takes the maximum and
//     publishes the decision, which one thread of every pair polls.  With few pairs (kAllToAllPairs) there
//     is no reducer: every pair's first wavefront polls all slots itself and takes the maximum, which halves the trips
//     through the fabric between a round's last candidate and its decision (the decisions are the same:
//     every pair applies the reducer's rule to the same words; pair 0 passes the decision on to the commit
//     workgroup).  Slots and the decision are pairs of
//     64-bit words, each carrying the generation number of the round it belongs to, written and polled
//     with relaxed device-scope atomics: a word is valid exactly when its generation matches, so no
//     fence is needed and a stale value can never be mistaken for the current one.  Both are double
//     buffered by generation parity (nobody can be more than one round ahead of anybody else: the
//     reducer needs every pair's slot of a round, every pair needs the reducer's decision of it);
//   * clock, round counter and window shifts follow from the decision and are replicated in every pair;
//   * the commit workgroup receives each decision through a ring entry, and the members of the chosen
//     batch through a ring of generation-tagged window positions written by the chosen application's
//     first pair, so the commits (outputs, totals, decision log) run beside the next round's scoring.
// With data-aware subgroups (Sec. 5.3.2) a pair serves every group of its application: the largest one
// (the "primary") keeps the LDS-resident window described above; the others take one wavefront each before
// the primary's block-wide work: groups of at most 64 requests are kept in LDS for the whole launch, larger ones are
// walked afresh every round; the pair publishes the best candidate over its groups together with the
// group's index.  The chosen batch's positions reach the commit workgroup after the decision: the chosen
// application's first pair writes them into the ring (from the primary's window, or from one more walk of
// the chosen secondary group, which every pair of that application does anyway to move its head pointer).
// The workgroups wait for each other, so all of them must be resident at once: the host launches this
// kernel only when the device can hold the whole grid (occupancy query), and every wait is bounded: a
// wait that runs out (the device was shared with other long-running work) raises kErrSync, every
// workgroup leaves its loop, and the call fails instead of hanging.
#pragma once
#include "sp_rounds.h"

namespace sp {

constexpr int kWinCap = 2 * kMaxBatch;          // window + look-ahead entries, one per thread
constexpr int kPersistRounds = 64;              // rounds per launch (ring depth)
constexpr int kSpinLimit = 1 << 20;             // polls before a wait is given up (about a second)
constexpr uint32_t kGenMask = 0x7FFFFFu;        // generation bits carried in a slot's first word
constexpr int kMaxPairs = 1024;                 // (application, variant) pairs the reducer can hold
constexpr int kSlotsPerThread = kMaxPairs / kRoundThreads;
// Requests per round of a window's first launch up to which the commit workgroup also fills the caller's outputs (one CU writes
// about 130 GB/s, beside rounds of 4 us and more that keep it busy for half of their time): a launch and its gap less per call.
constexpr int kOutputsPerRound = 1024;
constexpr int kMaxAppGroups = 64;               // groups of one application a resident pair can serve
constexpr int kAllToAllPairs = 2 * kWave;       // up to this many pairs, every pair polls every slot itself (two per lane)
static_assert(kWinCap <= kRoundThreads, "one window entry per thread");

struct Persist {
  const int32_t* pair_app;      // [n_pairs] application of each pair
  const int32_t* pair_model;    // [n_pairs] variant of each pair
  int32_t n_pairs;
  int32_t all_to_all;           // 1: every pair reads all pairs' slots and takes the maximum itself (no reducing workgroup)
  int32_t n_rounds;             // rounds this launch may run (<= kPersistRounds)
  int32_t spin_limit;           // polls before a wait between workgroups is given up (kSpinLimit unless a test shortens it)
  uint32_t gen_base;            // generations used by earlier launches
  unsigned long long* slots;    // [2 (parity), n_pairs, 4 (word)]
  unsigned long long* decision; // [2 (parity), 4 (word)]: latency bits << 32 | gen; (candidate id + 1, 0 = none)
                                //   << 32 | gen; swap-in cost bits << 32 | gen; unused
  unsigned long long* ring;     // [kPersistRounds, A, B]: generation << 32 | service position
  unsigned long long* dec;      // [kPersistRounds]: decision of each round, bit 63 set; zero once consumed
  Outputs out;                  // the caller's arrays, when this launch starts a window and fills them (else null)
  Decision* log_host;           // [kPersistRounds] pinned: the launch's decisions for the host
  int32_t* lost_host;           // pinned: set by any workgroup whose wait has run out
  long long* ticks;             // [kPersistRounds + 1]: constant-rate timestamps, launch start then each decision
  uint32_t* left;               // workgroups that have ended their work; zero between launches
};

__device__ __forceinline__ unsigned long long ld_dev(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// slot word 0: score bits << 32 | generation (23 bits) << 9 | valid << 8 | (b - 1)
// slot word 1: latency bits of the candidate (float) << 32 | group of the candidate (16 bits) << 16 | generation (16 bits)
//              (a slot is rewritten every round, so a stale word is two generations old: 16 bits tell)
// slot word 2: swap-in cost the pair would pay in this round (float bits) << 32 | generation (32 bits)
// slot word 3: group priority of the pair's application (eq. 14; float bits) << 32 | generation (32 bits)
__device__ __forceinline__ unsigned long long slot_word0(float score, uint32_t gen, bool valid, int b) {
  return ((unsigned long long)__float_as_uint(score) << 32) | ((unsigned long long)(gen & kGenMask) << 9) |
         (valid ? 0x100ull : 0ull) | (unsigned long long)((b - 1) & 0xff);
}

// Candidate ids inside this kernel: fields (group, variant, batch size - 1) instead of a product, which orders them the same way
// and needs no division to take apart on the way from one round to the next.
__device__ __forceinline__ uint32_t pcid(int grp, int m) { return ((uint32_t)grp << 12) | ((uint32_t)m << 8); }
__device__ __forceinline__ int pcid_group(uint32_t c) { return (int)(c >> 12); }
__device__ __forceinline__ int pcid_model(uint32_t c) { return (int)(c >> 8) & 15; }
__device__ __forceinline__ int pcid_batch(uint32_t c) { return (int)(c & 0xffu) + 1; }
static_assert(kMaxModels <= 16 && kMaxBatch <= 256, "fields of a candidate id (groups: at most 65,536)");

// A wait has run out.  The commit workgroup mirrors the state for the host when its own work ends, which may be before another
// workgroup gives up: each of them tells the host itself, past its die's L2 and before it counts itself among those that have left
// (persist_leave), so that the host finds it when it is told that all have ended.
__device__ __forceinline__ void raise_lost(State* st, const Persist& ps) {
  atomicOr(&st->err, kErrSync);
  __hip_atomic_store(ps.lost_host, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ void copy_output(int i, const Window& w, const Outputs& out) {
  if (out.model) out.model[i] = w.model[i];
  if (out.round_of) out.round_of[i] = w.round_of[i];
  if (out.order_of) out.order_of[i] = w.order_of[i];
  if (out.util) out.util[i] = w.util[i];
}

// The four per-request outputs into the caller's arrays, in a launch of its own: for long windows.
__global__ void k_copy_outputs(int n, Window w, Outputs out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) copy_output(i, w, out);
}

__device__ void persist_commit_loop(const Tables& tb, const Window& w, const Persist& ps, double (*dsum)[kMaxBatch],
                                    unsigned long long* bcast) {
  State* st = w.st;
  const int tid = threadIdx.x;
  // the caller's arrays as a window without rounds leaves them, before this workgroup's own commits go into both (it has
  // nothing to do until the first decision, and is ahead of the rounds after it)
  fill_output(ps.out.model, w.n, -1, tid, kRoundThreads);
  fill_output(ps.out.round_of, w.n, -1, tid, kRoundThreads);
  fill_output(ps.out.order_of, w.n, 0, tid, kRoundThreads);
  fill_output(reinterpret_cast<int32_t*>(ps.out.util), w.n, 0, tid, kRoundThreads);
  if (st->done || st->err) {
    if (tid == 0) mirror_state(w);
    return;
  }
  __syncthreads();
  int r = st->round, next_order = st->next_order, n_sched = st->n_sched;
  double t = st->t, twu = st->total_wu, tu = st->total_u, tv = st->total_viol;
  bool done = false, failed = false;
  Decision last = st->last;                 // app -1 before the window's first batch
  for (int rl = 0; rl < ps.n_rounds; ++rl) {
    const uint32_t gen = ps.gen_base + (uint32_t)rl + 1u;
    if (tid == 0) {
      unsigned long long v = 0ull;
      for (int i = 0; i < ps.spin_limit; ++i) {
        v = ld_dev(ps.dec + rl);
        if (v != 0ull) break;
        __builtin_amdgcn_s_sleep(4);
      }
      if (v != 0ull) st_dev(ps.dec + rl, 0ull);
      bcast[0] = v;
    }
    __syncthreads();
    const unsigned long long v = bcast[0];
    __syncthreads();
    if (v == 0ull) { failed = true; break; }
    const unsigned long long best = v & ~(1ull << 63);
    if (best == 0ull) { done = true; break; }
    const uint32_t cid = 0xFFFFFFFFu - (uint32_t)(best & 0xFFFFFFFFull);
    const float score = __uint_as_float((uint32_t)(best >> 32));
    const int B = tb.B;
    const int b = pcid_batch(cid), m = pcid_model(cid), grp = pcid_group(cid);
    const int a = group_app(tb, w, grp);              // group = application unless the requests are split into subgroups
    const double E = start_time(tb, last, t, a, m) + (double)tb.lat[((int64_t)a * tb.Mmax + m) * B + (b - 1)];
    const unsigned long long* row = ps.ring + ((size_t)rl * tb.A + a) * B;
    bool lost = false;
    double wu, su, viol;
    commit_members(tb, w, ps.out, a, m, b, r, next_order, E,
                   [&](int j) {
                     unsigned long long e = 0ull;
                     for (int i = 0; i < ps.spin_limit; ++i) {
                       e = ld_dev(row + j);
                       if ((uint32_t)(e >> 32) == gen) break;
                       __builtin_amdgcn_s_sleep(4);
                     }
                     if ((uint32_t)(e >> 32) != gen) { lost = true; return 0; }   // position 0 exists: b >= 1 request
                     return (int)(uint32_t)(e & 0xFFFFFFFFull);
                   },
                   nullptr, dsum, wu, su, viol);
    if (__syncthreads_or(lost ? 1 : 0)) { failed = true; break; }
    last.app = a; last.model = m; last.batch = b; last.round = r;
    last.t_start = t; last.t_end = E; last.score = score; last.batch_utility = (float)wu;
    if (tid == 0) {
      if (r < w.log_cap) w.log[r] = last;
      ps.log_host[rl] = last;
    }
    t = E; r += 1; next_order += b; n_sched += b;
    twu += wu; tu += su; tv += viol;
  }
  if (tid == 0) {
    // the host reads the pinned copy: nothing is copied behind the kernel.  It is written alongside, not read back from the other
    // one (a trip to memory at the end of every launch).
    for (State* s : {st, w.st_host}) {
      s->t = t; s->round = r; s->next_order = next_order; s->n_sched = n_sched;
      s->total_wu = twu; s->total_u = tu; s->total_viol = tv;
      s->last = last;
      s->done = done ? 1 : 0;
    }
    w.st_host->err = 0u;                    // (or this launch would have left at once)
    if (failed) raise_lost(st, ps);
  }
}

// The best of a set of candidates, with the latency and the swap-in cost that its pair has published.
struct Best {
  unsigned long long word;      // packed candidate, 0: none
  float lat, swap;
};
// Over a wavefront (candidate ids are unique, so one lane holds the maximum).
__device__ __forceinline__ Best wave_best(unsigned long long word, float lat, float swap) {
  Best b;
  b.word = wave_max_packed(word);
  const unsigned long long who = __ballot(word == b.word);
  const int lane = __builtin_amdgcn_readfirstlane(__ffsll((long long)who) - 1);
  b.lat = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lat), lane));
  b.swap = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(swap), lane));
  return b;
}

// The reducing workgroup: maximum over the pairs' slots of every round, published as the decision.
__device__ void persist_reduce_loop(const Tables& tb, const Window& w, const Persist& ps, unsigned long long* red,
                                    Best (*waves)[kRoundThreads / 64], int* timed_out) {
  const int tid = threadIdx.x;
  if (ps.all_to_all) return;                      // every pair takes the maximum itself
  const int my_slot = tid < ps.n_pairs ? tid : 0;
  const int my_m = ps.pair_model[my_slot];
  if (tid == 0) {
    *timed_out = 0;
    ps.ticks[0] = wall_clock64();
  }
  __syncthreads();
  for (int rl = 0; rl < ps.n_rounds; ++rl) {
    const uint32_t gen = ps.gen_base + (uint32_t)rl + 1u;
    unsigned long long mine = 0ull;
    float mine_lat = 0.f, mine_swap = 0.f;
    // with the group-first rule the slots are read once and compared twice: group priorities, then the
    // candidates of the winning application (a thread holds at most kSlotsPerThread slots)
    unsigned long long held[kSlotsPerThread];
    float held_lat[kSlotsPerThread], held_swap[kSlotsPerThread];
    unsigned long long top = 0ull;
#pragma unroll
    for (int q = 0; q < kSlotsPerThread; ++q) {
      held[q] = 0ull;
      const int i = tid + q * kRoundThreads;
      if (i >= ps.n_pairs) continue;
      const unsigned long long* slot = ps.slots + ((size_t)(gen & 1u) * ps.n_pairs + i) * 4;
      unsigned long long v0 = 0ull, v1 = 0ull, v2 = 0ull, v3 = 0ull;
      bool ok = false;
      for (int k = 0; k < ps.spin_limit; ++k) {
        v0 = ld_dev(slot);
        v1 = ld_dev(slot + 1);
        v2 = ld_dev(slot + 2);
        if (tb.pol_group_first) v3 = ld_dev(slot + 3);
        ok = ((uint32_t)(v0 >> 9) & kGenMask) == (gen & kGenMask) && (uint32_t)(v1 & 0xFFFFull) == (gen & 0xFFFFu) &&
             (uint32_t)(v2 & 0xFFFFFFFFull) == gen && (!tb.pol_group_first || (uint32_t)(v3 & 0xFFFFFFFFull) == gen);
        if (ok) break;
        __builtin_amdgcn_s_sleep(1);
      }
      if (!ok) {
        *timed_out = 1;
      } else if (v0 & 0x100ull) {
        const int pm = q == 0 ? my_m : ps.pair_model[i];
        const int pg = (int)((uint32_t)(v1 >> 16) & 0xFFFFu);      // the candidate's group (the pair's application when unsplit)
        const unsigned long long pk = pack_candidate(__uint_as_float((uint32_t)(v0 >> 32)), pcid(pg, pm) | (uint32_t)(v0 & 0xffull));
        held[q] = pk;
        held_lat[q] = __uint_as_float((uint32_t)(v1 >> 32));
        held_swap[q] = __uint_as_float((uint32_t)(v2 >> 32));
        const unsigned long long pt = ((unsigned long long)ordered_bits(__uint_as_float((uint32_t)(v3 >> 32))) << 32) |
                                      (unsigned long long)(0xFFFFFFFFu - (uint32_t)pg);
        top = pt > top ? pt : top;
      }
    }
    int a_star = -1;                                           // -1: every group competes
    if (tb.pol_group_first) {
      top = block_max_u64(top, red);
      if (top != 0ull) a_star = (int)(0xFFFFFFFFu - (uint32_t)(top & 0xFFFFFFFFull));
    }
#pragma unroll
    for (int q = 0; q < kSlotsPerThread; ++q) {
      if (held[q] == 0ull) continue;
      const uint32_t cid = 0xFFFFFFFFu - (uint32_t)(held[q] & 0xFFFFFFFFull);
      if (a_star >= 0 && pcid_group(cid) != a_star) continue;
      if (held[q] > mine) { mine = held[q]; mine_lat = held_lat[q]; mine_swap = held_swap[q]; }
    }
    // the wavefronts' maxima with what belongs to them, then one barrier; the array alternates between rounds
    {
      const Best b = wave_best(mine, mine_lat, mine_swap);
      if ((tid & 63) == 0) waves[rl & 1][tid >> 6] = b;
    }
    __syncthreads();
    if (*timed_out) {
      if (tid == 0) raise_lost(w.st, ps);
      break;
    }
    const Best of = waves[rl & 1][tid & (kRoundThreads / 64 - 1)];
    const Best top1 = wave_best(of.word, of.lat, of.swap);
    const unsigned long long all = top1.word;
    if (tid < 3) {                                             // three words side by side
      const uint32_t cidp1 = all != 0ull ? (0xFFFFFFFFu - (uint32_t)(all & 0xFFFFFFFFull)) + 1u : 0u;
      const uint32_t word = tid == 1 ? cidp1 : all == 0ull ? 0u : __float_as_uint(tid == 0 ? top1.lat : top1.swap);
      st_dev(ps.decision + (size_t)(gen & 1u) * 4 + tid, ((unsigned long long)word << 32) | (unsigned long long)gen);
    }
    if (tid == 0) {
      st_dev(ps.dec + rl, all | (1ull << 63));
      ps.ticks[rl + 1] = wall_clock64();
    }
    if (all == 0ull) break;                                    // nothing live anywhere
  }
}

// The first (up to) Bw live requests of a group from position `head` on, found by one wavefront: their
// service positions go to wpos (LDS of that wavefront), the count is returned.  Same rule as the walks of
// the other round kernels: pending, and the penalty on the earliest possible completion E0 below 1.
__device__ __forceinline__ int wave_window(const Window& w, int kind, int head, int seg_e, double E0, int Bw,
                                           int32_t* wpos, int lane) {
  int found = 0;
  for (int base = head & ~3; base < seg_e && found < Bw; base += 4 * kWave) {
    const int p0 = base + 4 * lane;
    const uint32_t mask = live_mask<1>(w, kind, E0, p0, head, seg_e);
    const int cnt = __popc(mask);
    const int incl = (int)wave_scan_incl((uint32_t)cnt);
    int rank = found + incl - cnt;
    uint32_t mk = mask;
    while (mk != 0 && rank < Bw) {
      const int j = __ffs((int)mk) - 1;
      mk &= mk - 1;
      wpos[rank++] = p0 + j;
    }
    found += __shfl(incl, kWave - 1);
  }
  wave_sync();
  return min(found, Bw);
}

// A workgroup's work has ended: the last one of the grid tells the host.  The commit workgroup alone writes through its L2, which it
// writes back first; what the others leave (raise_lost, first live positions) is written past it.
__device__ __forceinline__ void persist_leave(const Window& w, const Persist& ps, bool committed = false) {
  if (w.ended_host == nullptr) return;
  stores_arrived();
  __syncthreads();
  if (threadIdx.x != 0) return;
  if (committed) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
  if (atomicAdd(ps.left, 1u) + 1u != gridDim.x) return;
  __hip_atomic_store(ps.left, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  tell_host_ended(w);
}

// Requests of small secondary groups that a resident pair keeps in LDS (512: ten KB beside the windows, so that three
// workgroups still share a CU at batch sizes up to 128).
constexpr int kCachedRequests = 512;

// SPLIT: the window's groups are subgroups of the applications (tb.pol_split); the plain instantiation holds
// none of the secondary-group code.
// WGS: workgroups that must fit on a compute unit.  Three leave 80 registers (3 spilled with the looping triangles, 27 with
// subgroups); grids of up to one workgroup per compute unit (254 pairs on 256) get 128 (none, 3), and triangles with their entries
// held.
template <bool SPLIT, int WGS>
__global__ __launch_bounds__(kRoundThreads, 2 * WGS) void k_rounds_persistent(Tables tb, Window w, Persist ps) {
  __shared__ int32_t win[kWinCap];
  __shared__ float4 ent[kWinCap];
  __shared__ float om[kWinCap];              // ordering value of each entry (for the group priority)
  __shared__ float lat_s[kMaxBatch];
  __shared__ int32_t wave_cnt[kRoundThreads / 64], keep_cnt[kRoundThreads / 64];
  __shared__ unsigned long long red[kRoundThreads / 64];
  __shared__ unsigned long long cand_max[2][kRoundThreads / 64];   // a round's candidates per wavefront (alternating)
  __shared__ Best waves[2][kRoundThreads / 64];
  // this round's window without the entries that have died (every wavefront writes all of it), or the commit workgroup's sums
  __shared__ union { struct { float4 ent[kMaxBatch]; float om[kMaxBatch]; } now; double dsum[3][kMaxBatch]; } own;
  float4* const cent = own.now.ent;
  float* const com = own.now.om;
  __shared__ struct { uint32_t cid; float lat, swap; } decided[2];   // a round's decision (alternating)
  __shared__ int timed_out;
  __shared__ int32_t slot_model[kAllToAllPairs];                // variants behind the slots
  __shared__ int32_t head_s[kMaxAppGroups];                     // head pointer of each group of the application
  __shared__ unsigned long long sec_best[kRoundThreads / 64], sec_top[kRoundThreads / 64];   // per wavefront: its secondary groups' best
  __shared__ float sec_prio[kRoundThreads / 64];
  // secondary groups of at most one request per lane, as far as they fit: read once, so that a round looks at them without
  // a trip to memory (most subgroups are that small; a walk and its gathers are three trips for each)
  __shared__ int32_t end_s[SPLIT ? kMaxAppGroups : 1], cache_at[SPLIT ? kMaxAppGroups : 1];   // first cached entry, or -1
  __shared__ float4 cache_ent[SPLIT ? kCachedRequests : 1];
  __shared__ int32_t cache_pos[SPLIT ? kCachedRequests : 1];    // service position, or -1: not pending
  extern __shared__ __align__(16) unsigned char sec_lds[];      // with subgroups: per wavefront B window entries and B positions
  State* st = w.st;
  // more groups than a pair serves: the window is left as it is, and the host, which has not waited for their number, sees
  // no round done and takes two kernels per round
  if (SPLIT && w.grp_n[1] > kMaxAppGroups) {
    if ((int)blockIdx.x == ps.n_pairs + 1 && threadIdx.x == 0) mirror_state(w);
    persist_leave(w, ps, true);
    return;
  }
  if ((int)blockIdx.x == ps.n_pairs + 1) {
    persist_commit_loop(tb, w, ps, own.dsum, red);
    persist_leave(w, ps, true);
    return;
  }
  if (st->done || st->err) {                // the state is rewritten only when the commit workgroup ends
    persist_leave(w, ps);
    return;
  }
  if ((int)blockIdx.x == ps.n_pairs) {
    persist_reduce_loop(tb, w, ps, red, waves, &timed_out);
    persist_leave(w, ps);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int pair = blockIdx.x;
  const int a = ps.pair_app[pair], m = ps.pair_model[pair];
  const int B = tb.B, Bw = tb.Bcap, cap = kWinCap;   // B: row stride of the tables; Bw: largest batch
  const int kind = tb.penalty[a];
  const float lmin = tb.lmin[a];
  const float my_swap = tb.swap[a * tb.Mmax + m];
  bool prev_mine = st->last.app == a;                       // the previous batch ran a variant of this application ...
  int prev_m = st->last.model;                              // ... namely this one (-1 before the window's first batch)
  int r = st->round;
  double t = st->t;
  // the groups of this application: itself, or (Sec. 5.3.2) its non-empty subgroups, consecutive in the group table
  int glo = a, ng = 1;
  if (SPLIT) {
    const int G = w.grp_n[0];
    int lo = 0, hi = G;
    while (lo < hi) {                                        // first group of an application >= a
      const int mid = (lo + hi) >> 1;
      if (w.grp_app[mid] < a) lo = mid + 1; else hi = mid;
    }
    glo = lo;
    hi = G;
    while (lo < hi) {                                        // first group of an application > a
      const int mid = (lo + hi) >> 1;
      if (w.grp_app[mid] <= a) lo = mid + 1; else hi = mid;
    }
    ng = lo - glo;
  }
  // the primary group (largest remaining range; ties: the first) keeps the LDS-resident window
  int prim = 0, prim_size = -1;
  for (int i = 0; i < ng; ++i) {
    const int sz = w.grp_end[glo + i] - w.head[(r & 1) * w.gcap + glo + i];
    if (sz > prim_size) { prim_size = sz; prim = i; }
  }
  for (int i = tid; i < ng; i += kRoundThreads) {
    head_s[i] = w.head[(r & 1) * w.gcap + glo + i];
    if (SPLIT) end_s[i] = w.grp_end[glo + i];
  }
  const int gprim = glo + prim;
  const int seg_e = ng > 0 ? w.grp_end[gprim] : 0;
  int scan_end = ng > 0 ? w.head[(r & 1) * w.gcap + gprim] : 0;   // everything before it is consumed or dead
  int nb = 0, shift = 0;
  unsigned long long evals = 0ull;               // utility evaluations counted by this thread (lane 0 of a wavefront)
  for (int j = tid; j < B; j += kRoundThreads) lat_s[j] = tb.lat[((int64_t)a * tb.Mmax + m) * B + j];
  if (tid == 0) {
    timed_out = 0;
    if (ps.all_to_all && pair == 0) ps.ticks[0] = wall_clock64();
  }
  if (ps.all_to_all && tid < ps.n_pairs) slot_model[tid] = ps.pair_model[tid];
  float4* went = reinterpret_cast<float4*>(sec_lds) + (size_t)wave * B;
  int32_t* wpos = reinterpret_cast<int32_t*>(sec_lds + (size_t)(kRoundThreads / 64) * B * sizeof(float4)) + (size_t)wave * B;
  __syncthreads();
  if (SPLIT && ng > 1) {
    if (tid == 0) {
      int used = 0;
      for (int i = 0; i < ng; ++i) {
        const int sz = end_s[i] - head_s[i];
        const bool fits = i != prim && sz > 0 && sz <= kWave && used + sz <= kCachedRequests;
        cache_at[i] = fits ? used : -1;
        used += fits ? sz : 0;
      }
    }
    __syncthreads();
    for (int i = wave; i < ng; i += kRoundThreads / 64) {
      const int at = cache_at[i], pos = head_s[i] + lane;
      if (at < 0 || pos >= end_s[i]) continue;
      const bool pending = w.alive_s[pos] != 0;
      cache_pos[at + lane] = pending ? pos : -1;
      cache_ent[at + lane] = window_entry(tb, w, pos, m);
    }
    __syncthreads();
  }

  for (int rl = 0; rl < ps.n_rounds; ++rl) {
    const uint32_t gen = ps.gen_base + (uint32_t)rl + 1u;
    const double E0 = t + (double)lmin;
    const float swap_now = (prev_mine && prev_m == m) ? 0.f : my_swap;

    // ---- secondary groups: one wavefront each, walked afresh from their head pointers ----
    unsigned long long wbest = 0ull, wtop = 0ull;
    float wprio = 0.f;
    if (SPLIT && ng > 1) {
      for (int i = wave; i < ng; i += kRoundThreads / 64) {
        if (i == prim) continue;
        const int g = glo + i, se = end_s[i], at = cache_at[i];
        int nbs;
        if (at >= 0) {
          const bool has = lane < se - head_s[i];
          const int pos = has ? cache_pos[at + lane] : -1;
          const float4 e = cache_ent[has ? at + lane : at];
          const bool live = pos >= 0 && !is_dead(kind, e.y, E0);
          const unsigned long long m_live = __ballot(live);
          const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m_live >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m_live, 0u));
          nbs = min(__popcll(m_live), Bw);
          if (nbs == 0) continue;
          if (live && rank < Bw) { wpos[rank] = pos; went[rank] = e; }
        } else {
          nbs = wave_window(w, kind, head_s[i], se, E0, Bw, wpos, lane);
          if (lane == 0) head_s[i] = nbs > 0 ? wpos[0] : se;     // what lies before has been consumed or has died
          if (nbs == 0) continue;
          for (int j = lane; j < nbs; j += kWave) went[j] = window_entry(tb, w, wpos[j], m);
        }
        wave_sync();
        if (lane == 0) evals += triangle_evals(nbs, tb.pol_whole);
        const int only_b = tb.pol_whole ? nbs : 0;
        unsigned long long cand = nbs <= 16 && pair_lanes(Bw) == 16
            ? triangle_few(scoring_penalty(tb, kind), went, lat_s, nbs, t + (double)swap_now, pcid(g, m), only_b, lane)
            : triangle_best(scoring_penalty(tb, kind), went, lat_s, nbs, Bw, t + (double)swap_now, pcid(g, m), nullptr, only_b, kWave, lane);
        cand = wave_max_packed(cand);
        if (tb.pol_group_first) {
          // eq. (14) over the window: the fixed-order sum a single wavefront forms in k_round_score
          double part = 0.0;
          for (int j = lane; j < nbs; j += kWave) part += (double)ordering_value(tb, w, wpos[j]);
#pragma unroll
          for (int o = kWave / 2; o > 0; o >>= 1) part += __shfl_down(part, o);
          const float pr = (float)(__shfl(part, 0) / (double)nbs);
          const unsigned long long top = ((unsigned long long)ordered_bits(pr) << 32) | (unsigned long long)(0xFFFFFFFFu - (uint32_t)g);
          if (cand != 0ull && top > wtop) { wtop = top; wbest = cand; wprio = pr; }
        } else if (cand > wbest) {
          wbest = cand;
        }
        wave_sync();                                              // wpos and went are reused by the next group
      }
    }

    // The primary group's list without what the last decision consumed and what has died.  The whole workgroup.
    auto drop = [&] {
      const bool has = tid < nb;
      int pos = 0;
      float4 e = make_float4(0.f, 1.f, 0.f, 0.f);
      float ov = 0.f;
      if (has) { pos = win[tid]; e = ent[tid]; ov = om[tid]; }
      const bool keep = has && tid >= shift && !is_dead(kind, e.y, E0);
      const unsigned long long bal = __ballot(keep);
      if (lane == 0) keep_cnt[wave] = __popcll(bal);
      __syncthreads();
      int before = 0, total = 0;
      for (int i = 0; i < kRoundThreads / 64; ++i) {
        const int c = keep_cnt[i];
        if (i < wave) before += c;
        total += c;
      }
      if (total != nb) {
        before += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
        if (keep) { win[before] = pos; ent[before] = e; om[before] = ov; }
        nb = total;
        __syncthreads();
      }
      shift = 0;
    };

    // Walks on through the service order from scan_end and appends the live requests it meets, for at
    // most max_steps steps of 4 * nq positions per thread, until the list holds `enough` or the group's
    // range ends.  Uniform over the workgroup.
    auto walk = [&](int max_steps, int first_nq, int enough) {
      const int nb_old = nb;
      for (int step = 0; step < max_steps && nb < enough && scan_end < seg_e; ++step) {
        const int nq = step == 0 ? first_nq : 4;           // groups of 4 positions per thread
        const int base = scan_end & ~3;
        const int p0 = base + 4 * nq * tid;
        const uint32_t mask = nq == 1 ? live_mask<1>(w, kind, E0, p0, scan_end, seg_e) : live_mask<4>(w, kind, E0, p0, scan_end, seg_e);
        const int cnt = __popc(mask);
        const int incl = (int)wave_scan_incl((uint32_t)cnt);
        if (lane == 63) wave_cnt[wave] = incl;
        __syncthreads();
        int before = nb, total = nb;
        for (int i = 0; i < kRoundThreads / 64; ++i) {
          if (i < wave) before += wave_cnt[i];
          total += wave_cnt[i];
        }
        int rank = before + incl - cnt;
        uint32_t mk = mask;
        while (mk != 0 && rank < cap) {
          const int j = __ffs((int)mk) - 1;
          mk &= mk - 1;
          win[rank++] = p0 + j;
        }
        __syncthreads();
        if (total >= cap) {
          scan_end = win[cap - 1] + 1;                     // the rest of this step is looked at again later
          nb = cap;
        } else {
          scan_end = min(base + 4 * nq * kRoundThreads, seg_e);
          nb = total;
        }
      }
      for (int j = nb_old + tid; j < nb; j += kRoundThreads) {
        ent[j] = window_entry(tb, w, win[j], m);
        om[j] = ordering_value(tb, w, win[j]);
      }
      __syncthreads();
    };

    // ---- the round's window: the first Bw live entries of the list, from its first few chunks of 64 (those that hold Bw
    // entries and sixteen more).  Every wavefront finds and writes all of them, the same values to the same places: it then
    // reads what it has written itself, and no barrier is needed.  The list itself is put in order while candidates are exchanged. ----
    bool in_order = false;
    int nbe = 0;
    {
      const int look = min(nb, shift + (Bw + 16 + kWave - 1) / kWave * kWave);
      for (int j0 = shift; j0 < look; j0 += kWave) {
        const int j = j0 + lane;
        const float4 e = ent[min(j, kWinCap - 1)];
        const bool live = j < nb && !is_dead(kind, e.y, E0);
        const unsigned long long bal = __ballot(live);
        const int rank = nbe + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
        if (live && rank < Bw) {
          cent[rank] = e;
          if (tb.pol_group_first) com[rank] = om[j];
        }
        nbe += __popcll(bal);
      }
      if (nbe < Bw && (look < nb || scan_end < seg_e)) {           // (uniform) not enough there: the round has to wait for the rest
        in_order = true;
        drop();
        if (nb < Bw && scan_end < seg_e) walk(1 << 30, rl == 0 ? 1 : 4, Bw);       // (most requests are live at a window's start)
        nbe = nb;
        for (int j = lane; j < min(nb, Bw); j += kWave) {
          cent[j] = ent[j];
          if (tb.pol_group_first) com[j] = om[j];
        }
      }
      nbe = min(nbe, Bw);
      wave_sync();
    }

    // ---- triangle: the sums of k_round_score ----
    unsigned long long best = 0ull;
    if (tid == 0) evals += triangle_evals(nbe, tb.pol_whole);
    if (nbe > 0) {
      if (WGS == 2 && pair_lanes(Bw) == 16)
        best = triangle_held(scoring_penalty(tb, kind), cent, lat_s, nbe, Bw, t + (double)swap_now, pcid(gprim, m), tb.pol_whole ? nbe : 0, tid);
      else
        best = triangle_best(scoring_penalty(tb, kind), cent, lat_s, nbe, Bw, t + (double)swap_now, pcid(gprim, m), nullptr, tb.pol_whole ? nbe : 0);
    }
    float prio = 0.f;
    if (tb.pol_group_first && wave == 0) {   // eq. (14) over the window, in the order of block_sum_f64
      double v[kMaxBatch / kWave];
#pragma unroll
      for (int q = 0; q < kMaxBatch / kWave; ++q) v[q] = q * kWave + lane < nbe ? (double)com[q * kWave + lane] : 0.0;
      double sum = (v[0] + v[2]) + (v[1] + v[3]);
#pragma unroll
      for (int o = kWave / 2; o > 0; o >>= 1) sum += __shfl_down(sum, o);
      prio = nbe > 0 ? (float)(__shfl(sum, 0) / (double)nbe) : 0.f;
    }
    if (SPLIT && ng > 1 && lane == 0) {
      sec_best[wave] = wbest;
      sec_top[wave] = wtop;
      sec_prio[wave] = wprio;
    }
    best = wave_max_packed(best);
    if (lane == 0) cand_max[rl & 1][wave] = best;
    __syncthreads();                     // (also makes the wavefronts' secondary results visible)

    // ---- publish this pair's best candidate over its groups: four lanes, a word each ----
    if (wave == 0) {
      constexpr int kW = kRoundThreads / 64;
      best = wave_max_packed(lane < kW ? cand_max[rl & 1][lane] : 0ull);
      if (SPLIT && ng > 1) {
        const unsigned long long sec = lane < kW ? sec_best[lane] : 0ull;
        if (tb.pol_group_first) {
          // first the group with the highest priority among those that have a candidate, then its candidate
          unsigned long long top = sec != 0ull ? sec_top[lane] : 0ull;
          if (lane == kW && best != 0ull) top = ((unsigned long long)ordered_bits(prio) << 32) | (unsigned long long)(0xFFFFFFFFu - (uint32_t)gprim);
          const unsigned long long cand = lane == kW ? best : sec;
          const float pr = lane < kW ? sec_prio[lane] : prio;
          const unsigned long long ftop = wave_max_u64(top);
          const int who = __builtin_amdgcn_readfirstlane(__ffsll((long long)__ballot(top == ftop)) - 1);
          best = ftop != 0ull ? (unsigned long long)__shfl((long long)cand, who) : 0ull;
          prio = ftop != 0ull ? __shfl(pr, who) : prio;
        } else {
          best = wave_max_packed(sec > best ? sec : best);
        }
      }
      const bool valid = best != 0ull;
      const uint32_t bcid = 0xFFFFFFFFu - (uint32_t)best;
      const int b = valid ? pcid_batch(bcid) : 1;
      const uint32_t bg = valid ? (uint32_t)pcid_group(bcid) : (uint32_t)a;
      const unsigned long long w0 = slot_word0(__uint_as_float((uint32_t)(best >> 32)), gen, valid, b);
      const unsigned long long w1 = ((unsigned long long)__float_as_uint(lat_s[b - 1]) << 32) | ((unsigned long long)(bg & 0xFFFFu) << 16) |
                                    (unsigned long long)(gen & 0xFFFFu);
      const unsigned long long w23 = ((unsigned long long)__float_as_uint(lane == 2 ? swap_now : prio) << 32) | (unsigned long long)gen;
      if (lane < 4) st_dev(ps.slots + ((size_t)(gen & 1u) * ps.n_pairs + pair) * 4 + lane, lane == 0 ? w0 : lane == 1 ? w1 : w23);
    }

    // ---- while the candidates are exchanged: the list in order, the window's positions for the commit workgroup (with
    // subgroups after the decision), and one step of the walk once less than two windows are left ----
    if (!in_order) drop();
    if (!SPLIT && m == 0 && tid < nbe)
      st_dev(ps.ring + ((size_t)rl * tb.A + a) * B + tid, ((unsigned long long)gen << 32) | (unsigned long long)(uint32_t)win[tid]);
    if (nb < min(2 * Bw, cap) && scan_end < seg_e) walk(1, 4, cap);

    // ---- few pairs: the first wavefront takes the maximum over all pairs' slots (the reducer's rule on the same words), two
    // slots per lane, and passes it on behind one barrier; else its first lane waits for the reducer's decision ----
    if (wave == 0) {
      if (ps.all_to_all) {
        unsigned long long mine = 0ull, top = 0ull;
        float mine_lat = 0.f, mine_swap = 0.f;
        unsigned long long held[2] = {0ull, 0ull};
        float held_lat[2] = {0.f, 0.f}, held_swap[2] = {0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          int i = lane + q * kWave;
          asm volatile("" : "+v"(i));                            // (addresses formed here, not held from one round to the next)
          if (i >= ps.n_pairs) continue;
          const unsigned long long* slot = ps.slots + ((size_t)(gen & 1u) * ps.n_pairs + i) * 4;
          unsigned long long v0 = 0ull, v1 = 0ull, v2 = 0ull, v3 = 0ull;
          bool ok = false;
          for (int k = 0; k < ps.spin_limit; ++k) {
            v0 = ld_dev(slot);
            v1 = ld_dev(slot + 1);
            v2 = ld_dev(slot + 2);
            if (tb.pol_group_first) v3 = ld_dev(slot + 3);
            ok = ((uint32_t)(v0 >> 9) & kGenMask) == (gen & kGenMask) && (uint32_t)(v1 & 0xFFFFull) == (gen & 0xFFFFu) &&
                 (uint32_t)(v2 & 0xFFFFFFFFull) == gen && (!tb.pol_group_first || (uint32_t)(v3 & 0xFFFFFFFFull) == gen);
            if (ok) break;
            __builtin_amdgcn_s_sleep(1);
          }
          if (!ok) {
            timed_out = 1;
          } else if (v0 & 0x100ull) {
            const int pg = (int)((uint32_t)(v1 >> 16) & 0xFFFFu);
            held[q] = pack_candidate(__uint_as_float((uint32_t)(v0 >> 32)), pcid(pg, slot_model[i]) | (uint32_t)(v0 & 0xffull));
            held_lat[q] = __uint_as_float((uint32_t)(v1 >> 32));
            held_swap[q] = __uint_as_float((uint32_t)(v2 >> 32));
            const unsigned long long pt = ((unsigned long long)ordered_bits(__uint_as_float((uint32_t)(v3 >> 32))) << 32) |
                                          (unsigned long long)(0xFFFFFFFFu - (uint32_t)pg);
            top = pt > top ? pt : top;
          }
        }
        int g_star = -1;                                         // -1: every group competes
        if (tb.pol_group_first) {
          top = wave_max_u64(top);
          if (top != 0ull) g_star = (int)(0xFFFFFFFFu - (uint32_t)(top & 0xFFFFFFFFull));
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const uint32_t c2 = 0xFFFFFFFFu - (uint32_t)(held[q] & 0xFFFFFFFFull);
          if (held[q] == 0ull || (g_star >= 0 && pcid_group(c2) != g_star)) continue;
          if (held[q] > mine) { mine = held[q]; mine_lat = held_lat[q]; mine_swap = held_swap[q]; }
        }
        const Best all = wave_best(mine, mine_lat, mine_swap);
        if (lane == 0) {
          decided[rl & 1].cid = all.word != 0ull ? (0xFFFFFFFFu - (uint32_t)(all.word & 0xFFFFFFFFull)) + 1u : 0u;
          decided[rl & 1].lat = all.lat;
          decided[rl & 1].swap = all.swap;
          if (pair == 0) {                                       // for the commit workgroup, and the round's timestamp
            st_dev(ps.dec + rl, all.word | (1ull << 63));
            ps.ticks[rl + 1] = wall_clock64();
          }
        }
      } else if (lane == 0) {
        const unsigned long long* d = ps.decision + (size_t)(gen & 1u) * 4;
        unsigned long long v0 = 0ull, v1 = 0ull, v2 = 0ull;
        bool ok = false;
        for (int k = 0; k < ps.spin_limit; ++k) {
          v0 = ld_dev(d);
          v1 = ld_dev(d + 1);
          v2 = ld_dev(d + 2);
          ok = (uint32_t)(v0 & 0xFFFFFFFFull) == gen && (uint32_t)(v1 & 0xFFFFFFFFull) == gen &&
               (uint32_t)(v2 & 0xFFFFFFFFull) == gen;
          if (ok) break;
          __builtin_amdgcn_s_sleep(1);
        }
        if (!ok) timed_out = 1;
        decided[rl & 1].lat = __uint_as_float((uint32_t)(v0 >> 32));
        decided[rl & 1].cid = (uint32_t)(v1 >> 32);
        decided[rl & 1].swap = __uint_as_float((uint32_t)(v2 >> 32));
      }
    }
    __syncthreads();
    if (timed_out) {
      if (tid == 0) raise_lost(st, ps);
      break;
    }
    const uint32_t cidp1 = decided[rl & 1].cid;                // (written again two rounds from here)
    const float lat_sel = decided[rl & 1].lat, swap_sel = decided[rl & 1].swap;
    if (cidp1 == 0u) break;                                  // nothing live anywhere
    const uint32_t cid = cidp1 - 1u;
    const int bsel = pcid_batch(cid), gsel = pcid_group(cid), msel = pcid_model(cid);
    const bool mine = gsel >= glo && gsel < glo + ng;        // a group of this application
    if (mine && gsel == gprim) {
      shift = bsel;
      if (SPLIT && m == 0 && tid < bsel)
        st_dev(ps.ring + ((size_t)rl * tb.A + a) * B + tid, ((unsigned long long)gen << 32) | (unsigned long long)(uint32_t)win[tid]);
    } else if (SPLIT && mine) {
      // a secondary group was chosen: its window once more (same clock, nothing of it has changed since it was
      // scored), to move the head pointer past the batch and to hand the batch's positions to the commit workgroup
      const int isel = gsel - glo;
      const int at = cache_at[isel];
      if (wave == 0 && at >= 0) {
        const bool has = lane < end_s[isel] - head_s[isel];
        const int pos = has ? cache_pos[at + lane] : -1;
        const bool live = pos >= 0 && !is_dead(kind, cache_ent[has ? at + lane : at].y, E0);
        const unsigned long long m_live = __ballot(live);
        const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m_live >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m_live, 0u));
        if (live && rank < bsel) {
          if (m == 0) st_dev(ps.ring + ((size_t)rl * tb.A + a) * B + rank, ((unsigned long long)gen << 32) | (unsigned long long)(uint32_t)pos);
          cache_pos[at + lane] = -1;
        }
      } else if (wave == 0) {
        const int nbs = wave_window(w, kind, head_s[isel], w.grp_end[gsel], E0, Bw, wpos, lane);
        if (m == 0)
          for (int j = lane; j < bsel && j < nbs; j += kWave)
            st_dev(ps.ring + ((size_t)rl * tb.A + a) * B + j, ((unsigned long long)gen << 32) | (unsigned long long)(uint32_t)wpos[j]);
        const int last = bsel <= nbs ? wpos[bsel - 1] : w.grp_end[gsel] - 1;
        wave_sync();
        if (lane == 0) head_s[isel] = last + 1;
      }
      __syncthreads();
    }
    t = (t + (double)swap_sel) + (double)lat_sel;
    prev_mine = mine;
    prev_m = msel;
    r += 1;
  }
  {
    unsigned long long ev = evals;                           // lanes 0 of the wavefronts hold the counts
    if (lane == 0 && ev != 0ull) atomicAdd(&st->n_evals, ev);
  }
  // first position of every group of this application that may still be live, for whoever continues the window
  __syncthreads();
  if (m == 0)
    for (int i = tid; i < ng; i += kRoundThreads)            // (past this die's L2: another workgroup tells the host that all have ended)
      __hip_atomic_store(w.head + (r & 1) * w.gcap + glo + i, i == prim ? (shift < nb ? win[shift] : scan_end) : head_s[i], __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  persist_leave(w, ps);
}

__global__ void k_fill_u64(unsigned long long* p, int64_t n, unsigned long long v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

}  // namespace sp
