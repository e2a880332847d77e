// Scoring kernel on the matrix cores for the heads that the two kernels with a fixed input width do not take:
// logistic heads on bfloat16 features or on float32 features wider than 256, and one-hidden-layer heads (H <= 256)
// on float32 features or on bfloat16 features that those kernels pad too much (Def. 4.1.1, 4.1.2; Sec. 4.1 eq. (9);
// Sec. 5.1.1 eq. (12)).
//
// A wavefront owns 32 requests and keeps the whole transposed output tile of the first layer (32 NB rows: hidden
// units, or classes) in NB float32 accumulators while it streams its requests' features from memory, kStBytes per
// row and step; the matching weight slices, packed at context creation in the order the lanes read them, go through
// two LDS buffers shared by the workgroup's four wavefronts.  The order of a slice's channels is free as long as the weights
// are packed in the same one, so a lane takes 64 consecutive bytes of its request's row: straight from memory, or (stream_turns)
// out of LDS.  A step costs memory more than matrix cores in all of these shapes, so features travel two steps ahead.
//
// bfloat16: products are exact, float32 accumulation.  float32: every operand is scaled by a power of two and split
// into two half-precision numbers as in the logistic kernel (x.w = hi.hi + lo.hi + hi.lo), and so are the hidden activations
// and the second layer of either type; inputs of very different ranges are brought together first (equalizing_exponents).  A row's largest value is
// not known before the row has been read, so the scale follows a running maximum: when a step brings a larger value,
// the request's accumulators are rescaled by the exact power of two.
//
// Partial sums of a step are added to the accumulators in float32 registers, and the exponentials are split on a fixed grid:
// the matrix cores cut off the bits of a term that lie far below the largest one of an instruction, which in a chain of
// hundreds of them shows as a bias of 5e-8.
//
// Logistic heads then take the softmax and the table contraction straight from the accumulators; more than 32 NB
// classes go in groups, each of which streams the rows again.  One-hidden-layer heads add bias, ReLU and split in
// registers and walk the class tiles like the bfloat16 kernel; class blocks follow the slices through the same two
// buffers.
//
// Measured (rocprofv3, median us): 32,768 rows of 768 floats, 100 classes 32.9 (3.1 TB/s of rows; 38.1 without the second team, 1543 in the
// generic kernel); 65,536 rows of 512 bfloat16, 100 classes 24.5 (2.7 TB/s); 100,000 requests of 128-64-10/7/2 float32 heads 25.5
// (2.0 TB/s); 30,011 of 384-128-100/37/10 bfloat16 heads 17.4 (1.3 TB/s; 19.9 with rows read as they lie).  A large copy reaches 5.2 TB/s on
// this card (read and written).
#pragma once
#include "sp_common.h"
#include "sp_score_split.h"
#include "sp_score_mlp.h"

namespace sp {

// Wavefronts per workgroup: four, so that two or three workgroups share a CU and one's loads run beside another's
// matrix work; eight where the accumulators leave two wavefronts per SIMD anyway (fewer units of a stage per thread).
constexpr int stream_waves(int nb) { return nb == 8 ? 8 : 4; }
constexpr int stream_tile(int nb) { return stream_waves(nb) * 32; }    // requests per workgroup
// Logistic heads on up to 256 float32 features come here while no application has more classes than this: the scoring
// kernel then takes 10-30% less time than the one that keeps a request's features in registers and walks the classes
// (200,000 requests of 10 classes: 52 us against 65 with 256 features, 22 against 30 with 32; of 100 classes: 81 against
// 93).  From 129 classes on it would hold eight blocks of rows and lose (130 classes: 110 us against 103, 52 against 50).
constexpr int kStreamClasses = 128;
constexpr int kStBytes = 128;                    // bytes of a feature row per step (one cache line)

// Slices of a row from which two teams of wavefronts share a tile's rows (KS == 2), each with every other slice: a workgroup is alone on
// its compute unit while a window has no more tiles than there are units, and then waits at every step for the weights' and the rows'
// way from memory, with one wavefront per SIMD.  The teams' sums meet in LDS, each team takes half of the classes from there on.  Logistic
// heads; weights travel two steps ahead.  us per call, one team / two, no row turned: 100 classes, 32,768 rows of 768 floats 50.0 / 47.0, of 1024
// 57.8 / 53.3, 1,000 rows 39.6 / 36.0; 10 classes 47.8 / 40.9; 512 bfloat16 (8 slices) 35.0 / 34.0; 8 slices of floats 31.0 / 29.4, 4 slices
// 25.8 / 26.1; with more tiles than units (33,000 to 50,000 rows) no difference, and one team shares the unit with other workgroups.
constexpr int kTeamSlices = 6;
// Whether rows are read in whole lines and turned in LDS.  Without that an instruction of a wavefront touches 64 lines for 16 bytes each, 256
// cycles of address processing per step and wavefront (measured: 10 classes, 1,024 floats, one step in 1.0 us whatever else it did, now 0.55);
// with it 8 lines, and the turn takes four LDS writes and four reads.  us per call, as it lies in memory / turned: 10 classes, rows of 700 floats,
// 100,000 115.5 / 97.6, 30,000 39.9 / 37.8; 60 classes 108.7 / 99.7, 40.8 / 38.9; bfloat16 hidden layers of 64 and 128, 384 features, 30,000
// 32.6 / 30.7, 34.6 / 33.4.  Not where registers run out: 100 classes of floats 54.9 / 58.0 (60,000 rows of 512); nor for hidden layers on floats,
// which take fewer wavefronts per SIMD then: 100,000 of 100-32-10 46.0 / 48.9, of 128-64-10 49.7 / 50.2.  bfloat16 hidden layers of 33 to 64
// units turn rows while a window has at most two tiles per compute unit, the two wavefronts per SIMD that are left of three: 200,000 of
// 384-64-50 88.7 / 94.1.
template <typename T, int NB, bool MLP, int KS>
constexpr bool stream_turns() {
  if (sizeof(T) == 4) return !MLP && NB <= 2;
  return NB == 1 || (NB == 2 && !MLP) || (NB == 4 && (MLP || KS == 2));
}

template <typename T>
struct StreamIn {
  static constexpr bool kF32 = sizeof(T) == 4;
  static constexpr int kChunk = kStBytes / (int)sizeof(T);    // channels per step: 32 float32, 64 bfloat16
  static constexpr int kSteps = kChunk / 16;                  // k-steps of 16 per slice
  static constexpr int kParts = kF32 ? 2 : 1;                 // hi and lo, or the value itself
};

// What goes through the LDS buffers: a weight slice (256 NB units of 16 bytes), then per group of classes its table
// and bias (logistic), or per class tile its packed block (one hidden layer).  All have one size, a multiple of the
// workgroup, so that every stage is the same copy.
template <int NB, bool MLP>
struct StreamStage {
  static constexpr int kThreads = stream_waves(NB) * kWave;
  static constexpr int kSlice = 256 * NB;
  static constexpr int kBlock = MLP ? SplitBlock<32 * NB, 3>::kUnits : NB * (SplitBlock<32, 3>::kTabUnits + SplitBlock<32, 3>::kBiasUnits);
  static constexpr int kMax = kSlice > kBlock ? kSlice : kBlock;
  static constexpr int kPer = (kMax + kThreads - 1) / kThreads;    // units per thread
  static constexpr int kUnits = kPer * kThreads;
};

// Channel (inside a slice) of lane half g, k-step s, element e: a lane's share of a row is contiguous.
template <typename T>
inline int stream_channel(int s, int g, int e) { return g * (StreamIn<T>::kChunk / 2) + 8 * s + e; }

inline float host_times_2(float v, int e) { return std::ldexp(v, e); }
inline uint16_t host_times_2(uint16_t v, int e) {       // (bfloat16 bits)
  return (uint16_t)(__builtin_bit_cast(uint32_t, std::ldexp(__builtin_bit_cast(float, (uint32_t)v << 16), e)) >> 16);
}
// Largest absolute value (an infinity or a NaN if there is one), on the bits: every weight passes here a few times.
inline float host_abs_max(const float* v, size_t n) {
  uint32_t m = 0;
  for (size_t i = 0; i < n; ++i) m = std::max(m, __builtin_bit_cast(uint32_t, v[i]) & 0x7fffffffu);
  return __builtin_bit_cast(float, m);
}
inline float host_abs_max(const uint16_t* v, size_t n) {
  uint32_t m = 0;
  for (size_t i = 0; i < n; ++i) m = std::max(m, (uint32_t)v[i] & 0x7fffu);
  return __builtin_bit_cast(float, m << 16);
}
inline float host_value(float v) { return v; }
inline float host_value(uint16_t v) { return __builtin_bit_cast(float, (uint32_t)v << 16); }
// Which feature slot k of the padded row holds (-1: zero), and the part of its weight that counts there.  A piece of 16 bytes
// (`per` features) that would pass the row's end is read that much further left; the features that it repeats count by half
// in either place (exact in both types).  With the whole weight in one place and zero in the other an infinite feature would
// make NaNs, which a hidden layer's ReLU turns into zeros.  Pieces behind the row's end are zero.
struct StreamSlot { int feature; float part; };
inline StreamSlot stream_slot(int k, int d, int per) {
  const int full = d / per * per;
  if (k < full) return {k, k >= d - per && full < d ? 0.5f : 1.0f};
  if (k / per != full / per || full == d) return {-1, 0.f};
  const int f = d - per + k % per;
  return {f, f < full ? 0.5f : 1.0f};
}

// One weight slice: unit ((hb * kSteps + s) * kParts + part) * 64 + lane, halves e = 0..7 hold (part of)
// W[k = kChunk kc + channel(s, lane/32, e)][row0 + 32 hb + lane%32], zero beyond [d, O] (which input k is: stream_slot).
template <typename T, int NB>
inline void pack_stream_slice(const T* W /*[d, O]*/, int d, int O, int kc, int row0, float scale, uint16_t* out) {
  using I = StreamIn<T>;
  for (int hb = 0; hb < NB; ++hb)
    for (int s = 0; s < I::kSteps; ++s)
      for (int g = 0; g < 2; ++g)
        for (int e = 0; e < 8; ++e) {
          const StreamSlot slot = stream_slot(I::kChunk * kc + stream_channel<T>(s, g, e), d, 16 / (int)sizeof(T));
          const int k = slot.feature, o0 = row0 + 32 * hb;
          uint16_t* at = out + ((size_t)((hb * I::kSteps + s) * I::kParts) * 64 + 32 * g) * 8 + e;
          const T* from = W + (size_t)std::max(k, 0) * O + o0;
          for (int r = 0; r < 32 && k >= 0 && o0 + r < O; ++r) {      // (the buffer is zero to begin with)
            if constexpr (I::kF32) host_split((float)from[r] * (scale * slot.part), at[r * 8], at[(64 + r) * 8]);
            else at[r * 8] = slot.part == 1.0f ? (uint16_t)from[r] : host_times_2((uint16_t)from[r], -1);
          }
        }
}

// Inputs of very different ranges.  Halves that share one scale hold an input (or a weight) to 22 bits only down to 2^-18 of the
// largest, so an input that is small next to the others but has large weights to make up for it would lose bits that a
// float32 product keeps: with column scales of 10^+-4 expected accuracies were off by 1e-4.  What counts is an input's share in the sums,
// so inputs are multiplied by 2^e and their weights by 2^-e, e such that every input's largest weight has the same exponent.
// In front of a hidden layer's outputs this is exact and free (the ReLU commutes with it: it goes into the first layer's
// weights and biases); features are multiplied in the kernel (COLS), which only heads with a spread of more than kStreamSpread take:
// below it what is lost is less than 2^-28 of the largest product.  It costs 0.5 to 1.5 us: 41.4 -> 42.7 (32,768 rows of 768, 100
// classes), 29.4 -> 30.4 (100,000 of a 128-64-10 head), 42.8 -> 43.4 (60,000 of 200-256-40, which take 912 on the generic kernel).
constexpr int kStreamSpread = 10, kStreamShiftMax = 60;
// Exponents e (<= 0) of the rows of W [rows, cols], all zero where the rows' ranges are alike.  Rows of zeros get the smallest:
// such an input must not set the scale for the others.
template <typename T>
inline std::vector<int> equalizing_exponents(const T* W, int rows, int cols) {
  std::vector<int> e(rows, 0);
  int top = INT_MIN, low = INT_MAX;
  for (int k = 0; k < rows; ++k) {
    const float m = host_abs_max(W + (size_t)k * cols, (size_t)cols);
    if (!std::isfinite(m)) return std::vector<int>(rows, 0);
    if (m > 0.f) (void)std::frexp(m, &e[k]);
    else e[k] = INT_MIN;
    if (m > 0.f) top = std::max(top, e[k]);
    low = std::min(low, e[k]);
  }
  if (top == INT_MIN || (low != INT_MIN && top - low <= kStreamSpread)) return std::vector<int>(rows, 0);
  for (int k = 0; k < rows; ++k) e[k] = e[k] == INT_MIN ? -kStreamShiftMax : std::max(e[k] - top, -kStreamShiftMax);
  return e;
}

constexpr int kStreamMaxD = 1280;                // longest row: the context's limit on d + H (its generic kernel's LDS)

struct StreamHeads {
  const unsigned char* stages;    // per application: its stages, kUnits * 16 bytes each
  const int64_t* off;             // [A] byte offsets
  const float* b1;                // [A, 32 NB] first-layer bias of one-hidden-layer heads, padded with zeros
  const float* unscale1;          // [A] undoes the first layer's weight scale (1 for bfloat16)
  const float* unscale2;          // [A] undoes the second layer's
  const float* cols;              // [A, steps * channels] factor of every slot of a row (COLS), see equalizing_exponents
};

static __device__ f32x4 stream_zeros;            // what lies behind a row's end

// 16 bytes of a feature row: rows start at any multiple of the element size
typedef f32x4 f32x4_any __attribute__((aligned(2)));

template <typename T, int NB, bool MLP, bool COLS = false, int KS = 1, bool TURN = stream_turns<T, NB, MLP, KS>()>
__global__ __launch_bounds__(KS * stream_waves(NB) * kWave, 2) void k_score_stream(
    Tables tb, Window w, const T* __restrict__ x, const int32_t* __restrict__ ids, const float2* __restrict__ dw_g,
    uint32_t* __restrict__ sortkey, StreamHeads hd, float* __restrict__ logits_out) {
  using I = StreamIn<T>;
  using SG = StreamStage<NB, MLP>;
  constexpr int S = I::kSteps, CH = I::kChunk, D = 32 * NB;
  constexpr int kTurns = I::kF32 ? 3 : 2;                // matrix instructions per block and half of a slice
  static_assert(!COLS || I::kF32, "bfloat16 features are not scaled");
  static_assert(KS == 1 || (KS == 2 && !MLP && NB <= 4), "logistic heads with all classes in one group");
  __shared__ f32x4 bufs[KS][2][SG::kUnits];
  __shared__ f32x4 cols[COLS ? kStreamMaxD / 4 : 1];
  // (KS == 2: which of the two teams of wavefronts, and the place in it)
  const int team = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / SG::kThreads);
  const int tid = KS == 1 ? (int)threadIdx.x : (int)threadIdx.x & (SG::kThreads - 1), lane = tid & 63, wave = tid >> 6;
  f32x4 (&buf)[2][SG::kUnits] = bufs[team];
  const int r = lane & 31, g = lane >> 5;
  const int4 desc = w.tile_desc[blockIdx.x];
  if (desc.x < 0) return;
  // (uniform, which the compiler cannot know of a load: tables and stages are then addressed from scalar registers)
  const int a = __builtin_amdgcn_readfirstlane(desc.x), seg_e = __builtin_amdgcn_readfirstlane(desc.z);
  const int pos = desc.y + wave * 32 + r;
  const bool valid = pos < seg_e;
  const int id = ids[valid ? pos : seg_e - 1];           // padding lanes recompute the last request, never store
  const int d = tb.d, C = __builtin_amdgcn_readfirstlane(tb.n_classes[a]), M = __builtin_amdgcn_readfirstlane(tb.n_models[a]);
  const int CT = (C + kClassTile - 1) / kClassTile;
  const int nkc = (d + CH - 1) / CH;
  const int n_groups = MLP ? 1 : (CT + NB - 1) / NB;
  const int n_stages = MLP ? nkc + CT : n_groups * (nkc + 1);
  const int steps = (nkc + KS - 1) / KS;                 // a team's share of the slices: every KS-th
  const auto slice_of = [&](int i) { return KS * i + team; };
  const bool dump = logits_out != nullptr, split = tb.pol_split != 0;

  // ---- stages: loaded into registers one or (kAhead) two ahead, stored into the idle buffer when the running one is done ----
  constexpr bool kAhead = KS == 2;
  const f32x4* src;
  {
    const int64_t o = hd.off[a];
    const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)o), hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)o >> 32));
    src = reinterpret_cast<const f32x4*>(hd.stages + (int64_t)(((uint64_t)hi << 32) | lo));
  }
  typedef f32x4 Staged[SG::kPer];
  Staged w0, w1;
  auto fetch = [&](int st, Staged& wst) {
    // (a team whose last slice does not exist multiplies zeros by another one's weights)
    const int at = KS == 1 ? min(st, n_stages - 1) : st >= steps ? nkc : min(slice_of(st), nkc - 1);
    const f32x4* p = src + (size_t)at * SG::kUnits;
#pragma unroll
    for (int i = 0; i < SG::kPer; ++i) wst[i] = p[(uint32_t)(tid + i * SG::kThreads)];
  };
  auto park = [&](int st, const Staged& wst) {
    f32x4* b = buf[st & 1] + tid;
#pragma unroll
    for (int i = 0; i < SG::kPer; ++i) b[i * SG::kThreads] = wst[i];
  };

  // ---- features: this lane's 64 bytes of a step, 16 at a time.  kTurn: read in whole lines, eight lanes a row, and turned in LDS (a
  // wavefront its own rows), where piece p of row r lies in place p ^ (r % 8) of the row: no bank conflicts on either side ----
  constexpr bool kTurn = TURN;
  __shared__ f32x4 turn[KS * stream_waves(NB)][kTurn || KS == 2 ? 32 * 8 : 1];
  constexpr int kRows = kTurn ? 4 : 1;
  const unsigned char* rows[kRows];
#pragma unroll
  for (int q = 0; q < kRows; ++q)
    rows[q] = reinterpret_cast<const unsigned char*>(x + (int64_t)(kTurn ? __shfl(id, 8 * q + (lane >> 3)) : id) * d);
  const int row_bytes = d * (int)sizeof(T);              // >= 16
  auto load_x = [&](f32x4 (&xs)[4], int kc) {
    const int first = kStBytes * kc + (kTurn ? 16 * ((lane & 7) ^ (lane >> 3)) : 64 * g);
    const auto at = [&](int q) { return kTurn ? first : first + 16 * q; };
    if (kStBytes * (kc + 1) <= row_bytes) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const unsigned char* p = rows[kTurn ? q : 0] + at(q);
        if constexpr (I::kF32) xs[q] = *reinterpret_cast<const f32x4_dw*>(p);
        else xs[q] = *reinterpret_cast<const f32x4_any*>(p);
      }
    } else if (kc < nkc) {                               // the last, partial step (see stream_slot)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const unsigned char* p = rows[kTurn ? q : 0] + min(at(q), row_bytes - 16);
        xs[q] = *reinterpret_cast<const f32x4_any*>(at(q) < row_bytes ? p : reinterpret_cast<const unsigned char*>(&stream_zeros));
      }
    } else {                                             // past it
#pragma unroll
      for (int q = 0; q < 4; ++q) xs[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  auto turned = [&](const f32x4 (&xs)[4], f32x4 (&xv)[4]) {
    if constexpr (kTurn) {
      f32x4* const own = turn[threadIdx.x >> 6];
#pragma unroll
      for (int q = 0; q < 4; ++q) own[64 * q + lane] = xs[q];
      wave_sync();
#pragma unroll
      for (int q = 0; q < 4; ++q) xv[q] = own[8 * r + ((4 * g + q) ^ (r & 7))];
      wave_sync();
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) xv[q] = xs[q];
    }
  };

  float m2 = kNegBig, m2_rest = 0.f, best_z = kNegBig, ssum = 0.f, ssum_hi = 0.f;
  int best_c = 0x7fffffff;
  f32x4 ea_lo = {0.f, 0.f, 0.f, 0.f}, ea_hi = {0.f, 0.f, 0.f, 0.f};
  const int64_t dump_row = (int64_t)id * tb.Cmax;
  f32x16 acc[NB];
  int ex = 1000;                                         // float32: the row's running scale 2^ex (none yet)
  bool infinite = false;                                 // float32, hidden layer: the row holds an infinity
  const float un1 = I::kF32 ? hd.unscale1[a] : 1.f;

  fetch(0, w0);
  park(0, w0);
  if (kAhead) fetch(1, w1);
  if (COLS)
    for (int i = threadIdx.x; i < nkc * (CH / 4); i += KS * SG::kThreads) cols[i] = reinterpret_cast<const f32x4*>(hd.cols)[(size_t)a * nkc * (CH / 4) + i];
  __syncthreads();

  int st = 0;                                            // running stage
  for (int grp = 0; grp < n_groups; ++grp) {
    const int nbk = MLP ? NB : min(NB, CT - grp * NB);   // blocks of 32 rows that hold anything
    f32x4 x0[4], x1[4];
    int k0 = 0;
    asm volatile("" : "+s"(k0));                         // (a zero that the compiler cannot see: it would keep every address of the
    load_x(x0, slice_of(k0));                            // first steps in registers from one group to the next)
    load_x(x1, slice_of(k0 + 1));
    ex = 1000;
#pragma unroll
    for (int hb = 0; hb < NB; ++hb)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[hb][v] = 0.f;

    // The running slice's weight fragments, kFrags per block of 32 rows.  Two blocks run side by side: a matrix instruction that
    // takes the result of the one before can issue every 52 cycles only, an independent one every 32 (and the sums of one block
    // would wait for its last instruction with nothing to fill the time).  The fragments of half of a pair's steps are read ahead of the
    // instructions that take those of the other half.  With eight blocks the registers are needed for the accumulators: block by
    // block there.
    constexpr int kFrags = S * I::kParts;
    static_assert(kFrags == 4, "one block of a slice is four fragments for either type");
    auto blocks = [&](auto mfma /* (half of the steps, two fragments, sums) */) {
      const f32x4* cur = buf[st & 1] + lane;
      if constexpr (NB == 1 || NB == 8) {
        f32x4 wf[kFrags];
#pragma unroll
        for (int hb = 0; hb < NB; ++hb) {
#pragma unroll
          for (int i = 0; i < kFrags; ++i) wf[i] = cur[(hb * kFrags + i) * 64];
          __builtin_amdgcn_sched_barrier(0);
          if (hb < nbk) {
            f32x16 part;
#pragma unroll
            for (int v = 0; v < 16; ++v) part[v] = 0.f;
#pragma unroll
            for (int i = 0; i < kFrags / 2 * kTurns; ++i) mfma(i / kTurns, i % kTurns, wf[2 * (i / kTurns)], wf[2 * (i / kTurns) + 1], part);
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[hb][v] += part[v];
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
        f32x4 wf[2][kFrags];                                       // fragments of either block: 2 * block + i
        auto read = [&](int u) {                                   // half u of the slice: pair u / 2, its steps' half u % 2
#pragma unroll
          for (int i = 0; i < kFrags; ++i) wf[u & 1][i] = cur[((2 * (u >> 1) + (i >> 1)) * kFrags + 2 * (u & 1) + (i & 1)) * 64];
        };
        read(0);
#pragma unroll
        for (int p = 0; p < NB / 2; ++p) {
          if (2 * p >= nbk) continue;                              // (a last block that holds nothing keeps its neighbour company)
          f32x16 part[2];
#pragma unroll
          for (int v = 0; v < 16; ++v) part[0][v] = part[1][v] = 0.f;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int u = 2 * p + h;
            if (u + 1 < NB) read(u + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < kTurns; ++i) {
              mfma(h, i, wf[u & 1][0], wf[u & 1][1], part[0]);
              mfma(h, i, wf[u & 1][2], wf[u & 1][3], part[1]);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[2 * p][v] += part[0][v];
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[2 * p + 1][v] += part[1][v];
        }
      }
    };
    // one step: stage st + 1 and the features of step i + 2 start, the MFMAs of step i run, stage st + 1 is stored.
    // The features of step i are converted, or copied, first: that frees their registers for step i + 2.  (kAhead: stage st + 2 starts, and
    // stage st + 1 has been on its way since the step before.)
    auto slice_f32 = [&](int i, f32x4 (&xs)[4], Staged& w_new, Staged& w_next) {
      if (kAhead) fetch(st + 2, w_new); else fetch(st + 1, w0);
      __builtin_amdgcn_sched_barrier(0);
      f32x4 xv[4];
      turned(xs, xv);
      if (kTurn) {                                                 // (the registers are free already)
        load_x(xs, slice_of(i + 2));
        __builtin_amdgcn_sched_barrier(0);
      }
      if (COLS) {
#pragma unroll
        for (int q = 0; q < 4; ++q) xv[q] *= cols[(KS == 1 ? i : min(slice_of(i), nkc - 1)) * (CH / 4) + 4 * g + q];
      }
      float amax = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int j = 0; j < 4; ++j) amax = fmaxf(amax, fabsf(xv[q][j]));
      amax = fmaxf(amax, other_half(amax, g));
      // amax = f 2^e with f in [0.5, 1): |x| 2^(15 - e) < 2^15; bounded so that the scale stays a normal number
      const int e = (int)((__float_as_uint(amax) >> 23) & 0xffu) - 126;
      const int want = min(max(kSplitExp - e, -113), 128);
      if (MLP) infinite |= e > 128;
      if (__builtin_amdgcn_ballot_w64(want < ex) != 0ull) {
        // two bits of headroom, so that the maximum of a few more values rarely asks for another rescaling
        const int nex = want < ex ? want - 2 : ex;
        const float f = __builtin_amdgcn_ldexpf(1.0f, max(nex - ex, -1000));
#pragma unroll
        for (int hb = 0; hb < NB; ++hb)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[hb][v] *= f;
        ex = nex;
      }
      const float xsc = __builtin_amdgcn_ldexpf(1.0f, ex);
      f16x8 xh[S], xl[S];
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int j = 0; j < 4; j += 2) {
          f16x2 hi, lo;
          split_f16x2(xv[q][j] * xsc, xv[q][j + 1] * xsc, hi, lo);
          const int k = 4 * q + j;
          xh[k >> 3][k & 7] = hi[0]; xh[k >> 3][(k & 7) + 1] = hi[1];
          xl[k >> 3][k & 7] = lo[0]; xl[k >> 3][(k & 7) + 1] = lo[1];
        }
      __builtin_amdgcn_sched_barrier(0);
      if (!kTurn) {
        load_x(xs, slice_of(i + 2));
        __builtin_amdgcn_sched_barrier(0);
      }
      blocks([&](int half, int turn, const f32x4& whf, const f32x4& wlf, f32x16& part) {
        const f16x8 wh = __builtin_bit_cast(f16x8, whf), wl = __builtin_bit_cast(f16x8, wlf);
        part = __builtin_amdgcn_mfma_f32_32x32x16_f16(turn == 0 ? wl : wh, turn == 1 ? xl[half] : xh[half], part, 0, 0, 0);
      });
      park(st + 1, kAhead ? w_next : w0);
      __syncthreads();
      ++st;
    };
    auto slice_bf16 = [&](int i, f32x4 (&xs)[4], Staged& w_new, Staged& w_next) {
      if (kAhead) fetch(st + 2, w_new); else fetch(st + 1, w0);
      __builtin_amdgcn_sched_barrier(0);
      f32x4 xv[4];
      turned(xs, xv);
      bf16x8 xc[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) xc[q] = as_bf16x8(xv[q]);
      load_x(xs, slice_of(i + 2));
      __builtin_amdgcn_sched_barrier(0);
      blocks([&](int half, int turn, const f32x4& w0, const f32x4& w1, f32x16& part) {
        part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(turn == 0 ? w0 : w1), xc[2 * half + turn], part, 0, 0, 0);
      });
      park(st + 1, kAhead ? w_next : w0);
      __syncthreads();
      ++st;
    };
    for (int i = k0;; i += 2) {
      if constexpr (I::kF32) slice_f32(i, x0, w0, w1); else slice_bf16(i, x0, w0, w1);
      if (i + 1 < steps) {                               // (one way out of the loop: with two, the accumulators are copied)
        if constexpr (I::kF32) slice_f32(i + 1, x1, w1, w0); else slice_bf16(i + 1, x1, w1, w0);
      }
      if (i + 2 >= steps) break;
    }

    if constexpr (KS == 2) {
      // The teams' sums meet: each finishes half of the blocks (of one block the first team all) with what the other has summed for
      // them, both brought to the smaller of the two scales.
      constexpr int kOwn = NB == 1 ? 1 : NB / 2;
      // (a team's idle buffer and the places where its rows were turned; nobody reads either any more)
      static_assert(kOwn == 1 || SG::kUnits >= 4 * SG::kThreads, "room for a block in a buffer");
      const auto meet = [&](int of, int j) { return j + 1 == kOwn ? turn[of * stream_waves(NB)] : bufs[of][(st & 1) ^ 1]; };
      __shared__ int32_t meet_ex[2][SG::kThreads];
      const bool second = team != 0;
      f32x16 fin[kOwn];
#pragma unroll
      for (int j = 0; j < kOwn; ++j) {
        const int hi = NB == 1 ? 0 : kOwn + j;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          f32x4 give;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            fin[j][4 * q + v] = second ? acc[hi][4 * q + v] : acc[j][4 * q + v];
            give[v] = second ? acc[j][4 * q + v] : acc[hi][4 * q + v];
          }
          meet(team, j)[q * SG::kThreads + tid] = give;
        }
      }
      meet_ex[team][tid] = ex;
      __syncthreads();
      const int ex_other = meet_ex[team ^ 1][tid], ex_min = min(ex, ex_other);
      const float f_mine = I::kF32 ? __builtin_amdgcn_ldexpf(1.0f, max(ex_min - ex, -1000)) : 1.0f;
      const float f_other = I::kF32 ? __builtin_amdgcn_ldexpf(1.0f, max(ex_min - ex_other, -1000)) : 1.0f;
      const float un = I::kF32 ? __builtin_amdgcn_ldexpf(un1, -ex_min) : 1.f;
      const float4* tab = reinterpret_cast<const float4*>(buf[st & 1]);
      const int first = NB == 1 ? 2 * team : kOwn * team;          // (of one block the second team has none)
#pragma unroll
      for (int j = 0; j < kOwn; ++j) {
        const int hb = first + j;
        if (hb >= nbk) continue;                                   // (uniform)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 take = meet(team ^ 1, j)[q * SG::kThreads + tid];
#pragma unroll
          for (int v = 0; v < 4; ++v) fin[j][4 * q + v] = I::kF32 ? fmaf(fin[j][4 * q + v], f_mine, take[v] * f_other) : fin[j][4 * q + v] + take[v];
        }
        softmax_tile<true>(tab + hb * SplitBlock<32, 3>::kTabUnits, tab + NB * SplitBlock<32, 3>::kTabUnits + hb * SplitBlock<32, 3>::kBiasUnits,
                     fin[j], un, ea_lo, ea_hi, ssum, ssum_hi, m2, m2_rest, hb, C, g, lane, valid, dump_row, logits_out, best_z, best_c, dump, split);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (dump) return;
      // ... and so do their expected accuracies and denominators, in the first team's registers.
      __syncthreads();
      float* const part = reinterpret_cast<float*>(turn) + tid;
      constexpr int kParts = 14;
      static_assert(sizeof(turn) >= kParts * SG::kThreads * sizeof(float), "room for a team's results");
      const auto cell = [&](int k) -> float& { return part[k * SG::kThreads]; };
      if (second) {
        cell(0) = m2; cell(1) = m2_rest; cell(2) = ssum; cell(3) = ssum_hi; cell(4) = best_z; cell(5) = __int_as_float(best_c);
#pragma unroll
        for (int v = 0; v < 4; ++v) { cell(6 + v) = ea_lo[v]; cell(10 + v) = ea_hi[v]; }
      }
      __syncthreads();
      if (second) return;
      const float om2 = cell(0), orest = cell(1), top = fmaxf(m2, om2);
      const float rest = m2 > om2 ? m2_rest : m2 == om2 ? fmaxf(m2_rest, orest) : orest;
      // factors of this lane's request and, for the sums of the requests that the neighbouring row holds, of that one (see softmax_tile)
      const auto factors = [&](float scale, float& lo, float& hi) {
        typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
        const u32x2 sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(scale), __float_as_uint(scale), false, false);
        const bool odd = (lane & 16) != 0;
        const float nb = __uint_as_float(odd ? sw[0] : sw[1]);
        lo = odd ? nb : scale;
        hi = odd ? scale : nb;
      };
      float mine_lo, mine_hi, other_lo, other_hi;
      factors(__builtin_amdgcn_exp2f((m2 - top) + (m2_rest - rest)), mine_lo, mine_hi);
      factors(__builtin_amdgcn_exp2f((om2 - top) + (orest - rest)), other_lo, other_hi);
      ssum = fmaf(ssum, mine_lo, cell(2) * other_lo);
      ssum_hi = fmaf(ssum_hi, mine_hi, cell(3) * other_hi);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        ea_lo[v] = fmaf(ea_lo[v], mine_lo, cell(6 + v) * other_lo);
        ea_hi[v] = fmaf(ea_hi[v], mine_hi, cell(10 + v) * other_hi);
      }
      const float oz = cell(4);
      if (oz > best_z) { best_z = oz; best_c = __float_as_int(cell(5)); }     // (its classes come later)
      m2 = top;
      m2_rest = rest;
      break;
    }
    const float un = I::kF32 ? __builtin_amdgcn_ldexpf(un1, -ex) : 1.f;
    if constexpr (!MLP) {
      // the group's table and bias are the running stage; the next group's first slice follows
      const float4* tab = reinterpret_cast<const float4*>(buf[st & 1]);
      fetch(st + 1, w0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int hb = 0; hb < NB; ++hb) {
        if (hb < nbk)
          softmax_tile<true>(tab + hb * SplitBlock<32, 3>::kTabUnits, tab + NB * SplitBlock<32, 3>::kTabUnits + hb * SplitBlock<32, 3>::kBiasUnits,
                       acc[hb], un, ea_lo, ea_hi, ssum, ssum_hi, m2, m2_rest, grp * NB + hb, C, g, lane, valid, dump_row, logits_out, best_z, best_c,
                       dump, split);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (grp + 1 < n_groups) {
        park(st + 1, w0);
        __syncthreads();
        ++st;
        if (kAhead) fetch(st + 1, w1);
      }
    } else {
      // Rows with an infinity (their halves are NaN): every hidden unit by the features that are not finite, as float32
      // arithmetic has it; infinities swallow the finite products.  The weights come out of the packed slices.
      if (I::kF32 && __builtin_amdgcn_ballot_w64(infinite) != 0ull) {
#pragma unroll
        for (int hb = 0; hb < NB; ++hb)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[hb][v] = infinite ? 0.f : acc[hb][v];
        const int full = d & ~3;
        for (int k = 0; k < d; ++k) {
          const float xv = static_cast<float>(x[(int64_t)id * d + k]);
          const bool odd = infinite && !(fabsf(xv) < __builtin_inff());
          if (__builtin_amdgcn_ballot_w64(odd) == 0ull) continue;
          const int slot = k < full ? k : full + k - (d - 4), in = slot % CH, gk = in / (CH / 2), e = in % (CH / 2);   // (see stream_slot)
          const _Float16* wk = reinterpret_cast<const _Float16*>(src + (size_t)(slot / CH) * SG::kUnits + (e >> 3) * 128 + 32 * gk) + (e & 7);
#pragma unroll
          for (int hb = 0; hb < NB; ++hb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
              const int at = hb * S * 128 + 8 * (v >> 2) + 4 * g + (v & 3);       // units of 8 halves
              const float wv = (float)wk[at * 8] + (float)wk[(at + 64) * 8];
              acc[hb][v] = odd ? acc[hb][v] + xv * wv : acc[hb][v];
            }
        }
      }
      // bias, ReLU, per-request scale, split: acc[hb][v] of lane (r, g) is hidden unit 32 hb + 8 (v/4) + 4 g + v%4
      const float4* b1p = reinterpret_cast<const float4*>(hd.b1 + (size_t)a * D);
      float amax = 0.f;
#pragma unroll
      for (int hb = 0; hb < NB; ++hb)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 bq = b1p[8 * hb + 2 * q + g];
          const float bb[4] = {bq.x, bq.y, bq.z, bq.w};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            acc[hb][4 * q + j] = fmaxf(fmaf(acc[hb][4 * q + j], un, bb[j]), 0.f);
            amax = fmaxf(amax, acc[hb][4 * q + j]);
          }
        }
      amax = fmaxf(amax, other_half(amax, g));
      int hx = 0;
      if (amax < __builtin_inff()) hx = min(kSplitExp - ((int)((__float_as_uint(amax) >> 23) & 0xffu) - 126), 126);
      const float hs = __uint_as_float((uint32_t)(127 + hx) << 23);
      const float unscale = __uint_as_float((uint32_t)(127 - hx) << 23) * hd.unscale2[a];
      f16x8 xh[D / 16], xl[D / 16];
#pragma unroll
      for (int hb = 0; hb < NB; ++hb)
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
          f16x2 hi, lo;
          split_f16x2(acc[hb][v] * hs, acc[hb][v + 1] * hs, hi, lo);
          xh[2 * hb + (v >> 3)][v & 7] = hi[0]; xh[2 * hb + (v >> 3)][(v & 7) + 1] = hi[1];
          xl[2 * hb + (v >> 3)][v & 7] = lo[0]; xl[2 * hb + (v >> 3)][(v & 7) + 1] = lo[1];
        }
      for (int ct = 0; ct < CT; ++ct) {
        const float4* blk = reinterpret_cast<const float4*>(buf[st & 1]);
        if (ct + 1 < CT) fetch(st + 1, w0);
        __builtin_amdgcn_sched_barrier(0);
        f32x16 z;
        logits_phase<D>(blk, xh, xl, z, lane);
        softmax_tile<true>(blk + SplitBlock<D, 3>::kWUnits, blk + SplitBlock<D, 3>::kWUnits + SplitBlock<D, 3>::kTabUnits, z, unscale, ea_lo, ea_hi,
                     ssum, ssum_hi, m2, m2_rest, ct, C, g, lane, valid, dump_row, logits_out, best_z, best_c, dump, split);
        if (ct + 1 < CT) {
          park(st + 1, w0);
          __syncthreads();
        }
        ++st;
      }
    }
  }
  if (dump) return;
  // (the denominators lie like the numerators and span both lane halves; the epilogue adds the halves' sums)
  ssum = 0.5f * (r < 16 ? ssum : ssum_hi);
  score_epilogue<true>(tb, w, ea_lo, ea_hi, ssum, -m2, 16384.0f, m2_rest, best_z, best_c, a, M, pos, id, valid, lane, dw_g, sortkey, split);
}

}  // namespace sp
