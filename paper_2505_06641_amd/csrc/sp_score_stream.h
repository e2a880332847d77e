// Scoring kernel on the matrix cores for the heads that the two kernels with a fixed input width do not take:
// logistic heads on bfloat16 features or on float32 features wider than 256, and one-hidden-layer heads (H <= 256)
// on float32 features or on bfloat16 features that those kernels pad too much (Def. 4.1.1, 4.1.2; Sec. 4.1 eq. (9);
// Sec. 5.1.1 eq. (12)).
//
// A wavefront owns 32 requests and keeps the whole transposed output tile of the first layer (32 NB rows: hidden
// units, or classes) in NB float32 accumulators while it streams its requests' features from memory, kStBytes per
// row and step; the matching weight slices, packed at context creation in the order the lanes read them, go through
// two LDS buffers shared by the workgroup's four wavefronts.  Features never pass through LDS: the order of a slice's
// channels is free as long as the weights are packed in the same one, so a lane takes 64 consecutive bytes of its
// request's row.  A step costs memory more than matrix cores in all of these shapes, so features travel two steps ahead.
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
// Measured (rocprofv3, median us, before -> now): 32,768 rows of 768 floats, 100 classes 1543 -> 38.7 (2.6 TB/s of rows);
// 65,536 rows of 512 bfloat16, 100 classes 1273 -> 26.2 (2.6 TB/s); 100,000 requests of 128-64-10/7/2 float32 heads 185 -> 27.0
// (1.9 TB/s), all three from the generic kernel; 30,011 of 384-128-100/37/10 bfloat16 heads 29 -> 20.6 (1.1 TB/s), from the
// kernel that pads the hidden layer to 256.  A large copy reaches 5.2 TB/s on this card (read and written).
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

template <typename T, int NB, bool MLP, bool COLS = false>
__global__ __launch_bounds__(stream_waves(NB) * kWave, 2) void k_score_stream(
    Tables tb, Window w, const T* __restrict__ x, const int32_t* __restrict__ ids, const float2* __restrict__ dw_g,
    uint32_t* __restrict__ sortkey, StreamHeads hd, float* __restrict__ logits_out) {
  using I = StreamIn<T>;
  using SG = StreamStage<NB, MLP>;
  constexpr int S = I::kSteps, CH = I::kChunk, D = 32 * NB;
  constexpr int kTurns = I::kF32 ? 3 : 2;                // matrix instructions per block and half of a slice
  static_assert(!COLS || I::kF32, "bfloat16 features are not scaled");
  __shared__ f32x4 buf[2][SG::kUnits];
  __shared__ f32x4 cols[COLS ? kStreamMaxD / 4 : 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
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
  const bool dump = logits_out != nullptr, split = tb.pol_split != 0;

  // ---- stages: loaded into registers one ahead, stored into the idle buffer when the running one is done ----
  const f32x4* src;
  {
    const int64_t o = hd.off[a];
    const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)o), hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)o >> 32));
    src = reinterpret_cast<const f32x4*>(hd.stages + (int64_t)(((uint64_t)hi << 32) | lo));
  }
  f32x4 wst[SG::kPer];
  auto fetch = [&](int st) {
    const f32x4* p = src + (size_t)min(st, n_stages - 1) * SG::kUnits;
#pragma unroll
    for (int i = 0; i < SG::kPer; ++i) wst[i] = p[(uint32_t)(tid + i * SG::kThreads)];
  };
  auto park = [&](int st) {
    f32x4* b = buf[st & 1] + tid;
#pragma unroll
    for (int i = 0; i < SG::kPer; ++i) b[i * SG::kThreads] = wst[i];
  };

  // ---- features: this lane's 64 bytes of a step ----
  const unsigned char* row = reinterpret_cast<const unsigned char*>(x + (int64_t)id * d);
  const int row_bytes = d * (int)sizeof(T);              // >= 16
  auto load_x = [&](f32x4 (&xs)[4], int kc) {
    const int at = kStBytes * kc + 64 * g;
    if (kStBytes * (kc + 1) <= row_bytes) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if constexpr (I::kF32) xs[q] = *reinterpret_cast<const f32x4_dw*>(row + at + 16 * q);
        else xs[q] = *reinterpret_cast<const f32x4_any*>(row + at + 16 * q);
      }
    } else if (kc < nkc) {                               // the last, partial step (see stream_slot)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const unsigned char* p = row + min(at + 16 * q, row_bytes - 16);
        xs[q] = *reinterpret_cast<const f32x4_any*>(at + 16 * q < row_bytes ? p : reinterpret_cast<const unsigned char*>(&stream_zeros));
      }
    } else {                                             // past it
#pragma unroll
      for (int q = 0; q < 4; ++q) xs[q] = f32x4{0.f, 0.f, 0.f, 0.f};
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

  fetch(0);
  park(0);
  if (COLS)
    for (int i = tid; i < nkc * (CH / 4); i += SG::kThreads) cols[i] = reinterpret_cast<const f32x4*>(hd.cols)[(size_t)a * nkc * (CH / 4) + i];
  __syncthreads();

  int st = 0;                                            // running stage
  for (int grp = 0; grp < n_groups; ++grp) {
    const int nbk = MLP ? NB : min(NB, CT - grp * NB);   // blocks of 32 rows that hold anything
    f32x4 x0[4], x1[4];
    int k0 = 0;
    asm volatile("" : "+s"(k0));                         // (a zero that the compiler cannot see: it would keep every address of the
    load_x(x0, k0);                                      // first steps in registers from one group to the next)
    load_x(x1, k0 + 1);
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
    // one step: stage st + 1 and the features of step kc + 2 start, the MFMAs of step kc run, stage st + 1 is stored.
    // The features of step kc are converted, or copied, first: that frees their registers for step kc + 2.
    auto slice_f32 = [&](int kc, f32x4 (&xs)[4]) {
      fetch(st + 1);
      __builtin_amdgcn_sched_barrier(0);
      f32x4 xv[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) xv[q] = COLS ? xs[q] * cols[kc * (CH / 4) + 4 * g + q] : xs[q];
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
      load_x(xs, kc + 2);
      __builtin_amdgcn_sched_barrier(0);
      blocks([&](int half, int turn, const f32x4& whf, const f32x4& wlf, f32x16& part) {
        const f16x8 wh = __builtin_bit_cast(f16x8, whf), wl = __builtin_bit_cast(f16x8, wlf);
        part = __builtin_amdgcn_mfma_f32_32x32x16_f16(turn == 0 ? wl : wh, turn == 1 ? xl[half] : xh[half], part, 0, 0, 0);
      });
      park(st + 1);
      __syncthreads();
      ++st;
    };
    auto slice_bf16 = [&](int kc, f32x4 (&xs)[4]) {
      fetch(st + 1);
      __builtin_amdgcn_sched_barrier(0);
      bf16x8 xc[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) xc[q] = as_bf16x8(xs[q]);
      load_x(xs, kc + 2);
      __builtin_amdgcn_sched_barrier(0);
      blocks([&](int half, int turn, const f32x4& w0, const f32x4& w1, f32x16& part) {
        part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(turn == 0 ? w0 : w1), xc[2 * half + turn], part, 0, 0, 0);
      });
      park(st + 1);
      __syncthreads();
      ++st;
    };
    for (int kc = k0;; kc += 2) {
      if constexpr (I::kF32) slice_f32(kc, x0); else slice_bf16(kc, x0);
      if (kc + 1 < nkc) {                                // (one way out of the loop: with two, the accumulators are copied)
        if constexpr (I::kF32) slice_f32(kc + 1, x1); else slice_bf16(kc + 1, x1);
      }
      if (kc + 2 >= nkc) break;
    }

    const float un = I::kF32 ? __builtin_amdgcn_ldexpf(un1, -ex) : 1.f;
    if constexpr (!MLP) {
      // the group's table and bias are the running stage; the next group's first slice follows
      const float4* tab = reinterpret_cast<const float4*>(buf[st & 1]);
      fetch(st + 1);
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
        park(st + 1);
        __syncthreads();
        ++st;
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
        if (ct + 1 < CT) fetch(st + 1);
        __builtin_amdgcn_sched_barrier(0);
        f32x16 z;
        logits_phase<D>(blk, xh, xl, z, lane);
        softmax_tile<true>(blk + SplitBlock<D, 3>::kWUnits, blk + SplitBlock<D, 3>::kWUnits + SplitBlock<D, 3>::kTabUnits, z, unscale, ea_lo, ea_hi,
                     ssum, ssum_hi, m2, m2_rest, ct, C, g, lane, valid, dump_row, logits_out, best_z, best_c, dump, split);
        if (ct + 1 < CT) {
          park(st + 1);
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
