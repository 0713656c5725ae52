// A target row evaluated and sampled by one workgroup of 1024 threads, in fp64:
//   row_sweep    one pass over the row for the masses sum exp(s - ref) of its runs, kept in LDS
//   row_eval     the normaliser, and p and q_hat at the received set's entries
//   row_test     the acceptance test of one candidate, row_update the residual update after a rejection
//   row_locate, row_pick   the token at which the cumulative mass of p, or of what the updates made of it, passes
//                u * total, in ascending token index: the run that holds it, then the element
// fp64 is needed for the sampling: at V >= 128k the buckets of the inverse CDF are far narrower than fp32 prefix
// sums can resolve.  One workgroup per row keeps the sums in LDS and one pass serves the test and the sample.  Where few
// long rows leave compute units idle several workgroups sweep one, leave the sums in memory, and the one that finds those of all goes
// on with the row (row_shared; handover.h).
#pragma once
#include <algorithm>
#include <type_traits>
#include "common.h"
#include "exp64.h"
#include "handover.h"
#include "pow_table.h"
#include "rowops.h"

namespace tslt {

constexpr int kRowThreads = 1024;                   // one entry of a received set per thread (TSLT_MAX_K_CAP)
constexpr int kRowWaves = kRowThreads / 64;
// Waves per SIMD asked of the compiler: 4 (128 registers) while every row has a compute unit to itself, where a
// spilled value in the chain of steps after the sweep costs a memory latency; 8 (two workgroups on a compute unit)
// for more rows than that, where one sweeps while the other is in that chain.
constexpr int kAlone = 4, kShared = 8;
constexpr int kMaxStages = 16;                      // candidates of a node (TSLT_MAX_BRANCH)
constexpr int kMaxRuns = (kBlock - 2) * kSubChunks;
constexpr int kMaxItems = kMaxRuns + 2;             // a row's runs, and the elements before and after its aligned body
static_assert(kMaxItems <= kRowThreads, "one item per thread");

// The fp64 terms of a row are made in one of two ways, both referenced to 0 rather than to the row maximum,
// which is safe while s <= kTabMaxS and something lies above -kTabMaxS (what lies below is nothing beside it); a row
// that holds a larger s, or nothing but smaller ones, is swept again, referenced to its maximum.
//
// BitTerms, 16-bit rows: a table of exp(s), s = fl32(z / T), for every logit z of a magnitude range that holds
// the bulk of a row; a term costs five instructions and one LDS read.
//   bfloat16  2^-14 <= |z| < 2^7   5376 values, 42 KB  (logits centred on 0 have many small values)
//   binary16  2^-2  <= |z| < 2^5  14336 values, 112 KB: for the large batches of very long rows only (verify.h)
// With the 16 bits of an element rotated left by one (sign in bit 0), entry 1 + (rotated - 2*kLo) holds
// its value; entries 0 and kEntries + 1 hold NaN and stand for everything below and above the table's
// domain (tiny, huge, -inf, NaN), which is evaluated directly.
//
// PowTerms, every type: exp64.h's pow_exp on a table of 2^(i/2048) (16 KB).  19 instructions per term and one LDS
// read instead of the 30 of exp64; bound by the vector units.  Resampling 48 fp32 rows of 151936: 53.7 us by
// exp64, 29.9 so.  A bit table for binary16 (14336 values in 112 KB) costs as much
// as 100000 terms to build, and its gain on longer rows (40 x 5, V = 152064: 32.9 / 29.2 us) is lost twice over where
// a row's bulk lies near 0, outside it (32.8 / 59.9).
//
// Values below the range are the ordinary case: masks of a type's lowest value, or -1e9.  8 x 9 rows of 128255 with the last
// five masked: 67.6 us (fp32) and 50.9 (bfloat16) where one such value asked for the second sweep, 27.2 and 21.0 so; nine
// tenths of the row masked 69.7 and 74.9, 27.1 and 45.6; nothing masked 26.7 and 20.3.
constexpr float kTabMaxS = 600.0f;
constexpr double kSomeMass = 1e-238;      // e^-546: terms below e^-600, 2^31 of them, are less than an ulp beside it
template <typename T> struct ExpTab {
  static constexpr bool kHas = false;
  static constexpr size_t kBytes = 0;
};
template <> struct ExpTab<Bf16> {
  static constexpr bool kHas = true;
  static constexpr int kLo = (127 - 14) << 7;      // bits of the smallest magnitude covered
  static constexpr int kSpan = 21 << 7;            // magnitudes covered
  static constexpr int kEntries = 2 * kSpan;
  static constexpr size_t kBytes = size_t(kEntries + 2) * sizeof(double);
  static constexpr float kMaxAbs = 128.0f;
  static constexpr uint32_t kInf = 0x7F80u;
  static __device__ __forceinline__ float widen(uint32_t bits) { return __uint_as_float(bits << 16); }
};
template <> struct ExpTab<F16> {
  static constexpr bool kHas = true;
  static constexpr int kLo = (15 - 2) << 10;
  static constexpr int kSpan = 7 << 10;
  static constexpr int kEntries = 2 * kSpan;
  static constexpr size_t kBytes = size_t(kEntries + 2) * sizeof(double);
  static constexpr float kMaxAbs = 32.0f;
  static constexpr uint32_t kInf = 0x7C00u;
  static __device__ __forceinline__ float widen(uint32_t bits) { return f16_lo(bits); }
};
// Whether a launch may make its terms through the bit table: every entry's |s| is within the range.
template <typename T> inline bool exp_table_usable(float rT) {
  if constexpr (ExpTab<T>::kHas) return ExpTab<T>::kMaxAbs * rT <= kTabMaxS;
  return false;
}

// Fills the table with all `threads` threads of the workgroup; the caller synchronises.  `half` 0 / 1 fills the
// first / second half only (a kernel that has requests to make between the two does so: the entries are
// pure arithmetic, a good thing to have while data travels), -1 everything.  A magnitude's two entries lie side by side and are made
// together (exp64_pair; one by one bfloat16's table took 3.0 us of a round's kernel, 1.7 so).
template <typename T> __device__ __forceinline__ void build_exp_table(double* table, float rT, int threads, int half = -1) {
  using TB = ExpTab<T>;
  const int mid = ((TB::kSpan / 2 + threads - 1) / threads) * threads;
  const int lo = half == 1 ? mid : 0, hi = half == 0 ? mid : TB::kSpan;
  for (int j = lo + threadIdx.x; j < hi; j += threads)
    exp64_pair(double(__fmul_rn(TB::widen(uint32_t(TB::kLo + j)), rT)), table[1 + 2 * j], table[2 + 2 * j]);
  if (half != 1 && threadIdx.x == 0) table[0] = table[TB::kEntries + 1] = __longlong_as_double(0x7FF8000000000000ll);
}

// Sum of exp(s) over the 8 elements of a 16-bit vector through the table.  The index arithmetic runs on
// both halves of a 32-bit word at once (16-bit lanes: rotate, saturating subtract, minimum).  An element
// outside the table's domain reads a NaN entry, which shows in the sum: table_vec_sum_raw returns that NaN
// (so that a caller can add several vectors up and look once), table_vec_redo evaluates a vector element by
// element.
typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));
template <typename T>
__device__ __forceinline__ double table_vec_sum_raw(const uint4& d, const double* table) {
  using TB = ExpTab<T>;
  const uint32_t w[4] = {d.x, d.y, d.z, d.w};
  const ushort2_t base = {uint16_t(2 * TB::kLo - 1), uint16_t(2 * TB::kLo - 1)};
  const ushort2_t top = {uint16_t(TB::kEntries + 1), uint16_t(TB::kEntries + 1)};
  const ushort2_t one = {1, 1}, fifteen = {15, 15};
  double s0 = 0.0, s1 = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const ushort2_t x = __builtin_bit_cast(ushort2_t, w[k]);
    const ushort2_t rot = (x << one) | (x >> fifteen);            // sign into bit 0 of each half
    ushort2_t i2 = __builtin_elementwise_sub_sat(rot, base);
    i2 = __builtin_elementwise_min(i2, top);
    if constexpr (TB::kBytes <= 65536) {      // byte offsets fit the 16-bit lanes
      const ushort2_t three = {3, 3};
      const uint32_t off = __builtin_bit_cast(uint32_t, i2 << three);
      const char* tb = reinterpret_cast<const char*>(table);
      const double t0 = *reinterpret_cast<const double*>(tb + (off & 0xFFFFu));
      const double t1 = *reinterpret_cast<const double*>(tb + (off >> 16));
      s0 = k == 0 ? t0 : s0 + t0;
      s1 = k == 0 ? t1 : s1 + t1;
    } else {
      const uint32_t ix = __builtin_bit_cast(uint32_t, i2);
      const double t0 = table[ix & 0xFFFFu], t1 = table[ix >> 16];
      s0 = k == 0 ? t0 : s0 + t0;
      s1 = k == 0 ? t1 : s1 + t1;
    }
  }
  return s0 + s1;
}
// Every element of a vector directly; branch-free, so that a wave in which some lane comes here for every
// vector (a row with many values outside the table) runs at the pace of the direct path and not at that of
// a divergent loop.  flags: as of run_sum, below
template <typename T>
__device__ __forceinline__ double table_vec_redo(const uint4& d, float rT, int& flags) {
  using TB = ExpTab<T>;
  const uint32_t w[4] = {d.x, d.y, d.z, d.w};
  double s = 0.0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint32_t b = (w[e >> 1] >> ((e & 1) * 16)) & 0xFFFFu;
    const float sv = __fmul_rn(TB::widen(b), rT);
    flags |= ((b & 0x7FFFu) > TB::kInf || b == TB::kInf) ? 1 : 0;
    flags |= sv > kTabMaxS ? 2 : (sv < -kTabMaxS ? 4 : 0);
    s += exp64(double(sv));                                       // -inf gives exactly 0
  }
  return s;
}
__device__ __forceinline__ float max3_nan(float a, float b, float c) {      // v_maximum3_f32: a NaN among them is kept
  return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c);
}

// How a sweep makes its terms.  begin() asks for what comes from memory and finish() fills the LDS table (all threads of the
// workgroup, the caller synchronises; `half` as for build_exp_table, where a table is made in two); run_sum() gives the sum over a wave's run, of which every lane
// holds kSegVecs vectors (vector i is vector vbase + 64 i of the row and counts if that is below nvec), and
// raises flags: 1 = NaN or +inf among the elements, 2 = the row has to be swept by its maxima (which finds NaN
// and +inf for itself), 4 = so it has if the row turns out to hold nothing above the range's lower end.
template <typename T> struct BitTerms {
  using Walked = BitTerms<T>;
  static constexpr bool kBits = true;
  static constexpr size_t kBytes = ExpTab<T>::kBytes;
  struct Early {};
  static __device__ __forceinline__ Early begin() { return {}; }
  static __device__ __forceinline__ void first_half(double* table, float rT) { build_exp_table<T>(table, rT, kRowThreads, 0); }
  static __device__ __forceinline__ void finish(double* table, Early, float rT, int half) { build_exp_table<T>(table, rT, kRowThreads, half); }
  // (the four vectors' look-ups go out together and one look at their total says whether a value was outside
  // the table)
  static __device__ __forceinline__ double run_sum(const uint4 (&q)[kSegVecs], uint32_t vbase, uint32_t nvec,
                                                   const double* table, float rT, int& flags) {
    double sv[kSegVecs];
#pragma unroll
    for (int i = 0; i < kSegVecs; ++i) sv[i] = table_vec_sum_raw<T>(q[i], table);
#pragma unroll
    for (int i = 0; i < kSegVecs; ++i) sv[i] = vbase + i * 64 < nvec ? sv[i] : 0.0;
    double acc = (sv[0] + sv[1]) + (sv[2] + sv[3]);
    if (acc != acc) {
      acc = 0.0;
#pragma unroll
      for (int i = 0; i < kSegVecs; ++i)
        if (vbase + i * 64 < nvec) acc += sv[i] == sv[i] ? sv[i] : table_vec_redo<T>(q[i], rT, flags);
    }
    return wave_sum_f64(acc);
  }
};
template <typename T, bool kCopied = true> struct PowTerms {
  using Walked = PowTerms<T, false>;      // for kernels that go from row to row
  static constexpr bool kBits = false;
  static constexpr size_t kBytes = size_t(kPowEntries) * sizeof(uint64_t);
  // (Copied: made by each workgroup for itself, two entries a thread, the table took 1.0 us of a round's kernel and a fifth of the vector
  // instructions of a row of 20000.)
  // Not where a kernel goes from row to row, with the table made once: 64 binary16 trees <2,2,2> of 32000, the path, 38.5 us made, 39.5 copied.
  struct Early { uint4 two; };
  static_assert(kPowEntries == 2 * kRowThreads, "two entries a thread");
  static __device__ __forceinline__ Early begin() {
    if constexpr (kCopied) return {load_vec(reinterpret_cast<const uint4*>(kPowTable) + threadIdx.x)};
    return {};
  }
  static __device__ __forceinline__ void first_half(double*, float) {}
  static __device__ __forceinline__ void finish(double* table, const Early& e, float, int) {
    if constexpr (kCopied) {
      reinterpret_cast<uint4*>(table)[threadIdx.x] = e.two;
    } else {
      uint64_t* t = reinterpret_cast<uint64_t*>(table);
      for (int i = threadIdx.x; i < kPowEntries; i += kRowThreads) t[i] = pow_entry(i);
    }
  }
  // A term is made of max(s, -690), so that masked elements (-inf) need no branch: what they and other far ones
  // add, 2e-300 each, is nothing beside any s >= -kTabMaxS.  A run without such an s counts as 0.
  static __device__ __forceinline__ double run_sum(const uint4 (&q)[kSegVecs], uint32_t vbase, uint32_t nvec,
                                                   const double* table, float rT, int& flags) {
    constexpr int E = ElemTraits<T>::kPerVec;
    const uint64_t* t = reinterpret_cast<const uint64_t*>(table);
    double acc = 0.0;
    float top = -INFINITY;
#pragma unroll
    for (int i = 0; i < kSegVecs; ++i) {
      float v[E];
      unpack_scaled<T>(q[i], rT, v);
      double s0 = 0.0, s1 = 0.0;
#pragma unroll
      for (int e = 0; e < E; e += 2) {
        const float a = v[e], b = v[e + 1];
        top = max3_nan(a, b, top);
        const double ta = pow_exp(__builtin_amdgcn_fmed3f(a, -690.0f, 690.0f), t);
        const double tb = pow_exp(__builtin_amdgcn_fmed3f(b, -690.0f, 690.0f), t);
        s0 = e == 0 ? ta : s0 + ta;
        s1 = e == 0 ? tb : s1 + tb;
      }
      acc += vbase + i * 64 < nvec ? s0 + s1 : 0.0;
    }
    flags |= top <= kTabMaxS ? 0 : 2;                   // NaN too
    const double sum = wave_sum_f64(acc);
    const bool below = sum < 1e-262;                    // (the same in all lanes; e^-600 is 2.7e-261)
    flags |= below ? 4 : 0;
    return below ? 0.0 : sum;
  }
};

// A table beyond the LDS that a launch may ask for without leave.
template <typename Terms> constexpr bool kLargeTable = Terms::kBytes > 48 * 1024;

template <typename T> __device__ __forceinline__ float dword_element(uint32_t w, int i);
template <> __device__ __forceinline__ float dword_element<float>(uint32_t w, int) { return as_f32(w); }
template <> __device__ __forceinline__ float dword_element<Bf16>(uint32_t w, int i) { return as_f32(i ? w & 0xFFFF0000u : w << 16); }
template <> __device__ __forceinline__ float dword_element<F16>(uint32_t w, int i) { return i ? f16_hi(w) : f16_lo(w); }

// What a sweep is handed of the table: that it has been asked for (Terms::Early), or this, to ask for it with the row.  (fp32's kernels of
// 64 registers spill where it waits through what comes before the sweep: 24 trees <2,2,2> of 151936, sets of 1024, 65.4 us asked for with the
// row, 67.2 before it.)
struct AskWithRow {};
template <typename Terms> __device__ __forceinline__ typename Terms::Early table_asked(const typename Terms::Early& asked) { return asked; }
template <typename Terms> __device__ __forceinline__ typename Terms::Early table_asked(AskWithRow) { return Terms::begin(); }

// ---------------------------------------------------------------------------------------------
// The row.  Its mass is held in "items", in row order: the elements before the aligned body, every run of the
// body, the elements after it.  All sixteen waves sweep; what comes between the sweep and the search for the
// element is a chain of short dependent steps over a few hundred set entries.  The waves that hold entries, one a lane, make the
// tests and updates out of registers and leave their sums for each other, a barrier a stage; whatever all of them need they make
// each for itself.  The others wait, and the search is the first wave's alone (with redundant steps spread over sixteen waves an
// instruction costs sixteen issue slots).  us of a round's kernel, one binary16 row of 32000 with 320 entries: the tests by the first wave,
// four entries a lane at a time out of LDS, 1.28, so 0.7.
// ---------------------------------------------------------------------------------------------
struct RowShared {
  double items[kMaxItems];
  // the received set: token index (-1 outside the vocabulary), mass of the row at it, correction to that mass
  double set_e[kRowThreads], set_a[kRowThreads];
  int set_y[kRowThreads];
  double w_part[kRowWaves], e_part[kRowWaves];      // sums of weights and masses over the entries that a wave holds
  // what the waves leave of a test (two buffers: a wave may be at the next one), by stage whether one of them has found the candidate
  double t_part[2][kRowWaves], t_shared[2][kRowWaves], t_ratio[2][kRowWaves], t_q[2][kRowWaves];
  int found[kMaxStages];
  double wave_sum[kRowWaves];
  float wave_max[kRowWaves];
  double target, before;
  int flags, next_run, item, n_corr, pick, cmd, st, fetched, claim, stop_at;
};

template <typename T> struct RowWork {
  const void* row;
  RowSplit rs;
  int64_t V;
  float rT;
  int n_runs, n_items;
  int count;            // entries of the received set
  int y;                // this thread's entry: token index (-1: none), payload, target logit
  float ql, ql0, tv;
  double wt, e, a;      // ... its weight, the row's mass at it, and after an update the distribution at it
  float smax;           // the reference of the masses
};

// A residual of no more than this share of the row's mass is none: what is left to draw from, or to test the next
// candidate against, stays the distribution that it was taken from.  The masses are sums of terms within 1.5 ulp through
// about thirty additions on the longest way (a lane's terms, the wave, the items), the set's part of them of terms within
// an ulp through twenty: where the two should cancel they leave up to 6e-15 of the row.  (The least that a rejection of a
// token of the set leaves is the share 2^-24 of its q_hat.)
constexpr double kNoResidual = 0x1p-47;

// What the waves that hold entries know of the row (the same in all of them).
struct RowState {
  double zp, sum_e;     // total mass, the set's part of it
  double inv_zp;        // 1 / total mass: p is set_e * inv_zp before the first update
  double inv_w;         // 1 / sum of the set's weights: q_hat is set_w * inv_w, a stage's proposal q_hat * qscale
  double p_out, c, sum_a, qscale;
  double removed;       // q_hat of the candidates that have left the proposal
  int st, stages;
  bool ok;
};

template <typename T>
__device__ __forceinline__ void row_open(RowWork<T>& w, const void* row, int64_t V, float rT, RowShared& sh) {
  w.row = row;
  w.rs = split_row<T>(row, V);
  w.V = V;
  w.rT = rT;
  w.n_runs = int((w.rs.nvec + kRunVecs - 1) / kRunVecs);
  w.n_items = w.n_runs + 2;
  // (published by the sweep's first barrier)
  if (threadIdx.x == 0) { sh.flags = 0; sh.next_run = kRowWaves; sh.stop_at = 0; }
  if (threadIdx.x < kMaxStages) sh.found[threadIdx.x] = 0;
}

// This thread's entry of a received set; every request is unconditional (a slot beyond the set reads the set's
// last slot).
template <typename T>
__device__ __forceinline__ void row_take_set(RowWork<T>& w, const int32_t* qi, const float* ql, int count, int k_cap) {
  const int tid = threadIdx.x;
  const int slot = tid < k_cap ? tid : k_cap - 1;
  w.y = qi[slot];
  w.ql = ql[slot];
  w.ql0 = ql[0];
  w.count = count < 0 ? 0 : (count > k_cap ? k_cap : count);
}
// ... and the target logit at its index: a dependent request, to be made when the index has had time to arrive.
template <typename T> __device__ __forceinline__ void row_gather(RowWork<T>& w) {
  const bool valid = int(threadIdx.x) < w.count && w.y >= 0 && w.y < w.V;
  w.y = valid ? w.y : -1;
  w.tv = load_elem<T>(w.row, valid ? w.y : 0);
}
// The entry's weight and mass, and their sums.  A value that is not finite or an index outside the vocabulary makes the
// set unusable: the weight is NaN, which shows in the sum.
template <typename T> __device__ __forceinline__ void row_store_set(RowWork<T>& w, float smax, RowShared& sh) {
  const int tid = threadIdx.x;
  w.wt = w.e = 0.0;
  if (__builtin_amdgcn_readfirstlane(wave_id() * 64) < w.count) {       // whole waves
    if (tid < w.count) {
      w.wt = fabsf(w.ql) < INFINITY && w.y >= 0 ? exp64(double(w.ql) - double(w.ql0)) : __longlong_as_double(0x7FF8000000000000ll);
      w.e = w.y >= 0 && w.tv > -INFINITY ? exp64(double(__fmul_rn(w.tv, w.rT)) - double(smax)) : 0.0;
      sh.set_y[tid] = w.y;
      sh.set_e[tid] = w.e;
    }
    double sums[2] = {w.wt, w.e};
    wave_sums_f64(sums);
    if (lane_id() == 0) { sh.w_part[wave_id()] = sums[0]; sh.e_part[wave_id()] = sums[1]; }
  }
}
// Waves that hold entries (one, if there are none).
template <typename T> __device__ __forceinline__ int row_set_waves(const RowWork<T>& w) {
  return __builtin_amdgcn_readfirstlane(w.count > 64 ? (w.count + 63) / 64 : 1);
}

// The masses of the row's items, referenced to 0: of its runs run0 .. run1 - 1, and with `ends` of the elements before and
// after its aligned body; and sh.flags, as of run_sum.  A wave takes run run0 + `wave` first and then whichever run is next (a counter in
// LDS), so that the waves end together.  Every request of the loop is unconditional (a vector past the row's end
// is read from the row's last vector, or as zeros, and its sum dropped; a run past the part's last likewise, to no
// effect): with requests inside branches the number in flight is not known where a wait is placed, and the wait
// for the current run would wait for the run requested ahead as well.  While the first requests travel the terms'
// table is made: all of it (half -1), its second half (1) or nothing (-2).
// The elements outside the aligned body, one per lane of the last wave; their masses, referenced to m.
template <typename T> __device__ __forceinline__ bool row_edge_lane(const RowWork<T>& w) {
  return wave_id() == kRowWaves - 1 && lane_id() < w.rs.head + w.rs.tail;
}
template <typename T> __device__ __forceinline__ void row_edges(const RowWork<T>& w, float edge_v, float m, RowShared& sh) {
  const int lane = lane_id();
  const double t = row_edge_lane(w) ? exp64(double(__fmul_rn(edge_v, w.rT)) - double(m)) : 0.0;
  const double head = wave_sum_f64(lane < w.rs.head ? t : 0.0), tail = wave_sum_f64(lane < w.rs.head ? 0.0 : t);
  if (lane == 0) { sh.items[0] = head; sh.items[w.n_items - 1] = tail; }
}
// How PowTerms' rows are loaded: streamed past the caches through a buffer; and of fp32 rows, through a buffer into the caches, or by
// address.  A row that an earlier launch of the call has read may still be in a cache, but streaming keeps room for the ones that
// wait: the sampled rows of chains are better streamed in batches that fit the Infinity Cache (us streamed / cached: 400 x 4 fp32
// rows of 16000 30.9 / 32.3, 256 x 5 of 32000 36.5 / 37.8, 200 x 2 of 100000 38.6 / 39.7; 130 x 4 of 151936 70.6 / 69.8, 300 x 3 117.2 /
// 111.8, 512 x 2 of 100000 80.1 / 76.2) or where they do not fit it themselves (512 x 2 of 256000 175.8 / 181.7), those of quick walks up to more than that (64 trees <4,2> of 152064 61.5 / 62.2, 512 <1,1,1,1> of
// 32000 79.2 / 80.5; 512 of 64000 119.7 / 116.7, 400 <4,2> of 99968 112.2 / 108.0, 80 <3,3> of 256000 87.9 / 83.5).  A walk over
// rows of a run or two a wave is faster by address (streamed / so: 400 trees <4,2> of 20000 48.7 / 46.5, 1000 <3> of 32000 83.2 / 82.0, of
// 64000 118.2 / 121.2).
enum { kStreamed = 0, kCached = 1, kByAddress = 2 };
constexpr int64_t kStreamBytes = int64_t(256) << 20, kCachedBytes = int64_t(400) << 20, kStreamTreeBytes = int64_t(600) << 20;
constexpr int64_t kByAddressV = 48000;
template <typename T, typename Terms, bool kOneCopy = false, int kLoads = kStreamed, bool kPart = false, typename Asked>
__device__ __forceinline__ void row_pass(RowWork<T>& w, double* table, int half, const Asked& asked, int run0, int run1, bool ends, RowShared& sh) {
  const int lane = lane_id(), wave = wave_id();
  const RowSplit& rs = w.rs;
  const float rT = w.rT;
  int flags = 0;
  float edge_v = -INFINITY;
  if (ends && row_edge_lane(w)) {
    edge_v = load_elem<T>(w.row, edge_index<T>(rs, lane));
    flags |= (edge_v != edge_v || edge_v == INFINITY) ? 1 : 0;
    const float s = __fmul_rn(edge_v, rT);
    flags |= s > kTabMaxS ? 2 : (s < -kTabMaxS ? 4 : 0);
  }
  if (run0 < run1) {
    const uint32_t last_vec = uint32_t(rs.nvec - 1), nvec = uint32_t(rs.nvec);
    // (PowTerms: through a buffer, which takes the addresses out of the vector registers, streams past the caches and gives
    // zeros past the row's end; with 64 registers a thread the sweep spills less.  Two fp32 trees of 1365 nodes, V = 151936,
    // every node: 322 us by plain loads, 302 so; 60 binary16 trees <4,2,2,1> of 32000 94 and 86; 24 x 5 binary16 rows of 55257
    // 19.4 and 18.5.  BitTerms, bound by the LDS, gain nothing: 64 bfloat16 trees <2,2,2> of 128256 57 and 63.)
    // (A workgroup's row, a wave's run: said so, where the compiler cannot tell and would put a loop around each load.  64
    // binary16 trees <2,2,2> of 32000, the path: 40.3 us with the loops, 39.5 without.)
    const uint64_t row_at = reinterpret_cast<uint64_t>(rs.body);
    const uint32_t row_lo = __builtin_amdgcn_readfirstlane(uint32_t(row_at)), row_hi = __builtin_amdgcn_readfirstlane(uint32_t(row_at >> 32));
    // (A part's buffer ends where the part does: what lies behind is the next workgroup's, and the run that a wave requests
    // ahead of its last one would be fetched to be dropped.  48 x 6 fp32 rows of 151936, five parts of 30 runs each:
    // the sampled rows took 20.5 MB from memory and 10.1 us so, 14.3 and 9.9 now.)
    const uint32_t end_vec = kPart ? std::min(nvec, uint32_t(run1) * kRunVecs) : nvec;
    const __amdgpu_buffer_rsrc_t body =
        row_buffer(reinterpret_cast<const uint4*>((uint64_t(row_hi) << 32) | row_lo), uint32_t(__builtin_amdgcn_readfirstlane(end_vec)));
    auto request = [&](int run, uint4 (&q)[kSegVecs]) {
      if constexpr (!Terms::kBits && !(kLoads == kByAddress && ElemTraits<T>::kBytes == 4)) {
        const uint32_t at = uint32_t(__builtin_amdgcn_readfirstlane(run)) * (kRunVecs * 16u);
#pragma unroll
        for (int i = 0; i < kSegVecs; ++i)
          q[i] = kLoads == kCached ? buffer_load_vec(body, lane * 16u, at + i * 1024u) : buffer_load_vec_stream(body, lane * 16u, at + i * 1024u);
      } else {
        const uint32_t vbase = uint32_t(run < run1 ? run : run1 - 1) * kRunVecs + lane;
#pragma unroll
        for (int i = 0; i < kSegVecs; ++i) {
          const uint32_t vi = vbase + i * 64;
          q[i] = load_vec(&rs.body[vi < last_vec ? vi : last_vec]);
        }
      }
    };
    auto consume = [&](int run, const uint4 (&q)[kSegVecs]) {
      const double run_sum = Terms::run_sum(q, uint32_t(run) * kRunVecs + lane, nvec, table, rT, flags);
      if (lane == 0 && run < run1) sh.items[1 + run] = run_sum;
    };
    auto next = [&]() {
      int nr = 0;
      if (lane == 0) nr = atomicAdd(&sh.next_run, 1);
      return run0 + __builtin_amdgcn_readfirstlane(nr);
    };
    uint4 d[kSegVecs], dn[kSegVecs];
    int cur = run0 + wave;
    typename Terms::Early early;
    if (half > -2) early = table_asked<Terms>(asked);  // (before the row: loads are waited for in order)
    request(cur, d);
    if (half > -2) Terms::finish(table, early, rT, half);
    __syncthreads();                    // the table is complete
    // Behind the first run the set entry's target logit is requested, whose index has arrived by then.  kOneCopy: that run is
    // not apart, so that the code of a run (PowTerms of 16-bit rows: 700 instructions) is there once; a second copy, first met by the few
    // waves that take a second run, misses the instruction cache line by line.  Not where registers are short.  11 x 3
    // binary16 rows of 41445 17.9 us with two copies, 16.7 with one; resampling 300 of 128256, 64 registers, 65 and 77.
    int nxt;
    auto step = [&]() {
      nxt = next();
      request(nxt, dn);
      if (cur < run1) consume(cur, d);
    };
    auto advance = [&]() {
#pragma unroll
      for (int i = 0; i < kSegVecs; ++i) d[i] = dn[i];
      cur = nxt;
    };
    if constexpr (Terms::kBits || !kOneCopy || ElemTraits<T>::kPerVec < 8) {
      step();
      row_gather(w);
      advance();
      while (cur < run1) { step(); advance(); }
    } else if (run1 - run0 <= kRowWaves) {
      // A run for every wave at most: no counter, and nothing requested behind it, which through the buffer costs more than a
      // row read again would.  1 x 5 binary16 rows of 32000, the round's kernel 12.96 us with the loop, 12.68 so (12.88 by
      // plain loads with the loop); a row meets one of the two copies of the run's code.
      row_gather(w);
      if (cur < run1) consume(cur, d);
    } else {
      bool gathered = false;
      do {
        step();
        if (!gathered) { row_gather(w); gathered = true; }
        advance();
      } while (cur < run1);
    }
  } else {
    if (half > -2) Terms::finish(table, table_asked<Terms>(asked), rT, half);      // (the next row of a walk may have runs)
    __syncthreads();
    row_gather(w);
  }
  if constexpr (!kPart) row_store_set(w, 0.0f, sh);
  if (ends && wave == kRowWaves - 1) row_edges(w, edge_v, 0.0f, sh);
  flags = wave_or_i32(flags);
  if (lane == 0 && flags) atomicOr(&sh.flags, flags);
  __syncthreads();
}
// The masses of all the row's items, referenced to w.smax (0, or the row's maximum where it needs that), and sh.flags
// (bit 0: NaN or +inf).
template <typename T, typename Terms, bool kOneCopy = false, int kLoads = kStreamed, typename Asked>
__device__ __forceinline__ void row_sweep(RowWork<T>& w, double* table, int half, const Asked& asked, RowShared& sh) {
  constexpr int E = ElemTraits<T>::kPerVec;
  row_pass<T, Terms, kOneCopy, kLoads>(w, table, half, asked, 0, w.n_runs, true, sh);
  const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
  const RowSplit& rs = w.rs;
  const int n_runs = w.n_runs;
  const float rT = w.rT;
  w.smax = 0.0f;
  const int seen = __builtin_amdgcn_readfirstlane(sh.flags);
  if (__builtin_expect(seen & 6, 0)) {
    // beyond the range: the row again, in two passes, referenced to its maximum, if it has to be
    if (!(seen & 2)) {
      if (ballot(tid < w.n_items && sh.items[tid] > kSomeMass) != 0 && lane == 0) atomicOr(&sh.flags, 8);
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(sh.flags) & 8) return;
    }
    float vmax = -INFINITY;
    int bad = 0;
    for (int64_t vi = tid; vi < rs.nvec; vi += kRowThreads) {
      float v[E];
      unpack<T>(load_vec(&rs.body[vi]), v);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        bad |= (v[e] != v[e] || v[e] == INFINITY) ? 1 : 0;
        vmax = fmaxf(vmax, v[e]);
      }
    }
    float edge_v = -INFINITY;
    if (row_edge_lane(w)) {
      edge_v = load_elem<T>(w.row, edge_index<T>(rs, lane));
      bad |= (edge_v != edge_v || edge_v == INFINITY) ? 1 : 0;
      vmax = fmaxf(vmax, edge_v);
    }
    vmax = wave_max_f32(vmax);
    bad = wave_or_i32(bad);
    if (lane == 0) { sh.wave_max[wave] = vmax; if (bad) atomicOr(&sh.flags, 1); }
    __syncthreads();
    for (int k = 0; k < kRowWaves; ++k) vmax = fmaxf(vmax, sh.wave_max[k]);
    const float smax = __fmul_rn(vmax, rT);      // scaling is monotone
    if (smax > -INFINITY) {                      // (else nothing is above -inf: every item has been given 0)
      w.smax = smax;
      for (int run = wave; run < n_runs; run += kRowWaves) {
        double acc = 0.0;
        for (int i = 0; i < kSegVecs; ++i) {
          const int64_t vi = int64_t(run) * kRunVecs + i * 64 + lane;
          if (vi < rs.nvec) {
            float v[E];
            unpack<T>(load_vec(&rs.body[vi]), v);
#pragma unroll
            for (int e = 0; e < E; ++e) acc += exp64(double(__fmul_rn(v[e], rT)) - double(smax));    // -inf gives exactly 0
          }
        }
        acc = wave_sum_f64(acc);
        if (lane == 0) sh.items[1 + run] = acc;
      }
      if (wave == kRowWaves - 1) row_edges(w, edge_v, smax, sh);
      row_store_set(w, smax, sh);
    }
    __syncthreads();
  }
}

// One of `parts` workgroups that share a row: the masses of its runs, and the first one's of the elements outside the aligned
// body, left in memory; NaN where it met something that asks for a sweep by the row's maximum.  (The set's target logits are
// gathered on the way, as in row_sweep, by each of them: whoever goes on has them.)
template <typename T, typename Terms, int kLoads, typename Asked>
__device__ __forceinline__ void row_part(RowWork<T>& w, double* table, const Asked& asked, int part, int parts, double* out, RowShared& sh) {
  const int per = (w.n_runs + parts - 1) / parts;
  const int run0 = part * per, run1 = run0 + per < w.n_runs ? run0 + per : w.n_runs;
  row_pass<T, Terms, false, kLoads, true>(w, table, -1, asked, run0, run1, part == 0, sh);
  const bool broken = (sh.flags & 3) != 0;
  const double bad = __longlong_as_double(0x7FF8000000000000ll);
  auto leave = [&](int i) {
    store_through(reinterpret_cast<uint64_t*>(out) + i, uint64_t(__double_as_longlong(broken ? bad : sh.items[i])));
  };
  for (int i = run0 + threadIdx.x; i < run1; i += kRowThreads) leave(1 + i);
  if (part == 0 && threadIdx.x < 2) leave(threadIdx.x == 0 ? 0 : w.n_items - 1);
  w.smax = 0.0f;
  row_store_set(w, 0.0f, sh);                        // (while they travel; each for itself)
}

// The row as row_sweep leaves it, from the masses that its workgroups have left, in the one of them that claims it (which travels with
// the masses).
template <typename T, typename Terms>
__device__ __forceinline__ bool row_fetch(RowWork<T>& w, const double* items, double* table, uint64_t* words, int parts, Tag tag, RowShared& sh) {
  const int tid = threadIdx.x, lane = lane_id();
  const double mass = __longlong_as_double((long long)load_through(reinterpret_cast<const uint64_t*>(items) + (tid < w.n_items ? tid : 0)));
  if (wave_id() == 0) {
    const bool mine = claimed(words, parts, tag);
    if (lane == 0) sh.claim = mine ? 1 : 0;
  }
  if (tid < w.n_items) sh.items[tid] = mass;
  const int seen = (ballot(mass != mass) != 0 ? 1 : 0) | (ballot(mass > kSomeMass) != 0 ? 2 : 0);
  if (tid == 0) sh.flags = 0;                        // (its own part's, looked at before the last barrier)
  if (lane == 0 && seen) atomicOr(&sh.fetched, seen);
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(sh.claim) == 0) return false;
  if (__builtin_amdgcn_readfirstlane(sh.fetched) != 2) {
    if (tid == 0) sh.next_run = kRowWaves;           // (published by the sweep's first barrier)
    row_sweep<T, Terms>(w, table, -1, AskWithRow{}, sh);
  }
  return true;
}
// Both: whether this workgroup goes on with the row.
template <typename T, typename Terms, int kLoads = kStreamed, typename Asked>
__device__ __forceinline__ bool row_shared(RowWork<T>& w, double* table, const Asked& asked, int part, int parts, double* items, uint64_t* words,
                                           Tag tag, RowShared& sh) {
  if (threadIdx.x == 0) sh.fetched = 0;
  row_part<T, Terms, kLoads>(w, table, asked, part, parts, items, sh);
  if (!all_arrived(words, part, parts, tag, sh.cmd)) return false;
  return row_fetch<T, Terms>(w, items, table, words, parts, tag, sh);
}

constexpr int64_t kShareRows = 128;                  // at most, by two workgroups or more
constexpr int64_t kShareLeastV = 40000;              // of any type
// Masses of a row's items, of `per_vec` elements in a vector (as for row_segments).  16-bit rows have lines of memory of their own: what several
// XCDs write of one line goes there several times (8 x 4 binary16 rows of 100000 15.7 us side by side, 15.4 so).
inline int64_t items_stride(int64_t V, int per_vec = 4) {
  const int64_t n = int64_t(row_segments(V, per_vec)) * kSubChunks + 2;
  return per_vec > 4 ? std::min((n + 15) / 16 * 16, items_stride(V)) : n;
}
constexpr int64_t kShareWords = 512;                 // words that the workgroups of all shared rows leave, at most
// Workgroups that share each of `rows` rows (1: none do): as many as fill the chip, with eight runs each at least (a wave alone on its
// SIMD is done with a run in a third of the time that four of them take; fp32 and BitTerms, whose runs cost less: sixteen where eight
// would make more workgroups than half the chip).  Two trips to memory and the terms' table made by every part (some 2 us) against the
// sweep of a row by one compute unit, so rows from the length on where that is more: BitTerms' terms are the cheapest, and
// binary16 has twice fp32's in a run.  us a call by one workgroup a row / shared, chains 1 x 4, 4 x 4, 8 x 8 and two trees <2,2,2>, sets of 256:
//   binary16  32000 12.9 / 13.3, 13.0 / 14.1, 13.4 / 14.4, 15.9 / 16.6;  44000 14.7 / 13.7, 15.2 / 14.3, 15.2 / 14.9, 18.0 / 16.7
//   fp32      32000 12.9 / 12.4, 13.3 / 13.2, 13.5 / 14.4, 15.7 / 15.2;  44000 14.1 / 12.8, 14.8 / 13.5, 14.9 / 14.8, 16.9 / 15.4
//   bfloat16  44000 12.0 / 13.4, 12.5 / 13.6, 12.6 / 14.4, 15.1 / 15.8;  64000 13.1 / 12.6, 13.6 / 13.7, 13.6 / 14.9, 16.4 / 15.8;
//             90000 13.6 / 12.6, 14.7 / 14.1, 14.8 / 15.2, 17.9 / 16.2
// By sixteen runs a part / eight: binary16 64000 15.0 / 13.2, 16.3 / 14.0, 16.5 / 15.8; fp32 64000 13.3 / 12.6, 14.1 / 14.5, 90000 (4 x 4)
// 14.7 / 15.6, bfloat16 200000 15.7 / 16.3.  Sets of 16 and 1024: bfloat16 64000, 1 x 4 12.8 / 12.9 and 15.6 / 15.1, 5 x 4 13.0 / 13.1 and 15.7 / 15.3; fp32
// 44000 1 x 4 14.0 / 12.1 and 16.4 / 14.0; binary16 44000 8 x 8 15.1 / 14.3 and 17.5 / 16.8.  (Every part reads the set and gathers the row at it, so that the one
// that goes on has it at once: gathered by that one alone, behind the masses, sets of 1024 take 0.3 to 1.4 us more.)
// By two workgroups a row (more than a third as many rows as compute units) later; 16 x 7, 20 x 4 and the sampled rows of 128 x 4, sets of 256:
//   fp32      60000 17.0 / 18.2, 16.9 / 16.9, 39.5 / 40.9;  76000 19.3 / 19.8, 19.1 / 18.4, 46.2 / 46.9;  90000 20.7 / 20.6, 20.6 / 19.1, 53.4 / 53.2;
//             120000 24.3 / 23.1, 24.0 / 21.1, 62.9 / 61.9;  sets of 1024: 76000 21.5 / 22.6, 21.4 / 20.4, 55.4 / 54.9;  120000 26.8 / 27.5, 26.4 / 24.4, 73.1 / 71.0
//   bfloat16  125000 17.2 / 17.6, 17.1 / 17.0, 40.6 / 41.5;  150000 18.7 / 18.8, 18.7 / 17.9, 46.0 / 46.5;  180000 20.4 / 19.9, 20.4 / 18.5, 52.0 / 52.2;
//             sets of 1024: 150000 21.2 / 21.6, 21.3 / 19.9, 55.4 / 54.8
//   binary16  52000 16.2 / 16.7, 16.3 / 16.6, 29.2 / 29.3;  60000 17.9 / 16.9, 17.8 / 16.8, 31.6 / 31.1;  72000 18.8 / 18.7, 18.8 / 18.5, 34.1 / 34.3;
//             sets of 1024: 60000 20.2 / 19.5, 20.1 / 19.0, 39.3 / 38.5;  by the bit table 128 x 2 147456 36.6 / 36.2, 100 x 4 43.3 / 42.6
template <typename T, typename Terms> inline int64_t share_min_V(int64_t rows) {
  const int64_t cus = compute_units();
  const bool by_two = 3 * rows > cus;
  if (ElemTraits<T>::kBytes == 4) return by_two ? 76000 : (4 * rows > cus ? 50000 : kShareLeastV);
  if (kLargeTable<Terms>) return 100000;
  if (Terms::kBits) return by_two ? 150000 : (8 * rows > cus ? 100000 : 64000);
  return by_two ? 60000 : kShareLeastV;
}
template <typename T, typename Terms> inline int row_parts(int64_t V, int64_t rows) {
  if (rows > kShareRows || V < share_min_V<T, Terms>(rows)) return 1;
  const int64_t cus = std::min<int64_t>(compute_units(), kShareWords);
  const int64_t runs = V / (ElemTraits<T>::kPerVec * kRunVecs) + 1;
  int64_t parts = (runs + 7) / 8;
  if ((ElemTraits<T>::kBytes == 4 || Terms::kBits) && 2 * rows * parts > cus) parts = (runs + kRowWaves - 1) / kRowWaves;
  return int(std::max<int64_t>(1, std::min(cus / rows, std::min<int64_t>(parts, 64))));
}

// The waves that hold entries, each for itself: normaliser, and what p and q_hat at the set are made with.  A row that holds NaN
// or +inf, or nothing above -inf, is unusable.
template <typename T> __device__ __forceinline__ void row_eval(const RowWork<T>& w, RowState& r, RowShared& sh) {
  const int lane = lane_id();
  const int n_stored = (w.count + 63) / 64;        // waves that stored entries
  double sum_w = lane < n_stored ? sh.w_part[lane & 15] : 0.0, sum_e = lane < n_stored ? sh.e_part[lane & 15] : 0.0;
  double zp = 0.0;
  for (int i0 = lane; i0 < w.n_items; i0 += 256) {
    double t[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) t[k] = i0 + 64 * k < w.n_items ? sh.items[i0 + 64 * k] : 0.0;
    zp += (t[0] + t[1]) + (t[2] + t[3]);
  }
  double sums[3] = {zp, sum_w, sum_e};
  wave_sums_f64(sums);
  r.zp = sums[0];
  sum_w = sums[1];
  r.sum_e = sums[2];
  r.st = (sh.flags & 1) ? 1 : (r.zp > 0.0 ? 0 : 2);
  r.ok = r.st == 0;
  if (sum_w != sum_w) { r.st |= kRowBadSet; r.ok = false; }
  // (one reciprocal each instead of a division per entry: an fp64 division is some thirty instructions)
  r.inv_zp = r.ok ? 1.0 / r.zp : 0.0;
  r.inv_w = sum_w > 0.0 ? 1.0 / sum_w : 0.0;
  r.sum_a = r.sum_e * r.inv_zp;
  r.p_out = 1.0 - r.sum_a > 0.0 ? 1.0 - r.sum_a : 0.0;
  r.c = 1.0;
  r.qscale = 1.0;
  r.removed = 0.0;
  r.stages = 0;
}

// The test of candidate x against the distribution as it stands and the stage's proposal: its ratio (-1 if x is not in the
// set), the mass the two share (sum of their minima), and what an update needs.  The waves that hold entries leave their sums
// (row_test) and take up the total of all behind a barrier (row_tested).
struct RowTest {
  double ratio, shared, part, q_x;
  bool found;
};
template <typename T> __device__ __forceinline__ double row_at(const RowWork<T>& w, const RowState& r) { return r.stages ? w.a : w.e * r.inv_zp; }
// Returns the thread's max(0, p - q).
template <typename T>
__device__ __forceinline__ double row_test(const RowWork<T>& w, const RowState& r, int x, int stage, RowShared& sh) {
  const int lane = lane_id(), wave = wave_id(), k = stage & 1;
  const double a = row_at(w, r), qk = w.wt * r.inv_w, q = qk * r.qscale;
  const double d = a - q > 0.0 ? a - q : 0.0;
  const bool valid = w.y >= 0;
  double sums[2] = {valid ? d : 0.0, valid ? a - d : 0.0};      // the second: min(a, q)
  wave_sums_f64(sums);
  if (lane == 0) { sh.t_part[k][wave] = sums[0]; sh.t_shared[k][wave] = sums[1]; }
  const bool mine = valid && w.y == x && qk > 0.0;
  const uint64_t at = ballot(mine);
  if (at != 0 && lane == 63 - __clzll((long long)at)) {
    sh.t_ratio[k][wave] = a / q;
    sh.t_q[k][wave] = qk;
    atomicOr(&sh.found[stage], 1 << wave);
  }
  return d;
}
__device__ __forceinline__ RowTest row_tested(int waves, int stage, const RowShared& sh) {
  const int k = stage & 1, found = sh.found[stage];
  RowTest t;
  t.part = sh.t_part[k][0];
  t.shared = sh.t_shared[k][0];
  for (int i = 1; i < waves; ++i) {
    t.part += sh.t_part[k][i];
    t.shared += sh.t_shared[k][i];
  }
  t.found = found != 0;
  const int by = t.found ? 31 - __clz(found) : 0;
  t.ratio = t.found ? sh.t_ratio[k][by] : -1.0;
  t.q_x = t.found ? sh.t_q[k][by] : 0.0;
  return t;
}
template <typename T>
__device__ __forceinline__ int item_of(const RowWork<T>& w, int y) {
  const uint32_t v = uint32_t(y - w.rs.head) / ElemTraits<T>::kPerVec;
  return y < w.rs.head ? 0 : (v >= uint32_t(w.rs.nvec) ? w.n_items - 1 : int(1 + v / kRunVecs));
}
// The mass at the thread's entry becomes `mass`, in units of the row's terms: the item it falls into is corrected by the difference.
template <typename T> __device__ __forceinline__ void row_set_mass(const RowWork<T>& w, double mass, RowShared& sh) {
  if (w.y < 0) return;
  const double corr = mass - w.e;
  sh.set_a[threadIdx.x] = corr;
  atomicAdd(&sh.items[item_of(w, w.y)], corr);
}
// Whether max(0, p - proposal), with the sum over the set that a test returned, holds any mass.
__device__ __forceinline__ bool row_has_residual(const RowState& r, double part) {
  return same_in_wave(part + r.c * r.p_out > kNoResidual * r.c);
}
// p <- norm(max(0, p - proposal)), or p if that holds none; `gone` leaves the proposal (a candidate drawn without
// replacement; -1: none).
template <typename T>
__device__ __forceinline__ void row_update(RowWork<T>& w, RowState& r, double part, int gone) {
  const bool holds = row_has_residual(r, part);
  const double inv_Z = holds ? 1.0 / (part + r.c * r.p_out) : 1.0;
  const double d = row_at(w, r) - w.wt * (holds ? r.inv_w * r.qscale : 0.0);
  w.a = w.y >= 0 && d > 0.0 ? d * inv_Z : 0.0;
  if (w.y == gone && w.y >= 0) w.wt = 0.0;
  r.c *= inv_Z;
  r.sum_a = holds ? part * inv_Z : r.sum_a;
  ++r.stages;
}
// The masses after the updates made so far, and after one more with the sum `part` if it is pending: e_y off the set and
// a * z_p / c on it, in units of the row's terms.  Returns the total of the set's corrections.
template <typename T>
__device__ __forceinline__ double row_correct(const RowWork<T>& w, const RowState& r, bool pending, double part, RowShared& sh) {
  // with one more update a becomes max(0, a - q) / Z and c becomes c / Z: Z drops out of a * z_p / c
  const double zp_over_c = r.zp / r.c;
  const double a = row_at(w, r) - w.wt * (pending ? r.inv_w * r.qscale : 0.0);
  row_set_mass(w, (a > 0.0 ? a : 0.0) * zp_over_c, sh);
  return (pending ? part : r.sum_a) * zp_over_c - r.sum_e;
}
// First wave: the item in which the cumulative mass passes u * total, in row order, and what row_pick needs (item -1:
// there is none).  `corrected`: corrections have been added to the items, `corr` in all, and are in set_a; without them
// nothing has been written there.
template <typename T>
__device__ __forceinline__ void row_locate(const RowWork<T>& w, const RowState& r, float u, bool corrected, double corr,
                                           RowShared& sh) {
  const int lane = lane_id();
  const int n_items = w.n_items;
  double total = corrected ? r.zp + corr : r.zp;
  if (same_in_wave(corrected && !(total > kNoResidual * r.zp))) {      // the items as they were, and p itself
    for (int i = lane; i < w.count; i += 64) {
      const int y = sh.set_y[i];
      if (y >= 0) atomicAdd(&sh.items[item_of(w, y)], -sh.set_a[i]);
    }
    corrected = false;
    total = r.zp;
  }
  const double target = double(u) * total, none = kNoResidual * r.zp;
  if (lane == 0) {
    sh.target = target; sh.n_corr = corrected ? w.count : 0;
    sh.item = sh.pick = -1;
  }
  const int per = (n_items + 63) / 64;               // consecutive items per lane, four at a time
  for (;;) {
    double lsum = 0.0, t0, t1, t2, t3;               // (uniform branches: a row of 64 items or fewer has one a lane)
    auto four = [&](int q) {
      const int it = lane * per + q;
      t0 = it < n_items ? sh.items[it] : 0.0;
      t1 = t2 = t3 = 0.0;
      if (per > 1) {
        t1 = q + 1 < per && it + 1 < n_items ? sh.items[it + 1] : 0.0;
        t2 = q + 2 < per && it + 2 < n_items ? sh.items[it + 2] : 0.0;
        t3 = q + 3 < per && it + 3 < n_items ? sh.items[it + 3] : 0.0;
      }
    };
    for (int q = 0; q < per; q += 4) {
      four(q);
      lsum += t0 > 0.0 ? t0 : 0.0;
      if (per > 1) {
        lsum += t1 > 0.0 ? t1 : 0.0;
        lsum += t2 > 0.0 ? t2 : 0.0;
        lsum += t3 > 0.0 ? t3 : 0.0;
      }
    }
    double run = wave_incl_scan_f64(lsum) - lsum;
    int found = -1, last_pos = -1;
    double found_before = 0.0, last_before = 0.0;
    double found_mass = 0.0, last_mass = 0.0;
    auto look = [&](int it, double t) {
      const bool pos = t > 0.0, hit = pos && run + t > target && found < 0;
      last_pos = pos ? it : last_pos;
      last_before = pos ? run : last_before;
      last_mass = pos ? t : last_mass;
      found = hit ? it : found;
      found_before = hit ? run : found_before;
      found_mass = hit ? t : found_mass;
      run += pos ? t : 0.0;
    };
    for (int q = 0; q < per; q += 4) {
      if (per > 4) four(q);                          // (else they are at hand)
      look(lane * per + q, t0);
      if (per > 1) {
        look(lane * per + q + 1, t1);
        look(lane * per + q + 2, t2);
        look(lane * per + q + 3, t3);
      }
    }
    // the first lane that saw the target passed, else the last one that holds an item with mass
    const uint64_t hit = ballot(found >= 0), any = ballot(last_pos >= 0);
    const int src = hit != 0 ? __ffsll((long long)hit) - 1 : (any != 0 ? 63 - __clzll((long long)any) : 0);
    const int item = __builtin_amdgcn_readlane(hit != 0 ? found : last_pos, src);
    if (item < 0) {                                  // every one has been emptied: p in the last of them
      sh.n_corr = 0;
      return;
    }
    if (lane == src) { sh.item = item; sh.before = hit != 0 ? found_before : last_before; }
    const double mass = lane_f64(hit != 0 ? found_mass : last_mass, src);
    if (same_in_wave(!corrected || mass > none)) return;
    // so little: is it more than what rounding leaves where the corrections take an item's whole mass away?
    double e = 0.0;
    for (int i = lane; i < w.count; i += 64) e += sh.set_y[i] >= 0 && item_of(w, sh.set_y[i]) == item ? sh.set_e[i] : 0.0;
    if (same_in_wave(mass > kNoResidual * wave_sum_f64(e))) return;
    sh.items[item] = 0.0;
  }
}

// All waves: the token, from what row_locate left (behind a barrier): every thread takes one 32-bit word of the run.  (Bound by the fp64
// exponentials' issue: by four waves, a vector a thread, one on each SIMD, 1.25 us; so 0.5.)  `elem_corr`: LDS scratch of one double per
// element of a run (the terms' table, which is not needed any more), set to zero by all threads since (row_clear).
template <typename T> __device__ __forceinline__ void row_clear(double* elem_corr) {
  constexpr int kRun = kRunVecs * ElemTraits<T>::kPerVec;
#pragma unroll
  for (int i = 0; i < kRun / kRowThreads; ++i) elem_corr[threadIdx.x + i * kRowThreads] = 0.0;
}
template <typename T>
__device__ __forceinline__ int row_pick(const RowWork<T>& w, double* elem_corr, RowShared& sh) {
  constexpr int E = ElemTraits<T>::kPerVec;
  constexpr int kRun = kRunVecs * E;               // elements in a run
  constexpr int kOwn = kRun / kRowThreads;         // a thread's, in one word
  static_assert(kOwn * ElemTraits<T>::kBytes == 4, "a thread's share of a run is one word");
  const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
  const RowSplit& rs = w.rs;
  const double smax = double(w.smax), target = sh.target, before = sh.before;
  const int item = __builtin_amdgcn_readfirstlane(sh.item);
  if (item < 0) return -1;
  // the run's first element and its end (an edge: fewer than E elements, walked by one thread)
  const bool edge = item == 0 || item == w.n_items - 1;
  const int e0 = item == 0 ? 0 : rs.head, e1 = item == 0 ? rs.head : rs.head + rs.tail;
  const int64_t first = edge ? edge_index<T>(rs, e0) : rs.head + int64_t(item - 1) * kRun;
  const int64_t end = edge ? first + (e1 - e0) : first + kRun;
  const int64_t word = int64_t(item - 1) * (kRunVecs * 4) + tid;
  const bool inside = !edge && word < rs.nvec * 4;
  uint32_t bits = 0;
  if (inside) bits = as_global(reinterpret_cast<const uint32_t*>(rs.body))[word];      // travels while the corrections are laid out
  if (tid < sh.n_corr) {
    const int y = sh.set_y[tid];
    if (y >= first && y < end) elem_corr[y - first] = sh.set_a[tid];
  }
  __syncthreads();
  if (edge) {
    if (tid == 0) {
      double run_e = before;
      for (int e = e0; e < e1; ++e) {
        const int64_t y = edge_index<T>(rs, e);
        const double v = exp64(double(__fmul_rn(load_elem<T>(w.row, y), w.rT)) - smax) + elem_corr[e - e0];
        if (v > 0.0) {
          sh.pick = int(y);
          run_e += v;
          if (run_e > target) break;
        }
      }
    }
    __syncthreads();
    return sh.pick;
  }
  double v[kOwn], mine = 0.0;
#pragma unroll
  for (int i = 0; i < kOwn; ++i) {
    v[i] = exp64(double(__fmul_rn(dword_element<T>(bits, i), w.rT)) - smax) + elem_corr[tid * kOwn + i];      // -inf gives exactly 0
    v[i] = v[i] > 0.0 && inside ? v[i] : 0.0;
    mine += v[i];
  }
  const double inc = wave_incl_scan_f64(mine);
  if (lane == 63) sh.wave_sum[wave] = inc;
  __syncthreads();
  // the wave in which the cumulative mass passes the target, else the last one with mass, finds the element: the first that passes it,
  // else the last with mass
  const double sum = lane < kRowWaves ? sh.wave_sum[lane & (kRowWaves - 1)] : 0.0;
  const double upto = scan16_f64(sum);
  const uint64_t passes = ballot(sum > 0.0 && before + upto > target), holds = ballot(sum > 0.0);
  if (holds == 0) return -1;
  const int by = passes != 0 ? __ffsll((long long)passes) - 1 : 63 - __clzll((long long)holds);
  if (wave == by) {
    double run_e = before + lane_f64(upto - sum, by) + (inc - mine);
    int first_pass = -1, last_mass = -1;
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
      run_e += v[i];
      last_mass = v[i] > 0.0 ? tid * kOwn + i : last_mass;
      first_pass = v[i] > 0.0 && run_e > target && first_pass < 0 ? tid * kOwn + i : first_pass;
    }
    // (elements ascend with the lane)
    const uint64_t pass = ballot(first_pass >= 0), mass = ballot(last_mass >= 0);
    if (pass != 0 ? lane == __ffsll((long long)pass) - 1 : lane == 63 - __clzll((long long)mass)) sh.pick = pass != 0 ? first_pass : last_mass;
  }
  __syncthreads();
  return int(first + sh.pick);
}

}  // namespace tslt
