// Row-level building block of chain verification in large batches, of the quick walk through a tree and of the statistics:
//   eval_row_on_set  one streaming pass over a target row for its softmax normaliser, then p and
//                    q_hat at the indices of a received sparse set, in fp64;
#pragma once
#include "common.h"
#include "exp64.h"

namespace tslt {

constexpr int kSegVecs = 4;                         // 16-byte vectors per thread in a sweep segment
constexpr int kSegVecsTotal = kSegVecs * kBlock;    // vectors per segment
constexpr int kRunVecs = kSegVecs * 64;             // a run: the consecutive vectors one wave holds
constexpr int kSubChunks = kWaves;                  // runs per segment
// eval_row_on_set keeps kAccDepth batches of kAccVecs 16-byte vectors in flight per thread.  Its kernels ask for
// eight waves per SIMD (64 registers): 2048 rows of the headline shape are then resident at once, eight
// workgroups per compute unit, instead of 1280 followed by a thinly occupied second round.
constexpr int kAccDepth = 4;
constexpr int kAccVecs = 2;
constexpr int kAccWavesPerSimd = 8;
constexpr int kSetPer = 1024 / kBlock;              // set entries per thread (TSLT_MAX_K_CAP / kBlock)

constexpr int kRowBadSet = 8;      // TSLT_ROW_BAD_SET

// Segments of a row of V elements, `per_vec` of them in a 16-byte vector (4 for fp32, the default, which
// bounds every type and sizes the workspaces; 8 for the 16-bit types).
inline int row_segments(int64_t V, int per_vec = 4) {
  // one more segment covers a ragged end
  const int64_t nvec_max = V / per_vec + 1;
  return int((nvec_max + kSegVecsTotal - 1) / kSegVecsTotal);
}
inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

struct VerifyShared {
  BlockScratch red;
  double bcast_d[4];
  int bcast_i[4];
};
// Three sums over the workgroup with one pair of barriers.
template <int NW>
__device__ __forceinline__ void block_sum3_f64(double& a, double& b, double& c, BlockScratch& s) {
  static_assert(3 * NW <= int(sizeof(s.d) / sizeof(s.d[0])), "room for three partial sums a wave");
  a = wave_sum_f64(a); b = wave_sum_f64(b); c = wave_sum_f64(c);
  __syncthreads();
  if (lane_id() == 0) { s.d[wave_id()] = a; s.d[NW + wave_id()] = b; s.d[2 * NW + wave_id()] = c; }
  __syncthreads();
  a = 0.0; b = 0.0; c = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w) { a += s.d[w]; b += s.d[NW + w]; c += s.d[2 * NW + w]; }
}

// ---------------------------------------------------------------------------------------------
// One pass over a target row: partial sums of exp2(t*k2 - c), c referenced to the largest target
// logit found at the set's indices; then, in fp64 over the <= 1024 received entries, p at those
// indices (the set's fp32 terms are replaced by fp64 ones in the normaliser) and q_hat = softmax of
// the received values.  Entry i of the set is held by thread i % NT, slot i / NT (NT threads a workgroup).
//   p_s, q_s  target and draft probability of the entry (0 where the entry is unused)
//   yi        token index of the entry, -1 if unused or out of range
//   p_out     target mass outside the set
//   ok / st   false with TSLT_ROW_* bits when the row is unusable (NaN, +inf, nothing above -inf) or the set is
//             (a value that is not finite, an index outside the vocabulary)
// ---------------------------------------------------------------------------------------------
// log2 of a softmax term relative to the reference c: one fma with k2 = fl32(log2(e) / T).  (The
// definition rounds s = t / T to fp32 first; not doing so here moves a term by at most 2^-24 of its
// exponent, a few 1e-8 of the normaliser after the set's own terms have been replaced by fp64 ones.)
// kFine, for callers that know no other pass over the row: (z / T - s_ref) * log2(e) with log2(e) as a sum, two instructions
// more an element, so that what is left is random per term (the one fma is off by the rounding of k2 in all of them, and by
// that of the reference where a row lies far from 0); and a batch that holds a large term is added up in fp64 (else the
// set's terms, which are taken off again below, leave the rounding of the sums that they went through: 5e-8 of the ratios).
constexpr float kLargeTerm = 0x1p-5f;         // of the reference

template <typename T, bool kFine = false, int NT = kBlock>
__device__ __forceinline__ void eval_row_on_set(const void* row, const RowSplit& rs, int64_t V, float rT, float k2,
                                                const int32_t* qi, const float* ql, int count, VerifyShared& sh,
                                                double (&p_s)[1024 / NT], double (&q_s)[1024 / NT], int (&yi)[1024 / NT],
                                                double& p_out, bool& ok, int& st) {
  constexpr int kPer = 1024 / NT, NW = NT / 64;      // set entries per thread, waves
  auto reference = [&](float v) { return __fmul_rn(v, kFine ? rT : k2); };
  auto arg = [&](float v, float ref) {
    if constexpr (kFine) {
      const float d = __builtin_fmaf(v, rT, -ref);
      return __builtin_fmaf(d, 1.44269502f, __fmul_rn(d, 1.92596299e-8f));
    } else {
      return __builtin_fmaf(v, k2, -ref);
    }
  };
  constexpr int E = ElemTraits<T>::kPerVec;
  const int tid = threadIdx.x;
  const int n_edge = rs.head + rs.tail;
  const int64_t n_tiles = (rs.nvec + NT - 1) / NT;
  // The pass keeps kAccDepth batches of U vectors in flight per thread; the first ones are requested
  // before anything else, so that they travel while the reference is looked up.
  constexpr int U = kAccVecs;
  const uint32_t n_full = uint32_t(rs.nvec / (U * NT));      // batches of U complete tiles
  uint4 pipe[kAccDepth][U];
  // Every request of the pipeline is unconditional: one past the row's end comes back as zeros and is never
  // used.  With conditional requests the number of loads in flight is not known where a wait is placed, and
  // each wait for one batch waits for all of them.
  const __amdgpu_buffer_rsrc_t body = row_buffer(rs.body, uint32_t(rs.nvec));
  const uint32_t lane_bytes = uint32_t(tid) * 16u;
  auto issue = [&](uint32_t b, uint4 (&q)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) q[u] = buffer_load_vec_stream(body, lane_bytes, (b * U + u) * (NT * 16u));
  };
  if (n_full > 0) {
#pragma unroll
    for (int s = 0; s < kAccDepth; ++s) issue(uint32_t(s), pipe[s]);
  }

  float tv[kPer];       // raw target logit at entry
  float gmax = -INFINITY;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = tid + k * NT;
    tv[k] = -INFINITY; yi[k] = -1;
    if (i < count) {
      const int y = qi[i];
      if (y >= 0 && y < V) { yi[k] = y; tv[k] = load_elem<T>(row, y); }
      gmax = fmaxf(gmax, tv[k]);
    }
  }
  float vref = block_max_f32<NW>(gmax, sh.red);
  if (!(vref > -INFINITY && vref < INFINITY)) {
    // no usable reference in the set: take the start of the row
    float m0 = -INFINITY;
    for (int64_t i = tid; i < V && i < 4096; i += NT) m0 = fmaxf(m0, load_elem<T>(row, i));
    vref = block_max_f32<NW>(m0, sh.red);
  }
  st = 0;
  double z_c = 0.0;
  float c_ref = reference(vref);
  ok = vref > -INFINITY && vref < INFINITY;
  if (ok) {
    // fp32 sums only within a batch of U vectors: a long-lived fp32 accumulator that has met one large
    // term rounds away the many small ones that follow, always downwards
    double dacc = 0.0;
    auto consume = [&](const uint4 (&q)[U]) {
      if constexpr (kFine) {
        float t[U * E], sum = 0.0f;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          float v[E];
          unpack<T>(q[u], v);
#pragma unroll
          for (int e = 0; e < E; ++e) t[u * E + e] = fast_exp2(arg(v[e], c_ref));
        }
        float part[4] = {t[0], t[1], t[2], t[3]};
#pragma unroll
        for (int e = 4; e < U * E; ++e) part[e & 3] += t[e];
        sum = (part[0] + part[1]) + (part[2] + part[3]);
        if (ballot(sum > kLargeTerm) != 0) {
          double d = 0.0;
#pragma unroll
          for (int e = 0; e < U * E; ++e) d += double(t[e]);
          dacc += d;
        } else {
          dacc += double(sum);
        }
        return;
      }
      float acc0 = 0.f, acc1 = 0.f, acc2 = 0.f, acc3 = 0.f;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float v[E];
        unpack<T>(q[u], v);
#pragma unroll
        for (int e = 0; e < E; e += 4) {
          acc0 += fast_exp2(arg(v[e + 0], c_ref));
          acc1 += fast_exp2(arg(v[e + 1], c_ref));
          acc2 += fast_exp2(arg(v[e + 2], c_ref));
          acc3 += fast_exp2(arg(v[e + 3], c_ref));
        }
      }
      dacc += double((acc0 + acc1) + (acc2 + acc3));
    };
    for (uint32_t b = 0; b < n_full; b += kAccDepth) {
#pragma unroll
      for (int s = 0; s < kAccDepth; ++s) {
        if (b + s < n_full) consume(pipe[s]);
        issue(b + s + kAccDepth, pipe[s]);
      }
    }
    for (int64_t t0 = int64_t(n_full) * U; t0 < n_tiles; t0 += U) {      // the ragged end
      uint4 d[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t vi = (t0 + u) * NT + tid;
        d[u] = neg_inf_vec<T>();
        if (vi < rs.nvec) d[u] = load_vec_stream(&rs.body[vi]);
      }
      consume(d);
    }
    if (tid < n_edge) dacc += double(fast_exp2(arg(load_elem<T>(row, edge_index<T>(rs, tid)), c_ref)));
    z_c = block_sum_f64<NW>(dacc, sh.red);
    ok = z_c > 0.0 && z_c < INFINITY;
  }
  if (!ok) {
    // exact redo: validity and true maximum first, then the sum referenced to it
    int bad = 0, fin = 0;
    float vmax = -INFINITY;
    for (int64_t i = tid; i < V; i += NT) {
      float v = load_elem<T>(row, i);
      if (v != v || v == INFINITY) bad = 1;
      else if (v > -INFINITY) { fin = 1; vmax = fmaxf(vmax, v); }
    }
    bad = block_sum_i32<NW>(bad, sh.red);
    fin = block_sum_i32<NW>(fin, sh.red);
    vmax = block_max_f32<NW>(vmax, sh.red);
    if (bad) st |= 1;
    else if (!fin) st |= 2;
    else {
      vref = vmax;
      c_ref = reference(vref);
      double acc = 0.0;
      for (int64_t i = tid; i < V; i += NT) acc += double(fast_exp2(arg(load_elem<T>(row, i), c_ref)));
      z_c = block_sum_f64<NW>(acc, sh.red);
      ok = true;
    }
  }

  // ---- fp64 over the set ----------------------------------------------------------------------
  const float s_ref = __fmul_rn(vref, rT);
  const double ql0 = count > 0 ? double(ql[0]) : 0.0;
  double sum_e = 0.0, sum_t32 = 0.0, sum_w = 0.0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = tid + k * NT;
    p_s[k] = 0.0; q_s[k] = 0.0;
    if (i < count) {
      // a received value that is not finite, or a token index outside the vocabulary, makes the set unusable:
      // its weight is NaN, which shows in the sum below
      const float qv = ql[i];
      q_s[k] = (fabsf(qv) < INFINITY && yi[k] >= 0) ? exp64(double(qv) - ql0) : __longlong_as_double(0x7FF8000000000000ll);
      sum_w += q_s[k];
      if (yi[k] >= 0 && tv[k] > -INFINITY && ok) {
        p_s[k] = exp64(double(__fmul_rn(tv[k], rT)) - double(s_ref));
        sum_e += p_s[k];
        sum_t32 += double(fast_exp2(arg(tv[k], c_ref)));
      }
    }
  }
  block_sum3_f64<NW>(sum_e, sum_t32, sum_w, sh.red);
  if (sum_w != sum_w) { st |= kRowBadSet; ok = false; }
  double tail = z_c - sum_t32;
  if (tail < 0.0) tail = 0.0;
  if (!kFine) tail *= exp64((double(c_ref) - double(vref) * double(k2)) * 0.69314718055994530942);   // to the reference of the fp64 terms
  const double Z = tail + sum_e;
  // (one reciprocal each instead of a division per entry: an fp64 division is some thirty instructions)
  const double inv_Z = ok ? 1.0 / Z : 0.0, inv_w = sum_w > 0.0 ? 1.0 / sum_w : 0.0;
  p_out = tail * inv_Z;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    p_s[k] = ok ? p_s[k] * inv_Z : 0.0;
    q_s[k] = sum_w > 0.0 ? q_s[k] * inv_w : 0.0;
  }
}

}  // namespace tslt
