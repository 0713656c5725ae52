// tslt_truncate: Top-K / Top-rho truncation of draft logits (Section 3.1) and compaction to the
// sparse (index, logit) payload of Solution 1 (Section 3.2), one workgroup per row.
//
// One pass over the row.  The row's tiles are visited in batches of kBatch tiles taken at equal
// distances (tile b of every "quarter"), so that the first batch is a strided sample of the row.  From
// that sample a threshold tau0 is chosen that a little more than K elements of the whole row are
// expected to exceed.  The pass then does two things per 16-byte vector: it adds exp2(z*k2 - c) to the
// row's fp32 partial sums (the softmax normaliser, k2 = log2(e)/T, c a reference taken from the
// sample maximum), and, if any element of the vector is above tau0, it parks the vector in a small
// per-wave LDS ring; rings are expanded into (value, index) candidate records when they fill up.  If
// at least K elements were above tau0 the top-K set is among the candidates and is found exactly by
// sorting them; otherwise (ties, masked rows, unlucky sample, overflow of a buffer) the row is redone
// by an exact radix selection that makes several passes.  Either way the kept entries are then
// evaluated in fp64, which is also where Top-rho and the renormalisation are decided.
//
// Bound by memory in large batches (2048 bfloat16 rows of 128256: 91 us, of which 81 are the reading), by the instructions a
// row's waves issue one after the other in small ones.  The pass is written for the second: an fma takes its operands from
// vector registers without a sign to change (2.7 cycles a wave, 4.4 otherwise), binary16 is tested against the threshold as
// packed halves and never widened, addresses are a scalar offset into a buffer (but for large batches), the complete stages have a loop without a
// check for the row's end, and every exchange between waves behind the pass is one barrier (12 in all, 24 before).  Few long rows
// are shared by workgroups (truncate_parts: 64 bfloat16 rows of 128256, k 256, 17.6 us by one each, 16.1 by four).  us
// before / now: 1 binary16 row of 32000, k 320 12.4 / 10.4; 600 binary16 rows of 32000 17.7 / 15.8; 4096 bfloat16 rows of 256000, k 1024 407 / 396.
#pragma once
#include "common.h"
#include "wire.h"
#include "exp64.h"
#include "handover.h"

namespace tslt {

constexpr int kTruncThreads = 256;   // threads of a truncate workgroup (one row each)
constexpr int kBatch = 4;        // tiles of the threshold sample, taken at equal distances over the row
constexpr int kGroup = 2;        // tiles (one 16-byte vector per thread each) in a stage of the pass's pipeline
// The kernel comes in two shapes.  "Wide": two stages in flight per thread and eight waves per SIMD asked of the
// compiler (64 registers), so that eight workgroups share a compute unit; for launches whose LDS footprint
// allows that many (k_cap of a few hundred).  "Deep": four stages in flight and four waves per SIMD; for the
// launches whose candidate arrays leave room for fewer workgroups (k_cap 1024: three per compute unit), which
// then need more requests in flight each to keep the memory busy.
//   "Tall": 512 threads and four stages, for batches that leave the chip to one or two rows per compute unit, bound by
// a row's own latency: twice the requests in flight, rows shorter than the sample's distances through the same pipeline
// (they went pair by pair, a memory latency each), the threshold out of a histogram.  us by 256 / 512 threads: 1 row
// binary16 V = 32000 12.8 / 10.4, 64 bfloat16 V = 128256 24.7 / 17.6, 200 26.2 / 19.0, 384 30.5 / 26.2, 700 38.9 / 38.6;
// 100 fp32 V = 151936 38.1 / 24.4, 400 47.3 / 43.5.  (1024 threads, before the pass and the sort were shortened: slower
// again, 14.9, 23.4 and 25.6 us for the first three, which took 13.0, 21.7 and 23.2 then.)
constexpr int kTallThreads = 512;
constexpr int kStagesWide = 2, kWavesWide = 8;
constexpr int kStagesDeep = 4, kWavesDeep = 4;
// Vectors a wave can park.  256 threads: expanded when there are more than kRingExpand, one pass of 64 lanes, nearly all
// busy; a row in which they come faster than that loses some and is redone.  512: expanded before there would be no
// room for the next ones.
constexpr int kRingSmall = 96, kRingExpand = 58, kRingTall = 64;

struct TruncateParams {
  const void* logits;
  int64_t rows, V, row_stride;
  float rT;          // fl32(1/T)
  float k2;          // fl32(rT * log2(e))
  float top_p;       // 0 = off
  int k_sel;         // min(top_k (if on), k_cap)
  int k_cap;
  int payload;       // 0: the scaled logits as computed; 1 / 2: rounded to bfloat16 / binary16 before q_hat and the draws
  int jprime;        // rank (1-based) among the 256 per-thread sample maxima that gives tau0; 0 = always exact path
  int tau_bits;      // number of leading key bits resolved by the threshold search
  int sort_cap;      // capacity of the candidate array
  int ring_bytes;    // size of the ring space at the start of dynamic LDS
  int32_t* out_idx;
  float* out_logit;
  float* out_prob;
  int32_t* out_count;
  float* out_mass;
  int32_t* status;
  // optional draws from q_hat in the same launch (null u = none)
  int without_replacement;
  const float* u;    // [rows, n_samples]
  int n_samples;
  int32_t* out_token;
  int32_t* out_slot;
  // rows shared by workgroups (handover.h)
  int parts;                 // of a row
  float reach;       // the row's maximum, expected, above the threshold, in units of the sample's
  uint64_t* part_words;      // [rows, parts]
  uint64_t* part_found;      // [rows, parts, 2 + sort_cap]: the sum of its terms, the number of its candidates, those
  Tag tag;
};
// Memory for them: a word and a region of candidates for each workgroup.
constexpr int kTruncMaxParts = 4;
inline size_t truncate_part_bytes(int64_t rows, int64_t parts, int sort_cap) {
  return size_t(rows) * size_t(parts) * (8 + 8 * (2 + size_t(sort_cap))) + 256;
}

// Dynamic LDS: [ rings ] [ candidates ].  The ring space is reused for the sort's table and its scratch records behind it
// and, before the pass, for the per-thread sample maxima.
constexpr int kMaxDraws = 16;      // TSLT_MAX_BRANCH
constexpr int kTablesBytes = 3 * 256 * 4;             // also the few records behind the scratch
static_assert(kTallThreads * 4 + kRankAhead * 8 <= kTablesBytes, "the sort's table and those records");
inline int truncate_sort_scratch(int k_sel) { return k_sel + k_sel / 2 + 64; }   // records the sort may need
inline int truncate_ring_bytes(int n_waves, int k_sel) {
  const int rings = n_waves * (kRingSmall * 20), sort = (kTablesBytes + 8 * truncate_sort_scratch(k_sel) + 15) & ~15;
  return rings > sort ? rings : sort;                                            // per ring slot a vector and its index
}
// (512 threads: the sort's bins behind them, which are cleared before the rings are needed)
inline size_t truncate_lds_bytes(int ring_bytes, int sort_cap, int nt) {
  return size_t(ring_bytes) + size_t(8) * sort_cap + (nt > kTruncThreads ? size_t(4) * nt : 0);
}

struct TruncateShared {
  BlockScratch red;
  int cand_count;
  int overflow;
  float from, upto;      // the threshold, the sample's maximum
  int bcast_i[4];
  double bcast_d[2];
};

// ---------------------------------------------------------------------------------------------
// Exact multi-pass selection, the last resort: the k_eff largest elements of the row in the canonical order, found
// by a 4x8-bit radix search for the k-th largest key and an index-ordered collection of the ties.
// Also recomputes the fp32 sum with the true maximum as reference.  Returns the number of
// candidates written to cand[] (exactly k_eff), or 0 with `st` set.
// ---------------------------------------------------------------------------------------------
template <typename T, int NT>
__device__ __forceinline__ int exact_select(const void* row, int64_t V, int k_sel, float k2, uint64_t* cand, uint32_t* hist,
                            TruncateShared& sh, float& c_ref, double& z_c, int& st) {
  constexpr int NW = NT / 64;
  const int tid = threadIdx.x;
  // pass 1: validity, number of selectable elements, maximum
  int fin = 0, bad = 0;
  float vmax = -INFINITY;
  for (int64_t i = tid; i < V; i += NT) {
    float v = load_elem<T>(row, i);
    if (v != v || v == INFINITY) bad = 1;
    else if (v > -INFINITY) { ++fin; vmax = fmaxf(vmax, v); }
  }
  bad = block_sum_i32<NW>(bad, sh.red);
  fin = block_sum_i32<NW>(fin, sh.red);
  vmax = block_max_f32<NW>(vmax, sh.red);
  if (bad) { st |= 1; return 0; }
  if (fin == 0) { st |= 2; return 0; }
  const int k_eff = k_sel < fin ? k_sel : fin;

  // radix search, most significant digit first, over keys of elements > -inf
  uint32_t prefix = 0;
  int need = k_eff;
  for (int shift = 24; shift >= 0; shift -= 8) {
    for (int b = tid; b < 256; b += NT) hist[b] = 0;
    __syncthreads();
    const uint32_t hi_mask = shift == 24 ? 0u : (0xFFFFFFFFu << (shift + 8));
    for (int64_t i = tid; i < V; i += NT) {
      float v = load_elem<T>(row, i);
      uint32_t key = mono_key(v + 0.0f);
      if (v > -INFINITY && (key & hi_mask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1u);
    }
    __syncthreads();
    if (tid == 0) {
      int cum = 0, d = 255;
      for (; d > 0; --d) {
        int h = int(hist[d]);
        if (cum + h >= need) break;
        cum += h;
      }
      sh.bcast_i[0] = d;
      sh.bcast_i[1] = need - cum;
    }
    __syncthreads();
    prefix |= uint32_t(sh.bcast_i[0]) << shift;
    need = sh.bcast_i[1];
    __syncthreads();
  }
  const uint32_t key_k = prefix;   // key of the k_eff-th largest element; `need` ties are to be taken

  // collection in index order: everything above key_k, and the `need` lowest-index ties
  if (tid == 0) sh.cand_count = 0;
  __syncthreads();
  int eq_base = 0;
  constexpr int kChunk = 8;
  for (int64_t base = 0; base < V; base += int64_t(NT) * kChunk) {
    uint32_t eq_mask = 0;
    const int64_t i0 = base + int64_t(tid) * kChunk;
#pragma unroll
    for (int e = 0; e < kChunk; ++e) {
      int64_t i = i0 + e;
      if (i < V) {
        float v = load_elem<T>(row, i);
        uint32_t key = mono_key(v + 0.0f);
        if (v > -INFINITY) {
          if (key > key_k) {
            int pos = atomicAdd(&sh.cand_count, 1);
            cand[pos] = make_cand(v, uint32_t(i));
          } else if (key == key_k) {
            eq_mask |= 1u << e;
          }
        }
      }
    }
    int total;
    int off = block_excl_scan_i32<NW>(__popc(eq_mask), sh.red, total);
    if (eq_base < need) {
      int ord = eq_base + off;
#pragma unroll
      for (int e = 0; e < kChunk; ++e) {
        if ((eq_mask >> e) & 1u) {
          if (ord < need) {
            int pos = atomicAdd(&sh.cand_count, 1);
            cand[pos] = make_cand(load_elem<T>(row, i0 + e), uint32_t(i0 + e));
          }
          ++ord;
        }
      }
    }
    eq_base += total;
  }
  // the normaliser's fp32 partial sums, referenced to the true maximum
  c_ref = __fmul_rn(vmax, k2);
  double acc = 0.0;
  for (int64_t i = tid; i < V; i += NT) acc += double(fast_exp2(__builtin_fmaf(load_elem<T>(row, i), k2, -c_ref)));
  z_c = block_sum_f64<NW>(acc, sh.red);
  __syncthreads();
  return k_eff;
}

// ---------------------------------------------------------------------------------------------
// The threshold of a large set, whose rank is too near the 1024 groups' number to come out among a few more than k
// elements: up to 4096 groups (no fewer than two per element of the set), their maxima's keys in LDS where the candidates
// will be, the k-th largest by bisection.  2048 bfloat16 rows of 32000, k_cap 1024: 809 us by the radix selection, 133 so; 500
// fp32 rows of 12000, k_cap 800: 111 and 39.
// Returns false with `st` set for an unusable row.
template <typename T, int NT>
__device__ __forceinline__ bool many_groups_threshold(const void* row, const RowSplit& rs, int k_sel, uint32_t* group, int cap,
                                                   TruncateShared& sh, float& tau, float& vmax, int& st) {
  constexpr int E = ElemTraits<T>::kPerVec;
  constexpr int NW = NT / 64;
  const int tid = threadIdx.x;
  const int n_edge = rs.head + rs.tail;
  const int64_t n_tiles = (rs.nvec + NT - 1) / NT;
  const int per = 2 * cap / NT < 4096 / NT ? 2 * cap / NT : 4096 / NT;      // a thread's groups
  for (int u = 0; u < per; ++u) group[u * NT + tid] = 0u;                   // (its own throughout: no barrier)
  int fin = 0, bad = 0;
  vmax = -INFINITY;
  int slot = 0;
  for (int64_t t0 = 0; t0 < n_tiles; t0 += 4) {
    uint4 d[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t vi = (t0 + u) * NT + tid;
      d[u] = neg_inf_vec<T>();
      if (vi < rs.nvec) d[u] = load_vec(&rs.body[vi]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float v[E], m = -INFINITY;
      unpack<T>(d[u], v);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        bad |= (v[e] != v[e] || v[e] == INFINITY) ? 1 : 0;
        fin += v[e] > -INFINITY ? 1 : 0;
        m = fmaxf(m, v[e]);
      }
      vmax = fmaxf(vmax, m);
      const uint32_t key = m > -INFINITY ? mono_key(m + 0.0f) : 0u;
      uint32_t* g = &group[slot * NT + tid];
      *g = *g > key ? *g : key;
      slot = slot + 1 == per ? 0 : slot + 1;
    }
  }
  if (tid < n_edge) {
    const float v = load_elem<T>(row, edge_index<T>(rs, tid));
    bad |= (v != v || v == INFINITY) ? 1 : 0;
    fin += v > -INFINITY ? 1 : 0;
    vmax = fmaxf(vmax, v);
    const uint32_t key = v > -INFINITY ? mono_key(v + 0.0f) : 0u;
    group[tid] = group[tid] > key ? group[tid] : key;
  }
  bad = block_or_i32<NW>(bad, sh.red);
  fin = block_sum_i32<NW>(fin, sh.red);
  if (bad) { st |= 1; return false; }
  if (fin == 0) { st |= 2; return false; }
  const int k_eff = k_sel < fin ? k_sel : fin;
  vmax = block_max_f32<NW>(vmax, sh.red);
  uint32_t key = 0;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t trial = key | (1u << bit);
    int n = 0;
    for (int u = 0; u < per; ++u) n += group[u * NT + tid] >= trial ? 1 : 0;
    if (block_sum_i32<NW>(n, sh.red) >= k_eff) key = trial;
  }
  tau = key > kKeyNegInf ? key_to_f32(key) : -INFINITY;                     // fewer than k_eff groups: everything
  return true;
}

// ---------------------------------------------------------------------------------------------
// Two-pass selection, the first fallback.  Pass 1 takes the maximum of 1024 disjoint groups of the
// row (4 per thread); the k-th largest of those maxima is a threshold that at least k elements reach,
// so the top-k set is among the elements >= it, of which there are only a few more than k unless the
// row is full of ties.  Pass 2 collects them.  Returns the number of candidates, 0 with `st` set for
// an unusable row, or -1 when the candidates do not fit (then the radix selection is used).
// ---------------------------------------------------------------------------------------------
template <typename T, int NT, bool kLarge>
__device__ __forceinline__ int two_pass_select(const void* row, const RowSplit& rs, int k_sel, float k2, uint64_t* cand, int cap,
                               uint64_t* sort_tmp, int sort_tmp_cap, uint32_t* tables, TruncateShared& sh,
                               bool need_sum, float& c_ref, double& z_c, int& st) {
  constexpr int E = ElemTraits<T>::kPerVec;
  constexpr int NW = NT / 64;
  constexpr int GPT = 1024 / NT;       // groups per thread
  const int tid = threadIdx.x;
  const int n_edge = rs.head + rs.tail;
  const int64_t n_tiles = (rs.nvec + NT - 1) / NT;
  if (cap < GPT * NT + 2 * E) return -1;
  // pass 1
  float edge_v = -INFINITY;
  int64_t edge_i = 0;
  if (tid < n_edge) {
    edge_i = edge_index<T>(rs, tid);
    edge_v = load_elem<T>(row, edge_i);
  }
  float tau, vmax;
  // (beyond 768 the k-th largest of 1024 maxima is exceeded by nearly twice k elements or more, which do not fit; of g
  // groups it is where 1.25 k is more than g)
  if (kLarge && k_sel > 768 && 5 * int64_t(k_sel) <= 4 * (rs.nvec < 2 * int64_t(cap) ? rs.nvec : 2 * int64_t(cap))) {
    if (!many_groups_threshold<T, NT>(row, rs, k_sel, reinterpret_cast<uint32_t*>(cand), cap, sh, tau, vmax, st)) return 0;
  } else {
    float gmax[GPT];
#pragma unroll
    for (int u = 0; u < GPT; ++u) gmax[u] = -INFINITY;
    int fin = 0, bad = 0;
    for (int64_t t0 = 0; t0 < n_tiles; t0 += GPT) {
      uint4 d[GPT];
#pragma unroll
      for (int u = 0; u < GPT; ++u) {
        const int64_t vi = (t0 + u) * NT + tid;
        d[u] = neg_inf_vec<T>();
        if (vi < rs.nvec) d[u] = load_vec(&rs.body[vi]);
      }
#pragma unroll
      for (int u = 0; u < GPT; ++u) {
        float v[E];
        unpack<T>(d[u], v);
#pragma unroll
        for (int e = 0; e < E; ++e) {
          bad |= (v[e] != v[e] || v[e] == INFINITY) ? 1 : 0;
          fin += v[e] > -INFINITY ? 1 : 0;
          gmax[u] = fmaxf(gmax[u], v[e]);
        }
      }
    }
    if (tid < n_edge) {
      bad |= (edge_v != edge_v || edge_v == INFINITY) ? 1 : 0;
      fin += edge_v > -INFINITY ? 1 : 0;
    }
    bad = block_or_i32<NW>(bad, sh.red);
    fin = block_sum_i32<NW>(fin, sh.red);
    if (bad) { st |= 1; return 0; }
    if (fin == 0) { st |= 2; return 0; }
    const int k_eff = k_sel < fin ? k_sel : fin;
    vmax = gmax[0];
#pragma unroll
    for (int u = 1; u < GPT; ++u) vmax = fmaxf(vmax, gmax[u]);
    vmax = block_max_f32<NW>(fmaxf(vmax, edge_v), sh.red);
    // the k_eff-th largest group maximum (edge elements are groups of their own; empty groups are left out)
    if (tid == 0) sh.cand_count = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < GPT; ++u)
      if (gmax[u] > -INFINITY) cand[atomicAdd(&sh.cand_count, 1)] = make_cand(gmax[u], uint32_t(tid * GPT + u));
    if (tid < n_edge && edge_v > -INFINITY) cand[atomicAdd(&sh.cand_count, 1)] = make_cand(edge_v, uint32_t(GPT * NT + tid));
    __syncthreads();
    const int n_groups = sh.cand_count;
    tau = -INFINITY;                               // fewer than k_eff non-empty groups: take everything
    if (n_groups >= k_eff) {
      if (!bucket_sort_desc<NT>(cand, n_groups, sort_tmp, sort_tmp_cap, cand, k_eff, tables, sh.red))
        return -1;
      tau = cand_value(cand[k_eff - 1]);
    }
  }
  __syncthreads();
  // pass 2
  if (tid == 0) sh.cand_count = 0;
  __syncthreads();
  if (need_sum) c_ref = __fmul_rn(vmax, k2);
  double acc = 0.0;
  for (int64_t t0 = 0; t0 < n_tiles; t0 += 4) {
    uint4 d[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t vi = (t0 + u) * NT + tid;
      d[u] = neg_inf_vec<T>();
      if (vi < rs.nvec) d[u] = load_vec(&rs.body[vi]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float v[E];
      unpack<T>(d[u], v);
      const uint32_t base = uint32_t(rs.head) + uint32_t((t0 + u) * NT + tid) * E;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        if (need_sum) acc += double(fast_exp2(__builtin_fmaf(v[e], k2, -c_ref)));
        if (v[e] >= tau && v[e] > -INFINITY) {
          const int pos = atomicAdd(&sh.cand_count, 1);
          if (pos < cap) cand[pos] = make_cand(v[e], base + e);
        }
      }
    }
  }
  if (tid < n_edge) {
    if (need_sum) acc += double(fast_exp2(__builtin_fmaf(edge_v, k2, -c_ref)));
    if (edge_v >= tau && edge_v > -INFINITY) {
      const int pos = atomicAdd(&sh.cand_count, 1);
      if (pos < cap) cand[pos] = make_cand(edge_v, uint32_t(edge_i));
    }
  }
  if (need_sum) z_c = block_sum_f64<NW>(acc, sh.red);
  __syncthreads();
  const int n = sh.cand_count;
  __syncthreads();
  return n <= cap ? n : -1;
}

// A ring slot holds a 16-byte vector of which at least one element is above tau0, and its index (in
// vectors, within the row's aligned body).
//
// Expands the n vectors parked in a wave's ring into candidate records (elements above tau0).  Lane s
// takes slot s: it marks which of the vector's elements are above tau0, a wave scan of the counts gives
// every lane its place behind a single reservation in the shared candidate array.  Nearly every slot holds
// one such element, so they are then written one per round (as many rounds as the fullest slot needs),
// each read back from the slot by its position, instead of one branch per element position.
template <typename T> __device__ __forceinline__ float ring_element(const uint4* ring, int slot, int e);
template <> __device__ __forceinline__ float ring_element<float>(const uint4* ring, int slot, int e) {
  return reinterpret_cast<const float*>(ring)[slot * 4 + e];
}
template <> __device__ __forceinline__ float ring_element<Bf16>(const uint4* ring, int slot, int e) {
  return as_f32(uint32_t(reinterpret_cast<const uint16_t*>(ring)[slot * 8 + e]) << 16);
}
template <> __device__ __forceinline__ float ring_element<F16>(const uint4* ring, int slot, int e) {
  return f16_lo(reinterpret_cast<const uint16_t*>(ring)[slot * 8 + e]);
}

template <typename T>
__device__ __forceinline__ void expand_ring(const uint4* ring, const uint32_t* ring_vidx, int n, float tau0,
                                            uint32_t head, uint64_t* cand, int cap, TruncateShared& sh) {
  constexpr int E = ElemTraits<T>::kPerVec;
  const int lane = lane_id();
  for (int s0 = 0; s0 < n; s0 += 64) {
    const int s = s0 + lane;
    uint32_t mask = 0, vi = 0;          // bit e: element e of this lane's vector is above tau0
    if (s < n) {
      float v[E];
      unpack<T>(ring[s], v);
      vi = ring_vidx[s];
#pragma unroll
      for (int e = 0; e < E; ++e) mask |= v[e] > tau0 ? (1u << e) : 0u;
    }
    const int cnt = __popc(mask);
    const int incl = wave_incl_scan_i32(cnt);
    const int total = last_lane_i32(incl);
    if (total == 0) continue;
    int base = 0;
    if (lane == 0) base = atomicAdd(&sh.cand_count, total);
    base = __builtin_amdgcn_readfirstlane(base);
    int pos = base + incl - cnt;
    const uint32_t idx0 = head + vi * E;
    const int rounds = wave_max_i32(cnt);
    for (int r = 0; r < rounds; ++r) {
      if (mask != 0) {
        const int e = __builtin_ctz(mask);
        mask &= mask - 1;
        if (pos < cap) cand[pos] = make_cand(ring_element<T>(ring, s, e), idx0 + uint32_t(e));
        ++pos;
      }
    }
  }
  // more candidates than `cap` show in sh.cand_count, which the caller checks
}

template <typename T> __device__ __forceinline__ float vec_max(const float (&v)[ElemTraits<T>::kPerVec]);
template <> __device__ __forceinline__ float vec_max<float>(const float (&v)[4]) {
  return max3f(max3f(v[0], v[1], v[2]), v[3], v[3]);
}
__device__ __forceinline__ float vec_max8(const float (&v)[8]) {
  return max3f(max3f(max3f(v[0], v[1], v[2]), v[3], v[4]), max3f(v[5], v[6], v[7]), v[5]);
}
template <> __device__ __forceinline__ float vec_max<Bf16>(const float (&v)[8]) { return vec_max8(v); }
template <> __device__ __forceinline__ float vec_max<F16>(const float (&v)[8]) { return vec_max8(v); }

// Whether an element of a vector is above the threshold.  `at` makes the threshold what the test compares with, once a row.
// binary16: the maximum of the packed halves, two at a time, against the largest binary16 value that is not above the
// threshold; nothing is widened for it.  (bfloat16 has no such instructions, and its bits are not to be taken for
// binary16: -inf would be a NaN.)  A NaN among the elements may or may not be a hit: its row is redone in any case.
template <typename T> struct HitTest {
  using Threshold = float;
  static __device__ __forceinline__ float at(float tau0) { return tau0; }
  static __device__ __forceinline__ bool hit(const uint4& w, float tau) {
    float v[ElemTraits<T>::kPerVec];
    unpack<T>(w, v);
    return vec_max<T>(v) > tau;
  }
};
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
template <> struct HitTest<F16> {
  using Threshold = _Float16;
  static __device__ __forceinline__ _Float16 at(float tau0) {
    const _Float16 h = _Float16(tau0);                                    // to nearest; one step down if that is above
    uint16_t b = __builtin_bit_cast(uint16_t, h);
    if (float(h) > tau0) b = (b & 0x8000u) ? b + 1 : (b == 0 ? 0x8001u : b - 1);
    return __builtin_bit_cast(_Float16, b);
  }
  static __device__ __forceinline__ bool hit(const uint4& w, _Float16 tau) {
    const half2_t x = __builtin_bit_cast(half2_t, w.x), y = __builtin_bit_cast(half2_t, w.y);
    const half2_t z = __builtin_bit_cast(half2_t, w.z), u = __builtin_bit_cast(half2_t, w.w);
    half2_t m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(x, y), z);
    m = __builtin_elementwise_maximum(m, u);
    return __builtin_elementwise_max(m.x, m.y) > tau;
  }
};

// kParts: p.parts workgroups share a row.  Each makes the same sample and the same threshold, walks its part of the stages
// (with the sample tiles that lie there) and leaves the sum of its terms and its candidates in memory; the one that finds those of
// all goes on as if it had found them itself.
template <typename T, int NT, int kStages, int kWavesPerSimd, bool kParts = false>
__global__ __launch_bounds__(NT, kWavesPerSimd) void truncate_kernel(const TruncateParams p) {
  constexpr int E = ElemTraits<T>::kPerVec;
  constexpr int NW = NT / 64;
  static_assert(kBatch == 4, "the sample tiles are handled as two pairs");
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  __shared__ TruncateShared sh;
  constexpr bool kTall = NT > kTruncThreads;
  constexpr int kRing = kTall ? kRingTall : kRingSmall;
  uint4* ring_all = reinterpret_cast<uint4*>(dyn_lds);
  uint32_t* ring_vidx_all = reinterpret_cast<uint32_t*>(dyn_lds + NW * kRing * 16);
  uint32_t* tables = reinterpret_cast<uint32_t*>(dyn_lds);          // aliasing the rings
  uint64_t* cand = reinterpret_cast<uint64_t*>(dyn_lds + p.ring_bytes);
  uint64_t* sort_tmp = reinterpret_cast<uint64_t*>(dyn_lds + kTablesBytes - kRankAhead * 8);
  const int sort_tmp_cap = (p.ring_bytes - kTablesBytes) / 8;

  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wave = wave_id();
  const uint32_t row_u = kParts ? blockIdx.x / uint32_t(p.parts) : blockIdx.x;
  const int part = kParts ? int(blockIdx.x - row_u * p.parts) : 0;
  const int64_t row_i = row_u;
  const void* row = reinterpret_cast<const char*>(p.logits) + size_t(row_i) * size_t(p.row_stride) * ElemTraits<T>::kBytes;
  const RowSplit rs = split_row<T>(row, p.V);
  const int n_edge = rs.head + rs.tail;
  const uint32_t nvec = uint32_t(rs.nvec);
  const uint32_t n_tiles = (nvec + NT - 1) / NT;
  // The sample: kBatch tiles at equal distances, each the first of a stage; a row of fewer than kBatch complete stages
  // uses its first kBatch tiles.
  // (Every load of the pass below is unconditional: an address past the row's end is replaced by that of
  // the row's last vector and the value by -inf afterwards.  With conditional loads the number of loads in
  // flight is not known where a wait is placed, and a wait for one batch waits for all that were
  // requested after it as well.)
  constexpr int kUnit = kTall ? kGroup : kBatch;      // tiles that the distance is a multiple of
  const uint32_t n_full = nvec / (kUnit * NT);
  const bool long_row = n_full >= kBatch;
  const uint32_t s_stride = long_row ? (n_full / kBatch) * kUnit : 1;    // distance of the sample tiles, in tiles

  int st = 0;
  int n_cand = 0;
  float c_ref = 0.0f;
  if constexpr (kTall) reinterpret_cast<uint32_t*>(cand + p.sort_cap)[tid] = 0;
  double z_c = 0.0;
  bool fast_ok = p.jprime > 0 && n_tiles > 0;
  if (tid == 0) { sh.cand_count = 0; sh.overflow = 0; }

  if (fast_ok) {
    // ---- the sample: per-thread maxima ----------------------------------------------------------
    uint4 d[kBatch];
    auto load_sample = [&](const RowSplit& r, uint4 (&q)[kBatch]) {
      const uint32_t nv = uint32_t(r.nvec);            // > 0 here
      const uint32_t nf = nv / (kUnit * NT);
      const uint32_t stride = nf >= 4 ? (nf / 4) * kUnit : 1;
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const uint32_t vi = u * stride * NT + tid;
        q[u] = load_vec_stream(&r.body[vi < nv ? vi : nv - 1]);
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
        if (u * stride * NT + tid >= nv) q[u] = neg_inf_vec<T>();
    };
    load_sample(rs, d);
    // The pass keeps kStages stages of kGroup tiles in flight per thread; the first ones are requested now, so
    // that they travel while the threshold is being worked out.  In a long row a sample tile is the first tile of
    // its stage and is not read again; in a short one the stages begin behind the sample.  The row's ragged end
    // (the last tile possibly incomplete, the last stage possibly half empty) is the last stage.
    static_assert(kGroup == 2, "a stage is a pair of tiles");
    uint4 pipe[kStages][kGroup];
    const uint32_t tile0 = long_row ? 0u : uint32_t(kBatch);                    // of the first stage
    const uint32_t all_stages = n_tiles > tile0 ? (n_tiles - tile0 + kGroup - 1) / kGroup : 0u;
    const uint32_t stride_g = s_stride / kGroup;
    // this workgroup's stages (kParts: rows long enough that each has some)
    const uint32_t per_part = kParts ? (all_stages + uint32_t(p.parts) - 1) / uint32_t(p.parts) : 0u;
    const uint32_t first_g = kParts ? min(per_part * uint32_t(part), all_stages) : 0u;
    const uint32_t n_stage = kParts ? min(first_g + per_part, all_stages) : all_stages;
    // The row as a buffer: no vector instruction goes into addresses; what lies past the row's end comes back as zeros.  Not
    // in the wide shape, where other workgroups fill the vector units in any case and requests through a buffer are slower
    // (us by buffer / by address: 500 rows of 151936, sets of 200 to 256, bfloat16 37.2 / 35.0, binary16 35.5 / 33.9; 450 fp32 rows,
    // sets of 32, 51.0 / 48.5; 2728 254.9 / 253.0; the deep shape, 1000 fp32 rows of 151936, sets of 1024, 114.8 / 116.5).
    constexpr bool kBuffer = kWavesPerSimd < kWavesWide;
    // (A part's buffer ends where the part does: what its last requests ahead reach is the next workgroup's.)
    const uint32_t end_vec = kParts && (tile0 + n_stage * kGroup) * NT < nvec ? (tile0 + n_stage * kGroup) * NT : nvec;
    const __amdgpu_buffer_rsrc_t body = row_buffer(rs.body, end_vec);
    const uint32_t lane_bytes = uint32_t(tid) * 16u;
    auto request = [&](uint32_t at) -> uint4 {          // of a tile that begins `at` bytes into the row's body
      if constexpr (kBuffer) return buffer_load_vec_stream(body, lane_bytes, at);
      const uint32_t vi = at / 16u + tid;
      return load_vec_stream(&rs.body[vi < nvec - 1 ? vi : nvec - 1]);
    };
    // stages 0, stride_g, 2 stride_g, 3 stride_g begin with a sample tile
    constexpr uint32_t kNever = 0xFFFFFFFFu;
    auto next_sample = [&](uint32_t g) { return g == (kBatch - 1) * stride_g ? kNever : g + stride_g; };
    uint32_t first_sample = long_row ? 0u : kNever;                  // the first stage from first_g on that begins with one
    if constexpr (kParts) {
#pragma unroll
      for (int u = 1; u < kBatch; ++u)
        if (first_sample < first_g) first_sample = u * stride_g;
      if (first_sample < first_g || !long_row) first_sample = kNever;
    }
    uint32_t skip_g = first_sample, issue_at = (tile0 + first_g * kGroup) * (NT * 16u);
    // (called with g = 0, 1, 2, ...: its scalar instructions count where a pair of fp32 vectors has eight logits)
    auto issue = [&](uint32_t g, uint4 (&q)[kGroup]) {
      // the first tile of a sample stage is in registers already: its slot repeats the second tile's load
      uint32_t at_a = issue_at;
      const uint32_t at_b = issue_at + NT * 16u;
      if (__builtin_expect(g == skip_g, 0)) {
        at_a = at_b;
        skip_g = next_sample(g);
      }
      issue_at = at_b + NT * 16u;
      q[0] = request(at_a);
      q[1] = request(at_b);
    };
    // (not yet for the short rows of a large batch, whose sample it would hold up: 2000 fp32 rows of 16000 27.2 and 25.6 us)
    const bool early = kTall || long_row;
    auto issue_first = [&]() {
#pragma unroll
      for (int s = 0; s < kStages; ++s) issue(first_g + uint32_t(s), pipe[s]);
    };
    if (n_stage > first_g && early) issue_first();
    float tmax = -INFINITY;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      float v[E];
      unpack<T>(d[u], v);
      tmax = fmaxf(tmax, vec_max<T>(v));
    }
    // the sample is looked at again after the threshold is known; it is to wait in its packed form (the
    // compiler would otherwise keep the unpacked values, twice the registers, across the threshold search)
#pragma unroll
    for (int u = 0; u < kBatch; ++u) asm volatile("" : "+v"(d[u].x), "+v"(d[u].y), "+v"(d[u].z), "+v"(d[u].w));
    // ---- tau0: the jprime-th largest of the per-thread sample maxima, to the leading tau_bits of its key
    uint32_t tau_key = 0, top_key;                     // top_key: the sample's maximum
    if constexpr (!kTall) {                            // a bit at a time, every wave for itself
      tables[tid] = mono_key(tmax);
      __syncthreads();
      uint32_t kq[NW];
#pragma unroll
      for (int q = 0; q < NW; ++q) kq[q] = tables[lane + 64 * q];
      for (int bit = 31; bit >= 32 - p.tau_bits; --bit) {
        const uint32_t trial = tau_key | (1u << bit);
        int reach = 0;
#pragma unroll
        for (int q = 0; q < NW; ++q) reach += __popcll(ballot(kq[q] >= trial));
        if (reach >= p.jprime) tau_key = trial;
      }
      top_key = kq[0];
#pragma unroll
      for (int q = 1; q < NW; ++q) top_key = kq[q] > top_key ? kq[q] : top_key;
      top_key = wave_max_u32(top_key);
    } else {
      // By a histogram over 256 value bins and the few maxima in the bin of the jprime-th: three barriers.  Where that does not
      // tell them apart (masked rows, rows full of ties) four bits of the key at a time, with a barrier for each four.  (Bits
      // alone, three at a time: 5000 cycles of the 26000 that a binary16 row of 32000 took, 3400 so.)
      const uint32_t key = mono_key(tmax);
      const uint32_t hi = wave_max_u32(key), lo = ~wave_max_u32(~key);
      if (lane == 0) { sh.red.i[wave] = int(hi); sh.red.f[wave] = as_f32(lo); }
      uint32_t* counts = tables + NT;                  // the bins; eight steps of sixteen; the list's length, the list
      uint32_t* list_n = counts + 256 + 8 * 16;
      uint32_t* list = list_n + 4;
      tables[tid] = key;                               // (read by its own wave)
      if (tid < 256 + 8 * 16 + 4) counts[tid] = 0;
      __syncthreads();
      top_key = uint32_t(sh.red.i[0]);
      uint32_t low_key = as_u32(sh.red.f[0]);
#pragma unroll
      for (int w = 1; w < NW; ++w) {
        top_key = uint32_t(sh.red.i[w]) > top_key ? uint32_t(sh.red.i[w]) : top_key;
        low_key = as_u32(sh.red.f[w]) < low_key ? as_u32(sh.red.f[w]) : low_key;
      }
      const int last = 32 - 3 * ((p.tau_bits + 2) / 3);                      // the lowest bit that counts
      const float vmin = key_to_f32(low_key), span = key_to_f32(top_key) - vmin;
      int n_list = 65;
      if (span > 0.0f && span < 3.0e38f) {
        const int in_bin = int((key_to_f32(key) - vmin) * (255.0f / span)), bin = in_bin > 255 ? 255 : in_bin;
        atomicAdd(&counts[bin], 1u);
        __syncthreads();
        // every wave: the bin in which the count from the top passes jprime; lane l has bins 255 - 4 l downwards
        const uint4 h = reinterpret_cast<const uint4*>(counts)[63 - lane];
        const int h4[4] = {int(h.w), int(h.z), int(h.y), int(h.x)};
        const int mine = (h4[0] + h4[1]) + (h4[2] + h4[3]);
        int run = wave_incl_scan_i32(mine) - mine, at = -1, before = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool here = run < p.jprime && run + h4[j] >= p.jprime;
          at = here ? 255 - 4 * lane - j : at;
          before = here ? run : before;
          run += h4[j];
        }
        const int src = __ffsll((long long)ballot(at >= 0)) - 1;             // (jprime is not more than the maxima)
        at = __builtin_amdgcn_readlane(at, src);
        const int rank = p.jprime - __builtin_amdgcn_readlane(before, src);  // among the bin's
        if (bin == at) {
          const uint32_t pos = atomicAdd(list_n, 1u);
          if (pos < 64) list[pos] = key;
        }
        __syncthreads();
        n_list = __builtin_amdgcn_readfirstlane(int(*list_n));
        if (n_list <= 64) {
          const uint32_t k = lane < n_list ? list[lane] : 0u;
          int above = 0, reach = 0;                                           // of the list: larger, no smaller
          for (int i = 0; i < n_list; ++i) {
            const uint32_t x = uint32_t(__builtin_amdgcn_readlane(int(k), i));
            above += x > k ? 1 : 0;
            reach += x >= k ? 1 : 0;
          }
          const int of = __ffsll((long long)ballot(lane < n_list && above < rank && reach >= rank)) - 1;
          tau_key = (uint32_t(__builtin_amdgcn_readlane(int(k), of)) >> last) << last;
        }
      }
      if (n_list > 64) {                                                      // the same in all waves
        uint4 kq[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) kq[q] = reinterpret_cast<const uint4*>(tables)[wave * 16 + (lane >> 4) * 4 + q];
        uint32_t* step = counts + 256;
        int above = 32;
        for (tau_key = 0u; above > last; step += 16) {
          const int bits = above - last < 4 ? above - last : 4, value = lane & 15;
          above -= bits;
          const uint32_t trial = tau_key | (uint32_t(value) << above);
          uint32_t reach = 0;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            reach += kq[q].x >= trial ? 1u : 0u;
            reach += kq[q].y >= trial ? 1u : 0u;
            reach += kq[q].z >= trial ? 1u : 0u;
            reach += kq[q].w >= trial ? 1u : 0u;
          }
          atomicAdd(&step[value], reach);
          __syncthreads();
          const bool tries = lane > 0 && lane < (1 << bits);                 // falls with the value
          tau_key |= uint32_t(__popcll(ballot(tries && int(step[value]) >= p.jprime))) << above;
        }
      }
    }
    const float smax = key_to_f32(top_key);
    const float tau0 = tau_key <= kKeyNegInf ? -INFINITY : key_to_f32(tau_key);
    fast_ok = smax > -INFINITY && smax < INFINITY;   // false for NaN too
    if (tid == 0) { sh.from = tau0; sh.upto = smax; }  // (for the sort: not in registers, which are short during the pass)
    c_ref = __fmul_rn(smax, p.k2);
    __syncthreads();                                  // the maxima are read; the space becomes the rings

    if (kParts && !fast_ok && part != 0) return;      // (the same for all of them)
    if (fast_ok) {
      // ---- the pass -------------------------------------------------------------------------
      // (The two operands that every term's fma shares stand in vector registers, without a sign to change: from a scalar
      // register, or negated on the way, it would issue at half the rate.)
      float k2 = p.k2, neg_c = -c_ref;
      asm volatile("" : "+v"(k2), "+v"(neg_c));
      const typename HitTest<T>::Threshold tau = HitTest<T>::at(tau0);
      // fp32 sums live for a few vectors only and are then added to an fp64 total: a long-lived fp32
      // accumulator that has met one large term rounds away the many small ones that follow
      double dacc = 0.0;
      int wave_cnt = 0;                                // vectors parked in this wave's ring
      bool lost = false;                               // wave-uniform: a ring overflowed
      uint4* ring = ring_all + wave * kRing;
      uint32_t* ring_vidx = ring_vidx_all + wave * kRing;
      const uint32_t head = uint32_t(rs.head);
      auto expand = [&]() {
        expand_ring<T>(ring, ring_vidx, wave_cnt, tau0, head, cand, p.sort_cap, sh);
        wave_cnt = 0;
      };
      // A vector with an element above tau0 is parked in the ring, which is expanded when it has no room for the next ones.
      auto put = [&](bool hit, uint64_t mask, const uint4& w, uint32_t vidx) {
        if (hit) {
          const int pos = wave_cnt + lanes_below(mask);
          ring[pos] = w;
          ring_vidx[pos] = vidx;
        }
        wave_cnt += __popcll(mask);
      };
      auto park = [&](bool hit_a, bool hit_b, const uint4& w0, const uint4& w1, uint32_t vidx0, uint32_t vidx1) {
        const uint64_t mask_a = ballot(hit_a), mask_b = ballot(hit_b);
        if constexpr (kTall) {
          if (mask_a != 0) {
            if (wave_cnt + __popcll(mask_a) > kRing) expand();        // wave-uniform; 64 at most
            put(hit_a, mask_a, w0, vidx0);
          }
          if (mask_b != 0) {
            if (wave_cnt + __popcll(mask_b) > kRing) expand();
            put(hit_b, mask_b, w1, vidx1);
          }
        } else if ((mask_a | mask_b) != 0) {
          if (wave_cnt + __popcll(mask_a) + __popcll(mask_b) > kRing) {      // wave-uniform: the row is to be redone
            lost = true;
            wave_cnt = 0;
          } else {
            put(hit_a, mask_a, w0, vidx0);
            put(hit_b, mask_b, w1, vidx1);
            if (wave_cnt > kRingExpand) expand();
          }
        }
      };
      // The sum of a vector's, or of a pair's, exp2 terms, in a tree without an addition of zero.
      auto sum_of = [&](auto& t) -> float {
#pragma unroll
        for (int w = int(sizeof(t) / sizeof(t[0])) / 2; w >= 1; w >>= 1)
#pragma unroll
          for (int e = 0; e < w; ++e) t[e] += t[e + w];
        return t[0];
      };
      auto process_pair = [&](uint4 w0, uint4 w1, uint32_t vidx0, uint32_t vidx1) -> float {
        float a[E], b[E], t[2 * E];
        const bool hit_a = HitTest<T>::hit(w0, tau), hit_b = HitTest<T>::hit(w1, tau);
        unpack<T>(w0, a);
        unpack<T>(w1, b);
#pragma unroll
        for (int e = 0; e < E; ++e) {
          t[e] = fast_exp2(__builtin_fmaf(a[e], k2, neg_c));
          t[E + e] = fast_exp2(__builtin_fmaf(b[e], k2, neg_c));
        }
        const float pair_sum = sum_of(t);
        park(hit_a, hit_b, w0, w1, vidx0, vidx1);
        return pair_sum;
      };
      // the second vector of a pair whose first is done
      auto process_second = [&](const uint4& w1, uint32_t vidx1) -> float {
        float b[E];
        unpack<T>(w1, b);
        const bool hit_b = HitTest<T>::hit(w1, tau);
#pragma unroll
        for (int e = 0; e < E; ++e) b[e] = fast_exp2(__builtin_fmaf(b[e], k2, neg_c));
        const float sum = sum_of(b);
        park(false, hit_b, w1, w1, vidx1, vidx1);
        return sum;
      };

      if (n_stage > 0 && !early) issue_first();
      // the sample tiles, already in registers
      if constexpr (kParts) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          const uint32_t g = u * stride_g;
          if (long_row ? g >= first_g && g < n_stage : part == 0) dacc += double(process_second(d[u], u * s_stride * NT + tid));
        }
      } else {
        const uint32_t t1 = s_stride;
        float both = 0.0f;
#pragma unroll 1
        for (uint32_t t = 0; t <= 2 * t1; t += 2 * t1) {              // (s_stride > 0)
          both += process_pair(d[0], d[1], t * NT + tid, (t + t1) * NT + tid);
          d[0] = d[2];
          d[1] = d[3];
        }
        dacc += double(both);
      }
      uint32_t seen_g = first_sample;
      // stages before this one are complete
      uint32_t ragged_g = nvec / NT > tile0 ? (nvec / NT - tile0) / kGroup : 0u;
      if (kParts && n_stage < ragged_g) ragged_g = n_stage;
      // (a short row's stages go to the fp64 total one by one where 256 threads take it)
      const bool apart = !kTall && !long_row;
      static_assert(kStages % 2 == 0, "the fp32 sums of two stages are added up before they go to the fp64 total");
      auto sample_stage = [&](uint32_t g) {                         // its first tile is done
        const bool seen = __builtin_expect(g == seen_g, 0);
        if (seen) seen_g = next_sample(g);
        return seen;
      };
      uint32_t g0 = first_g;
      for (; g0 + kStages <= ragged_g; g0 += kStages) {
        float two = 0.0f;
#pragma unroll
        for (int s = 0; s < kStages; ++s) {
          const uint32_t g = g0 + s;
          const uint32_t v0 = (tile0 + g * kGroup) * NT + tid;
          // (their distance is a multiple of kUnit tiles)
          const bool seen = (kParts || s % (kUnit / kGroup) == 0) && sample_stage(g);
          const float ps = seen ? process_second(pipe[s][1], v0 + NT) : process_pair(pipe[s][0], pipe[s][1], v0, v0 + NT);
          two = (s & 1) && !apart ? two + ps : ps;
          if ((s & 1) || apart) dacc += double(two);
          issue(g + kStages, pipe[s]);
        }
      }
      // the row's end: fewer than kStages complete stages, then perhaps one that is not
      float two = 0.0f;
#pragma unroll 1
      for (uint32_t g = g0; g < n_stage; ++g) {
        const uint32_t v0 = (tile0 + g * kGroup) * NT + tid;
        if (sample_stage(g)) pipe[0][0] = neg_inf_vec<T>();
        if (v0 >= nvec) pipe[0][0] = neg_inf_vec<T>();
        if (v0 + NT >= nvec) pipe[0][1] = neg_inf_vec<T>();
        const float ps = process_pair(pipe[0][0], pipe[0][1], v0, v0 + NT);
        const bool odd = (g - g0) & 1;
        two = odd && !apart ? two + ps : ps;
        if (odd || apart || g + 1 == n_stage) dacc += double(two);    // (a lone last stage's sum is added as it is)
#pragma unroll
        for (int s = 0; s + 1 < kStages; ++s) { pipe[s][0] = pipe[s + 1][0]; pipe[s][1] = pipe[s + 1][1]; }
      }
      expand();
      if (lost && lane == 0) sh.overflow = 1;
      // edge elements (row not 16-byte aligned, or V not a whole number of vectors)
      if (tid < n_edge && part == 0) {
        const int64_t edge_i = edge_index<T>(rs, tid);
        const float edge_v = load_elem<T>(row, edge_i);
        dacc += double(fast_exp2(__builtin_fmaf(edge_v, k2, neg_c)));
        if (edge_v > tau0) {
          const int pos = atomicAdd(&sh.cand_count, 1);
          if (pos < p.sort_cap) cand[pos] = make_cand(edge_v, uint32_t(edge_i));
        }
      }
      dacc = wave_sum_f64(dacc);
      if (lane == 0) sh.red.d[wave] = dacc;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < NW; ++w) z_c += sh.red.d[w];
      n_cand = sh.cand_count;
      if constexpr (kParts) {
        uint64_t* found = p.part_found + (size_t(row_i) * p.parts) * (2 + p.sort_cap);
        {
          uint64_t* mine = found + size_t(part) * (2 + p.sort_cap);
          const int n = n_cand < p.sort_cap ? n_cand : p.sort_cap;
          for (int i = tid; i < n; i += NT) store_through(&mine[2 + i], cand[i]);
          if (tid == 0) {
            store_through(&mine[0], uint64_t(__double_as_longlong(z_c)));
            store_through(&mine[1], uint64_t(n_cand));
          }
        }
        if (!all_arrived(p.part_words + size_t(row_i) * p.parts, part, p.parts, p.tag, sh.bcast_i[0])) return;
        // (a part's first candidates are asked for with its numbers, the others behind them)
        z_c = 0.0;
        n_cand = 0;
        uint64_t sum[kTruncMaxParts], count[kTruncMaxParts], rec[kTruncMaxParts];
#pragma unroll
        for (int k = 0; k < kTruncMaxParts; ++k) {
          if (k >= p.parts) break;
          const uint64_t* from = found + size_t(k) * (2 + p.sort_cap);
          sum[k] = load_through(&from[0]);
          count[k] = load_through(&from[1]);
          rec[k] = load_through(&from[2 + tid]);       // (sort_cap is more than NT)
        }
        if (wave == 0) {                               // (travels with them)
          const bool mine = claimed(p.part_words + size_t(row_i) * p.parts, p.parts, p.tag);
          if (lane == 0) sh.bcast_i[1] = mine ? 1 : 0;
        }
#pragma unroll
        for (int k = 0; k < kTruncMaxParts; ++k) {
          if (k >= p.parts) break;
          const uint64_t* from = found + size_t(k) * (2 + p.sort_cap);
          const int n = int(count[k]);
          z_c += __longlong_as_double((long long)sum[k]);
          if (n_cand + n <= p.sort_cap) {              // (more than that do not fit: the row is redone)
            if (tid < n) cand[n_cand + tid] = rec[k];
            for (int i = NT + tid; i < n; i += NT) cand[n_cand + i] = load_through(&from[2 + i]);
          }
          n_cand += n;
        }
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(sh.bcast_i[1]) == 0) return;
      }
      fast_ok = !sh.overflow && n_cand <= p.sort_cap && n_cand >= p.k_sel && z_c > 0.0 && z_c < INFINITY;
    }
  }

  // a row's uniforms, one per lane, travel during the sort
  static_assert(kMaxDraws <= 64, "a lane to a draw");
  const float u_lane = p.u && lane < p.n_samples ? p.u[size_t(row_i) * p.n_samples + lane] : 0.0f;
  if (!fast_ok) {
    __syncthreads();                                  // the counts and sums above have been read
    st |= 256;
    const bool need_sum = !(z_c > 0.0 && z_c < INFINITY);
    n_cand = two_pass_select<T, NT, kWavesPerSimd == 4>(row, rs, p.k_sel, p.k2, cand, p.sort_cap, sort_tmp, sort_tmp_cap, tables, sh, need_sum,
                                c_ref, z_c, st);
  }

  // ---- sort the candidates into canonical order ------------------------------------------------
  // (behind a barrier since the candidates were written; what the sort writes first is not what was read since)
  // Out of the pass few candidates are counted directly; of many the bins lie between the threshold and where the row's maximum is
  // to be expected (p.reach).  us of a 512-thread kernel's sort: 2.1 by its extremes, 1.7
  // so, 100 candidates 0.9; 30 bfloat16 rows of 9000 8.8 / 8.5, 2000 of 32000 34.5 / 33.9, 2000 of 60000, k 1000 127.3 / 126.3.  (With the bins up
  // to the sample's maximum as many candidates crowd the top one as the sample is smaller than the row: 464 binary16 rows of 180544, sets
  // of 59, 38.2 by the extremes, 39.1 so, 38.1 as it is; 464 bfloat16 of 256000, sets of 32, 46.7 / 48.8 / 46.3.)  Not for fp32
  // in the wide shape: 2728 rows of 151936 253.1 / 254.4.
  const uint64_t* sorted = cand;
  bool done = false;
  constexpr bool kAsBefore = kWavesPerSimd == kWavesWide && E == 4;
  if (!kAsBefore && fast_ok && n_cand <= NT / 4) {
    rank_sort_desc<NT>(cand, n_cand, sort_tmp, p.k_sel);
    sorted = sort_tmp;
    done = true;
  } else if (!kAsBefore && fast_ok) {
    uint32_t* bins = kTall ? reinterpret_cast<uint32_t*>(cand + p.sort_cap) : tables;
    if constexpr (!kTall) {
      bins[tid] = 0;
      __syncthreads();
    }
    done = bucket_sort_desc<NT, true>(cand, n_cand, sort_tmp, sort_tmp_cap, cand, p.k_sel, bins, sh.red, sh.from, sh.from + (sh.upto - sh.from) * p.reach);
    if (!done) __syncthreads();
  }
  while (!done) {
    if (n_cand < 0) n_cand = exact_select<T, NT>(row, p.V, p.k_sel, p.k2, cand, tables, sh, c_ref, z_c, st);
    if (bucket_sort_desc<NT>(cand, n_cand, sort_tmp, sort_tmp_cap, cand, p.k_sel, tables, sh.red)) break;
    // the bin at the k-th place is too crowded for the scratch space (a row full of ties): radix selection
    // delivers exactly k candidates, which always fit
    st |= 256;
    n_cand = -1;
  }
  const int k_eff = n_cand < p.k_sel ? n_cand : p.k_sel;

  // ---- fp64 evaluation of the kept head: Top-rho, renormalisation, outputs -----------------------
  // thread t owns entries [t*per, t*per + per) so that a block scan gives prefix masses in order
  // (Every exchange between waves below is one barrier: what a wave leaves in sh.red is read behind it, and is not written
  // again until another has passed.)
  const int per = (k_eff + NT - 1) / NT;       // 0..kMaxPer
  constexpr int kMaxPer = 1024 / NT;
  double e64[kMaxPer];
  float s32[kMaxPer];
  uint32_t idx[kMaxPer];
  double local = 0.0, head32 = 0.0;
  float v0 = 0.0f, m_s = 0.0f;
  if (k_eff > 0) {
    v0 = cand_value(sorted[0]);
    m_s = __fmul_rn(v0, p.rT);
  }
#pragma unroll
  for (int r = 0; r < kMaxPer; ++r) {
    e64[r] = 0.0; s32[r] = 0.0f; idx[r] = 0;
    const int i = tid * per + r;
    if (r < per && i < k_eff) {
      const uint64_t c = sorted[i];
      const float v = cand_value(c);
      idx[r] = cand_index(c);
      s32[r] = __fmul_rn(v, p.rT);
      e64[r] = exp64(double(s32[r]) - double(m_s));
      local += e64[r];
      head32 += double(fast_exp2(__builtin_fmaf(v, p.k2, -c_ref)));
    }
  }
  double excl = wave_incl_scan_f64(local), head64 = 0.0;
  head32 = wave_sum_f64(head32);
  if (lane == 63) { sh.red.d[wave] = excl; sh.red.d[NW + wave] = head32; }
  __syncthreads();
  {
    double base = 0.0;
    head32 = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      base += w < wave ? sh.red.d[w] : 0.0;
      head64 += sh.red.d[w];
      head32 += sh.red.d[NW + w];
    }
    excl = base + excl - local;
  }
  // normaliser relative to the row maximum: fp32 tail rescaled to that reference + fp64 head
  double tail = z_c - head32;
  if (tail < 0.0) tail = 0.0;
  const double Z = k_eff > 0 ? tail * exp64((double(c_ref) - double(v0) * double(p.k2)) * 0.69314718055994530942) + head64 : 0.0;

  int count = k_eff;
  if (p.top_p > 0.0f && k_eff > 0) {
    const double thr = double(p.top_p) * Z;
    int below = 0;
    double run = excl;
#pragma unroll
    for (int r = 0; r < kMaxPer; ++r) {
      const int i = tid * per + r;
      if (r < per && i < k_eff) {
        run += e64[r];
        below += run < thr ? 1 : 0;
      }
    }
    below = wave_sum_i32(below);
    if (lane == 0) sh.red.i[wave] = below;
    __syncthreads();
    below = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) below += sh.red.i[w];
    count = below + 1 < k_eff ? below + 1 : k_eff;
  }
  // mass of the kept set: inclusive prefix at entry count-1
  {
    double run = excl;
#pragma unroll
    for (int r = 0; r < kMaxPer; ++r) {
      const int i = tid * per + r;
      if (r < per && i < k_eff) {
        run += e64[r];
        if (i == count - 1) sh.bcast_d[0] = run;
      }
    }
  }
  __syncthreads();
  const double c_sel = count > 0 ? sh.bcast_d[0] : 1.0;

  // what prob and the draws are made of: the kept entries' terms, or, with a 16-bit payload, the terms of
  // the rounded values (q_hat is the softmax of what the receiver gets)
  double pw[kMaxPer];
  double p_excl = excl, p_total = c_sel;
  auto scan_again = [&](double v, double& before, double& total) {      // exclusive scan in thread order, and the sum
    const double inc = wave_incl_scan_f64(v);
    if (lane == 63) sh.red.d[wave] = inc;
    __syncthreads();
    double base = 0.0;
    total = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      base += w < wave ? sh.red.d[w] : 0.0;
      total += sh.red.d[w];
    }
    before = base + inc - v;
  };
#pragma unroll
  for (int r = 0; r < kMaxPer; ++r) pw[r] = e64[r];
  if (p.payload != kPayloadF32) {
    const double m_r = double(round_payload(m_s, p.payload));
    double mine = 0.0;
#pragma unroll
    for (int r = 0; r < kMaxPer; ++r) {
      const int i = tid * per + r;
      pw[r] = 0.0;
      if (r < per && i < count) {
        s32[r] = round_payload(s32[r], p.payload);
        pw[r] = exp64(double(s32[r]) - m_r);
        mine += pw[r];
      }
    }
    scan_again(mine, p_excl, p_total);
    if (!(p_total > 0.0)) p_total = 1.0;
  }

  const size_t out0 = size_t(row_i) * size_t(p.k_cap);
  const double inv_total = 1.0 / p_total;        // one reciprocal instead of a division per entry
#pragma unroll
  for (int r = 0; r < kMaxPer; ++r) {
    const int i = tid * per + r;
    if (r < per && i < k_eff && i < count) {
      p.out_idx[out0 + i] = int32_t(idx[r]);
      p.out_logit[out0 + i] = s32[r];
      if (p.out_prob) p.out_prob[out0 + i] = float(pw[r] * inv_total);
    }
  }
  for (int i = count + tid; i < p.k_cap; i += NT) {
    p.out_idx[out0 + i] = -1;
    p.out_logit[out0 + i] = -INFINITY;
    if (p.out_prob) p.out_prob[out0 + i] = 0.0f;
  }
  if (tid == 0) {
    p.out_count[row_i] = count;
    if (p.out_mass) p.out_mass[row_i] = count > 0 ? float(c_sel / Z) : 0.0f;
    if (p.status) p.status[row_i] = st;
  }
  // ---- draws from q_hat: the first entry whose inclusive prefix exceeds u * (mass of the kept set) ---
  // Without replacement a drawn entry's weight becomes 0 and the prefix masses are scanned again, so the
  // next draw is from the renormalised rest; when nothing is left the draw gives -1.
  if (p.u) {
    double w_total = count > 0 ? p_total : 0.0;
    for (int c = 0; c < p.n_samples; ++c) {
      const size_t o = size_t(row_i) * p.n_samples + c;
      const double target = double(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(u_lane), c))) * w_total;
      int not_above = 0, last_pos = -1;
      double run = p_excl;
#pragma unroll
      for (int r = 0; r < kMaxPer; ++r) {
        const int i = tid * per + r;
        if (r < per && i < count) {
          run += pw[r];
          not_above += run > target ? 0 : 1;
          if (pw[r] > 0.0) last_pos = i;
        }
      }
      int slot = -1;
      if (w_total > 0.0) {                                             // uniform
        int* part = c & 1 ? reinterpret_cast<int*>(sh.red.f) : sh.red.i;
        not_above = wave_sum_i32(not_above);
        if (lane == 0) part[wave] = not_above;
        __syncthreads();
        slot = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) slot += part[w];
      }
      if (slot >= count) {                                             // only for u >= 1 (uniform branch)
        slot = block_max_i32<NW>(last_pos, sh.red);
        __syncthreads();
      }
#pragma unroll
      for (int r = 0; r < kMaxPer; ++r)
        if (r < per && tid * per + r == slot) p.out_token[o] = int32_t(idx[r]);
      if (tid == 0) {
        if (slot < 0) p.out_token[o] = -1;
        if (p.out_slot) p.out_slot[o] = slot;
      }
      if (p.without_replacement && c + 1 < p.n_samples && slot >= 0) {       // uniform
        double rest = 0.0;
#pragma unroll
        for (int r = 0; r < kMaxPer; ++r) {
          const int i = tid * per + r;
          if (r < per && i == slot) pw[r] = 0.0;
          if (r < per && i < count) rest += pw[r];
        }
        scan_again(rest, p_excl, w_total);
      }
    }
  }
}

}  // namespace tslt
