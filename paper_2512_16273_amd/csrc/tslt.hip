// C ABI of the TSLT hot path (see include/tslt.h): argument checks, launch plans, kernel launches.
#include "tslt.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <mutex>
#include <string>

#include "common.h"
#include "sample.h"
#include "truncate.h"
#include "wire.h"
#include "tree.h"
#include "verify.h"
#include "stats.h"
#include "calib.h"

// Scratch memory of tslt_verify_static: what tslt_verify keeps in its caller's workspace, the per-position decisions and status
// words and, where there is room behind them, the masses of rows that workgroups share.  Every GPU the library runs on holds its own copy until the process ends.  In host
// code the name is only a handle for hipGetSymbolAddress; kernels are given the address that call returns.
#define TSLT_STATIC_SCRATCH_BYTES (2 * 4 * TSLT_STATIC_MAX_POSITIONS)
static __device__ __align__(256) unsigned char scratch[TSLT_STATIC_SCRATCH_BYTES];

namespace {

thread_local std::string g_last_error;

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return code;
}

int hip_fail(hipError_t e, const char* what) {
  return fail(TSLT_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

bool valid_dtype(tslt_dtype dt) { return dt == TSLT_F32 || dt == TSLT_BF16 || dt == TSLT_F16; }
int elem_bytes(tslt_dtype dt) { return dt == TSLT_F32 ? 4 : 2; }
// a row is addressed with 32-bit byte offsets from its start
bool row_too_long(int64_t V, tslt_dtype dt) { return V > 0x7FFFFFFF || V * elem_bytes(dt) >= (int64_t(1) << 32); }

// fl32(1/T), the one scaling constant every side derives the same way
float reciprocal_temperature(float T) { return float(1.0 / double(T)); }
float log2e_over_T(float rT) { return float(double(rT) * 1.4426950408889634074); }

constexpr size_t kMaxLds = 160 * 1024;   // LDS of one gfx950 compute unit

// Launch plan of the truncate kernel: which rank among the per-thread sample maxima gives the
// threshold, and how large the candidate array has to be.  Returns the bytes of dynamic LDS.
size_t plan_truncate(tslt_dtype dt, int64_t V, int nt, tslt::TruncateParams& p) {
  const int E = 16 / elem_bytes(dt);
  const double G = nt;                                 // per-thread sample maxima
  const int64_t tile = int64_t(nt) * E;
  const int64_t n_tiles = (V + tile - 1) / tile;
  const int64_t ns = n_tiles < tslt::kBatch ? n_tiles : tslt::kBatch;
  const double n_sample = double(ns * tile < V ? ns * tile : V);
  const double f = n_sample / double(V);               // fraction of the row in the sample
  const double kp = p.k_sel * f;                       // expected sample elements inside the top-k
  const double j = f >= 1.0 ? kp + 1.0 : kp + 4.0 * std::sqrt(kp) + 4.0;
  const double jc = G * (1.0 - std::exp(-j / G));      // distinct threads holding the top j
  const int jprime = int(std::ceil(jc + 2.0 * std::sqrt(j > jc ? j - jc : 0.0) + 1.0));
  // every bf16 value is told apart by the leading 16 bits of its fp32 key, every binary16 value (11
  // significant bits) by the leading 19
  p.tau_bits = dt == TSLT_BF16 ? 16 : (dt == TSLT_F16 ? 19 : 20);
  p.jprime = 0;
  // candidate capacity: always room for the fallback's 1024 group maxima and for 2 * k_sel records.
  const int min_cap = (1024 + 16 > 2 * p.k_sel) ? 1024 + 16 : 2 * p.k_sel;
  p.ring_bytes = tslt::truncate_ring_bytes(nt / 64, p.k_sel);
  p.sort_cap = min_cap;
  if (jprime <= int(0.8 * G)) {
    const double j_eff = -G * std::log(1.0 - double(jprime) / G);
    int sort_cap = int((j_eff + 5.0 * std::sqrt(j_eff) + 4.0) / f) + 16;   // mean + 5 sigma of the hits
    if (sort_cap < min_cap) sort_cap = min_cap;
    if (tslt::truncate_lds_bytes(p.ring_bytes, sort_cap, nt) + sizeof(tslt::TruncateShared) + 256 <= kMaxLds) {
      p.jprime = jprime;
      p.sort_cap = sort_cap;
      // (of n values above a threshold, in a tail that falls exponentially, the largest is ln n + 0.577 scales above it.  Not where the sample
      // itself has many: few are beyond it, and wider bins crowd the first ones.  us so / up to the sample's maximum: j_eff 130 to 220, 1 binary16
      // row of 90000, sets of 1024, 24.8 / 24.1, 1 bfloat16 of 60000 of 1000 22.6 / 22.2, 500 fp32 of 30000 of 700 23.2 / 23.0; 78, 2000
      // bfloat16 of 32000 of 200 33.2 / 33.5; 40, 200 fp32 of 100000 of 256 20.7 / 21.0; less, 1064 bfloat16 of 242880 of 356 98.8 / 100.5)
      p.reach = j_eff >= 100.0 ? 1.0f : float((std::log(j_eff / f) + 0.577) / (std::log(j_eff) + 0.577));
    }
  }
  return tslt::truncate_lds_bytes(p.ring_bytes, p.sort_cap, nt);
}

// Device address of `scratch` on the current device, looked up once per device.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};
hipError_t scratch_on_current_device(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (ptr == nullptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

constexpr int kLargeLds = int(kMaxLds - 4096);

// One shape of the truncation kernel (see truncate.h): NT threads to a row.
template <typename T, int NT, int kStages, int kWavesPerSimd, bool kParts = false>
hipError_t launch_truncate_shape(const tslt::TruncateParams& p, size_t lds, hipStream_t s) {
  constexpr auto fn = &tslt::truncate_kernel<T, NT, kStages, kWavesPerSimd, kParts>;
  if (lds + sizeof(tslt::TruncateShared) > 48 * 1024) {
    const hipError_t e = tslt::allow_dynamic_lds<fn>(kLargeLds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(fn, dim3(unsigned(kParts ? p.rows * p.parts : p.rows)), dim3(NT), lds, s, p);
  return hipSuccess;
}
// Workgroups that share each row of a small batch (1: none do): four where that makes no more of them than compute units, else
// two, for rows long enough that the walk saved is worth two trips to memory (some 3 us).  What follows the walk is the smaller, and with it
// the other workgroups' part in the time, the smaller the set: so rows of narrow sets from a greater length on (k_sel: the most that are selected).
// us by one workgroup a row / four, sets of 32, 256 and 1024:
//   1 row     binary16 64000 10.9 / 12.2, 11.8 / 12.8; 90000 11.9 / 12.4, 13.4 / 13.3; 110000 12.9 / 12.3, 14.0 / 12.9, 17.4 / 15.4;
//             bfloat16 90000 12.4 / 12.5, 13.6 / 13.1; 128256 14.4 / 12.4, 15.5 / 13.0, 19.5 / 15.4
//             fp32 45000 10.5 / 11.9, 11.1 / 12.2; 56000 11.1 / 11.9, 12.5 / 12.5; 64000 11.7 / 11.8, 13.0 / 12.5, 16.2 / 14.3;
//             50000, 60000 sets of 1024 and 900 14.6 / 14.4, 15.2 / 13.1
//   32 rows   binary16 90000 13.7 / 14.4, 14.9 / 14.8; 110000 14.5 / 14.8, 16.0 / 15.3, 19.5 / 17.1; 128256 15.4 / 14.7
//             bfloat16 90000 14.0 / 14.5, 15.1 / 14.8; fp32 45000 12.6 / 13.9, 13.5 / 14.2; 56000 12.9 / 14.0, 14.2 / 14.5;
//             64000 14.0 / 14.2, 15.0 / 14.5; 72000 14.2 / 14.3, 15.5 / 14.9; 90000 15.9 / 14.9
//             (sets of 100: binary16 95000 14.5 / 14.8, 103000 14.6 / 15.0, 112000 14.9 / 14.7; fp32 64000 14.2 / 14.2)
//   64 rows   binary16 128256 15.7 / 15.5, 17.1 / 15.6; fp32 64000 14.2 / 15.0, 15.2 / 15.0, 18.2 / 17.2; 72000 14.6 / 15.1, 15.6 / 15.7;
//             90000 16.4 / 15.8, 17.4 / 16.1
// and by one / two: 128 rows, binary16 128256 16.0 / 16.8, 17.4 / 17.1; 200000 19.1 / 19.4 (sets of 16), 19.9 / 19.4 (of 100); 256000 22.0 / 21.4,
// 23.8 / 21.8; bfloat16 128256 16.3 / 16.9, 17.9 / 17.2, 21.5 / 20.9; fp32 90000 17.5 / 18.2, 18.4 / 18.5, 21.0 / 21.7; 100000 17.7 / 18.8, 18.6 / 19.0;
// 115000 20.4 / 20.2, 21.2 / 20.5; 80 rows, binary16 150000 16.8 / 16.7 (sets of 16); fp32 100000 16.9 / 16.8, 17.9 / 17.2.
// (Eight: 16 rows of half a megabyte 2 % faster than four, the others slower.)
int truncate_parts(tslt_dtype dt, int64_t V, int64_t rows, int k_sel) {
  const int64_t cus = tslt::compute_units(), kb = V * elem_bytes(dt) >> 10;
  const bool f32 = dt == TSLT_F32;
  if (8 * rows <= cus) {
    if (kb >= (k_sel < 64 ? (f32 ? 300 : 210) : k_sel < 160 ? (f32 ? 270 : 190) : (!f32 ? 170 : k_sel < 512 ? 240 : 200))) return 4;
  } else if (4 * rows <= cus) {
    if (kb >= (f32 && k_sel < 512 ? 310 : 220)) return 4;
  }
  if (5 * rows <= 2 * cus) return kb >= (f32 ? 350 : 240) ? 2 : 1;
  return 2 * rows <= cus && kb >= (f32 ? 440 : k_sel < 64 ? 400 : 240) ? 2 : 1;
}
// Whether a row's vectors with an element above the threshold come so thinly that a ring of kRingSmall slots, expanded
// beyond kRingExpand, loses one less than once in a million rows.
bool sparse_hits(tslt_dtype dt, int64_t V, int nt, const tslt::TruncateParams& p) {
  const int E = 16 / elem_bytes(dt);
  const double f = std::min(1.0, double(tslt::kBatch) * nt * E / double(V));
  const double hits = -nt * std::log(1.0 - double(p.jprime) / nt) / f;         // expected above the threshold
  const double h = 1.0 - std::pow(1.0 - std::min(1.0, hits / double(V)), E);   // ... of a vector
  return 128.0 * h + 5.0 * std::sqrt(128.0 * h) <= tslt::kRingSmall - tslt::kRingExpand;
}
// Whether 512 threads take a row: where every row has a compute unit to itself (but for the shortest, of few tiles more than
// the sample or less than that, where there is little to gain: 70 fp32 rows of 9088 9.8 us by 256 threads, 9.4 by 512; binary16
// 9.6 / 9.5; 16000 10.7 / 10.0 and 10.1 / 9.7),
// and up to three rows for two compute units if a row is neither short nor very long (us by 256 / 512 threads, 306
// rows: bfloat16 16000 11.1 / 11.5, 41000 15.4 / 16.3, 82000 21.8 / 20.7, 128256 28.9 / 24.4, 256000 46.0 / 40.3; fp32 16000 12.2 /
// 12.9, 60000 23.9 / 20.1, 128256 41.0 / 36.4, 213696 54.9 / 55.8, 256000 63.5 / 67.4.  Sets of 64; the lines are on the safe side:
// 25240 fp32 values 15.7 / 15.0, 180000 53.3 / 49.1.)
bool tall_rows(tslt_dtype dt, int64_t V, int64_t rows) {
  const int64_t cus = tslt::compute_units(), kb = V * elem_bytes(dt) >> 10;
  if (rows <= cus) return V >= 10240;
  return 2 * rows <= 3 * cus && kb >= 160 && kb < 700;
}
// What a call whose rows are shared has to be given, whatever is selected (a smaller selection has fewer candidates, and no more workgroups).
size_t truncate_share_bytes(tslt_dtype dt, int64_t rows, int64_t V, int32_t k_cap) {
  const int parts = truncate_parts(dt, V, rows, k_cap);
  if (parts == 1 || k_cap < 1 || k_cap > TSLT_MAX_K_CAP) return 0;
  tslt::TruncateParams p{};
  p.k_sel = k_cap;
  plan_truncate(dt, V, tslt::kTallThreads, p);
  return p.jprime > 0 ? tslt::truncate_part_bytes(rows, parts, p.sort_cap) : 0;
}
// The shapes of the truncation kernel (see truncate.h): 512 threads for such rows, but not where a row may be redone under
// 256 threads because its large logits are many (sets of more than a few per cent of the row: its status tells, and does
// not depend on the batch.  A row whose large logits are crowded together may still lose ring slots under 256 threads
// alone, and say so).  Else 256: eight workgroups of this footprint on a compute unit, the wide shape; else the deep one.
template <typename T> hipError_t launch_truncate(tslt_dtype dt, tslt::TruncateParams& p, void* ws, size_t ws_bytes, hipStream_t s) {
  constexpr int NT = tslt::kTruncThreads, TT = tslt::kTallThreads;
  const size_t lds = plan_truncate(dt, p.V, NT, p);
  if (tall_rows(dt, p.V, p.rows) && p.jprime > 0 && sparse_hits(dt, p.V, NT, p)) {
    tslt::TruncateParams tall = p;
    const size_t tall_lds = plan_truncate(dt, p.V, TT, tall);
    if (tall.jprime > 0) {
      tall.parts = truncate_parts(dt, p.V, p.rows, p.k_sel);
      if (tall.parts > 1 && ws != nullptr && reinterpret_cast<uintptr_t>(ws) % 256 == 0 &&
          ws_bytes >= tslt::truncate_part_bytes(p.rows, tall.parts, tall.sort_cap)) {
        tall.part_words = reinterpret_cast<uint64_t*>(ws);
        tall.part_found = tall.part_words + p.rows * tall.parts;
        tall.tag = tslt::next_tag();
        return launch_truncate_shape<T, TT, tslt::kStagesDeep, tslt::kWavesDeep, true>(tall, tall_lds, s);
      }
      return launch_truncate_shape<T, TT, tslt::kStagesDeep, tslt::kWavesDeep>(tall, tall_lds, s);
    }
  }
  if (8 * (lds + sizeof(tslt::TruncateShared) + 256) <= kMaxLds)
    return launch_truncate_shape<T, NT, tslt::kStagesWide, tslt::kWavesWide>(p, lds, s);
  return launch_truncate_shape<T, NT, tslt::kStagesDeep, tslt::kWavesDeep>(p, lds, s);
}

}  // namespace

extern "C" {

int tslt_version(void) { return 100; }

const char* tslt_last_error(void) { return g_last_error.c_str(); }

size_t tslt_workspace_bytes(int op, int64_t n_outer, int64_t n_inner, int64_t V, int32_t k_cap) {
  if (n_outer <= 0 || V <= 0) return 0;
  switch (op) {
    case TSLT_OP_VERIFY:
      return tslt::verify_workspace_bytes(n_outer, n_inner, V, k_cap);
    case TSLT_OP_TRUNCATE_SHARED:
      return std::max({truncate_share_bytes(TSLT_F32, n_outer, V, k_cap), truncate_share_bytes(TSLT_BF16, n_outer, V, k_cap),
                       truncate_share_bytes(TSLT_F16, n_outer, V, k_cap)});
    case TSLT_OP_VERIFY_TREE:
      return n_inner > 0 ? tslt::tree_workspace_bytes(n_outer, n_inner, V, true) : 0;
    case TSLT_OP_VERIFY_TREE_PATH:
      return n_inner > 0 ? tslt::tree_workspace_bytes(n_outer, n_inner, V, false) : 0;
    default:
      return 0;
  }
}

// tslt_truncate and tslt_truncate_sample: the second also draws from q_hat in the same launch.
static int truncate_impl(const void* logits, tslt_dtype dt, int64_t rows, int64_t V, int64_t row_stride,
                         float temperature, int32_t top_k, float top_p, int32_t k_cap, tslt_dtype payload, int32_t* out_idx,
                         float* out_logit, float* out_prob, int32_t* out_count, float* out_mass, int32_t* status,
                         const float* u, int32_t n_samples, int32_t without_replacement, int32_t* out_token, int32_t* out_slot,
                         void* ws, size_t ws_bytes, void* stream) {
  if (!valid_dtype(dt)) return fail(TSLT_ERR_INVALID_ARG, "tslt_truncate: unknown dtype %d", int(dt));
  if (rows < 0 || V <= 0 || row_stride < V) return fail(TSLT_ERR_INVALID_ARG, "tslt_truncate: bad shape rows=%lld V=%lld stride=%lld", (long long)rows, (long long)V, (long long)row_stride);
  if (row_too_long(V, dt) || rows > 0x7FFFFFFF) return fail(TSLT_ERR_UNSUPPORTED, "tslt_truncate: rows must fit 31 bits, a row 4 GiB");
  if (!(temperature > 0.0f) || !std::isfinite(temperature)) return fail(TSLT_ERR_INVALID_ARG, "tslt_truncate: temperature must be > 0");
  if (k_cap < 1 || k_cap > TSLT_MAX_K_CAP) return fail(TSLT_ERR_UNSUPPORTED, "tslt_truncate: k_cap must be in 1..%d", TSLT_MAX_K_CAP);
  if (top_k < 0 || !(top_p >= 0.0f)) return fail(TSLT_ERR_INVALID_ARG, "tslt_truncate: top_k and top_p must be >= 0");
  if (payload != TSLT_F32 && payload != TSLT_BF16 && payload != TSLT_F16) return fail(TSLT_ERR_INVALID_ARG, "tslt_truncate: unknown payload format %d", int(payload));
  if (rows == 0) return TSLT_OK;
  if (!logits || !out_idx || !out_logit || !out_count) return fail(TSLT_ERR_INVALID_ARG, "tslt_truncate: null pointer");
  if (reinterpret_cast<uintptr_t>(logits) % elem_bytes(dt)) return fail(TSLT_ERR_INVALID_ARG, "tslt_truncate: logits not aligned to their element type");

  tslt::TruncateParams p{};
  p.logits = logits; p.rows = rows; p.V = V; p.row_stride = row_stride;
  p.rT = reciprocal_temperature(temperature);
  p.k2 = log2e_over_T(p.rT);
  p.top_p = (top_p > 0.0f && top_p < 1.0f) ? top_p : 0.0f;
  p.k_cap = k_cap;
  p.payload = int(payload);
  p.k_sel = (top_k > 0 && top_k < k_cap) ? top_k : k_cap;
  p.out_idx = out_idx; p.out_logit = out_logit; p.out_prob = out_prob; p.out_count = out_count;
  p.out_mass = out_mass; p.status = status;
  p.u = u; p.n_samples = n_samples; p.without_replacement = without_replacement ? 1 : 0;
  p.out_token = out_token; p.out_slot = out_slot;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  hipError_t e = dt == TSLT_BF16 ? launch_truncate<tslt::Bf16>(dt, p, ws, ws_bytes, s)
                 : dt == TSLT_F16 ? launch_truncate<tslt::F16>(dt, p, ws, ws_bytes, s) : launch_truncate<float>(dt, p, ws, ws_bytes, s);
  if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute");
  if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "tslt_truncate launch");
  return TSLT_OK;
}

int tslt_truncate(const void* logits, tslt_dtype dt, int64_t rows, int64_t V, int64_t row_stride,
                  float temperature, int32_t top_k, float top_p, int32_t k_cap, tslt_dtype payload, int32_t* out_idx,
                  float* out_logit, float* out_prob, int32_t* out_count, float* out_mass, int32_t* status,
                  void* ws, size_t ws_bytes, void* stream) {
  return truncate_impl(logits, dt, rows, V, row_stride, temperature, top_k, top_p, k_cap, payload, out_idx, out_logit, out_prob,
                       out_count, out_mass, status, nullptr, 0, 0, nullptr, nullptr, ws, ws_bytes, stream);
}

int tslt_truncate_sample(const void* logits, tslt_dtype dt, int64_t rows, int64_t V, int64_t row_stride,
                         float temperature, int32_t top_k, float top_p, int32_t k_cap, tslt_dtype payload, int32_t* out_idx,
                         float* out_logit, float* out_prob, int32_t* out_count, float* out_mass, int32_t* status,
                         const float* u, int32_t n_samples, int32_t without_replacement, int32_t* out_token, int32_t* out_slot,
                         void* ws, size_t ws_bytes, void* stream) {
  if (n_samples < 1 || n_samples > TSLT_MAX_BRANCH)
    return fail(TSLT_ERR_INVALID_ARG, "tslt_truncate_sample: n_samples must be in 1..%d", TSLT_MAX_BRANCH);
  if (rows > 0 && (!u || !out_token)) return fail(TSLT_ERR_INVALID_ARG, "tslt_truncate_sample: null pointer");
  return truncate_impl(logits, dt, rows, V, row_stride, temperature, top_k, top_p, k_cap, payload, out_idx, out_logit, out_prob,
                       out_count, out_mass, status, u, n_samples, without_replacement, out_token, out_slot, ws, ws_bytes, stream);
}

int64_t tslt_pack_bound_words(int64_t rows, int32_t k_cap, int64_t V) {
  if (rows <= 0 || k_cap < 1 || k_cap > TSLT_MAX_K_CAP || V < 1 || V > 0x7FFFFFFF) return 0;
  return rows * tslt::wire_row_words(k_cap, tslt::wire_index_bits(V));
}

static int pack_impl(bool clear, const int32_t* idx, const float* logit, const int32_t* count, int64_t rows, int32_t k_cap,
                     int64_t V, tslt_dtype payload, uint32_t* out_words, int64_t out_capacity_words, int64_t* out_row_offset,
                     void* stream) {
  if (rows < 0 || V < 1 || V > 0x7FFFFFFF) return fail(TSLT_ERR_INVALID_ARG, "tslt_pack: bad shape");
  if (k_cap < 1 || k_cap > TSLT_MAX_K_CAP) return fail(TSLT_ERR_UNSUPPORTED, "tslt_pack: k_cap must be in 1..%d", TSLT_MAX_K_CAP);
  if (payload != TSLT_BF16 && payload != TSLT_F16) return fail(TSLT_ERR_INVALID_ARG, "tslt_pack: the value format must be bfloat16 or binary16");
  if (!out_row_offset) return fail(TSLT_ERR_INVALID_ARG, "tslt_pack: null pointer");
  if (rows > 0 && (!idx || !logit || !count || !out_words)) return fail(TSLT_ERR_INVALID_ARG, "tslt_pack: null pointer");
  if (out_capacity_words < tslt_pack_bound_words(rows, k_cap, V))
    return fail(TSLT_ERR_WORKSPACE, "tslt_pack: room for %lld words, %lld may be needed", (long long)out_capacity_words,
                (long long)tslt_pack_bound_words(rows, k_cap, V));
  tslt::WireParams p{};
  p.idx = idx; p.logit = logit; p.count = count; p.rows = rows; p.k_cap = k_cap; p.b_idx = tslt::wire_index_bits(V);
  p.payload = int(payload); p.words = out_words; p.row_offset = out_row_offset;
  p.clear = clear ? 1 : 0;
  p.rows_per = tslt::wire_rows_per_group(rows);
  const int64_t groups = rows > 0 ? (rows + p.rows_per - 1) / p.rows_per : 1;      // (no rows: the total alone)
  const bool narrow = tslt::wire_row_words(k_cap, p.b_idx) <= 64;                  // a word a lane
  hipLaunchKernelGGL((narrow ? tslt::wire_pack_kernel<1> : tslt::wire_pack_kernel<4>), dim3(unsigned(groups)), dim3(tslt::kPackThreads), 0,
                     reinterpret_cast<hipStream_t>(stream), p);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "tslt_pack launch");
  return TSLT_OK;
}

int tslt_pack(const int32_t* idx, const float* logit, const int32_t* count, int64_t rows, int32_t k_cap, int64_t V,
              tslt_dtype payload, uint32_t* out_words, int64_t out_capacity_words, int64_t* out_row_offset, void* stream) {
  return pack_impl(false, idx, logit, count, rows, k_cap, V, payload, out_words, out_capacity_words, out_row_offset, stream);
}

int tslt_pack_cleared(const int32_t* idx, const float* logit, const int32_t* count, int64_t rows, int32_t k_cap, int64_t V,
                      tslt_dtype payload, uint32_t* out_words, int64_t out_capacity_words, int64_t* out_row_offset,
                      void* stream) {
  return pack_impl(true, idx, logit, count, rows, k_cap, V, payload, out_words, out_capacity_words, out_row_offset, stream);
}

int tslt_unpack(const uint32_t* words, const int64_t* row_offset, int64_t rows, int32_t k_cap, int64_t V,
                tslt_dtype payload, int32_t* out_idx, float* out_logit, int32_t* out_count, void* stream) {
  if (rows < 0 || V < 1 || V > 0x7FFFFFFF) return fail(TSLT_ERR_INVALID_ARG, "tslt_unpack: bad shape");
  if (k_cap < 1 || k_cap > TSLT_MAX_K_CAP) return fail(TSLT_ERR_UNSUPPORTED, "tslt_unpack: k_cap must be in 1..%d", TSLT_MAX_K_CAP);
  if (payload != TSLT_BF16 && payload != TSLT_F16) return fail(TSLT_ERR_INVALID_ARG, "tslt_unpack: the value format must be bfloat16 or binary16");
  if (rows == 0) return TSLT_OK;
  if (!words || !row_offset || !out_idx || !out_logit || !out_count) return fail(TSLT_ERR_INVALID_ARG, "tslt_unpack: null pointer");
  tslt::WireParams p{};
  p.in_words = words; p.in_row_offset = row_offset; p.rows = rows; p.k_cap = k_cap; p.b_idx = tslt::wire_index_bits(V);
  p.payload = int(payload); p.out_idx = out_idx; p.out_logit = out_logit; p.out_count = out_count;
  hipLaunchKernelGGL(tslt::wire_unpack_kernel, dim3(unsigned(rows)), dim3(64), 0, reinterpret_cast<hipStream_t>(stream), p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "tslt_unpack launch");
  return TSLT_OK;
}

int tslt_sample(const int32_t* idx, const float* logit, const int32_t* count, int64_t rows, int32_t k_cap,
                const float* u, int32_t n_samples, int32_t without_replacement, int32_t* out_token,
                int32_t* out_slot, void* stream) {
  if (rows < 0 || rows > 0x7FFFFFFF) return fail(TSLT_ERR_INVALID_ARG, "tslt_sample: bad row count");
  if (k_cap < 1 || k_cap > TSLT_MAX_K_CAP) return fail(TSLT_ERR_UNSUPPORTED, "tslt_sample: k_cap must be in 1..%d", TSLT_MAX_K_CAP);
  if (n_samples < 0) return fail(TSLT_ERR_INVALID_ARG, "tslt_sample: n_samples < 0");
  if (rows == 0 || n_samples == 0) return TSLT_OK;
  if (!idx || !logit || !count || !u || !out_token) return fail(TSLT_ERR_INVALID_ARG, "tslt_sample: null pointer");
  tslt::SampleParams p{idx, logit, count, rows, k_cap, u, n_samples, without_replacement ? 1 : 0, out_token, out_slot};
  hipLaunchKernelGGL(tslt::sample_kernel, dim3(unsigned(rows)), dim3(64), 0, reinterpret_cast<hipStream_t>(stream), p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "tslt_sample launch");
  return TSLT_OK;
}

static int verify_impl(int phases, int stage0, const char* name, const void* target_logits, tslt_dtype dt, int64_t B,
                       int32_t gamma, int64_t V, int64_t row_stride, float target_temperature, const int32_t* q_idx,
                       const float* q_logit, const int32_t* q_count, int32_t k_cap, const int32_t* draft_tokens,
                       const float* u_accept, const float* u_resample, int32_t* out_accept_len, int32_t* out_tokens,
                       float* out_ratio, float* out_beta, int32_t* status, void* ws, size_t ws_bytes, void* stream) {
  if (!valid_dtype(dt)) return fail(TSLT_ERR_INVALID_ARG, "%s: unknown dtype %d", name, int(dt));
  if (B < 0 || gamma < 1 || V <= 0 || row_stride < V) return fail(TSLT_ERR_INVALID_ARG, "%s: bad shape", name);
  if (V > 0x7FFFFFFF || B * (int64_t(gamma) + 1) > 0x7FFFFFFF) return fail(TSLT_ERR_UNSUPPORTED, "%s: sizes must fit 31 bits", name);
  if (gamma > 4096) return fail(TSLT_ERR_UNSUPPORTED, "%s: gamma > 4096", name);
  if (stage0 < 0) return fail(TSLT_ERR_INVALID_ARG, "%s: first_stage must be >= 0", name);
  if (tslt::row_segments(V, 16 / elem_bytes(dt)) + 2 > tslt::kBlock)
    return fail(TSLT_ERR_UNSUPPORTED, "%s: V too large (at most %d elements of this type)", name, (tslt::kBlock - 2) * tslt::kSegVecsTotal * (16 / elem_bytes(dt)) - 16);
  if (B * int64_t(tslt::row_segments(V)) > 0x7FFFFFFF) return fail(TSLT_ERR_UNSUPPORTED, "%s: B too large", name);
  if (!(target_temperature > 0.0f) || !std::isfinite(target_temperature)) return fail(TSLT_ERR_INVALID_ARG, "%s: temperature must be > 0", name);
  if (k_cap < 1 || k_cap > TSLT_MAX_K_CAP) return fail(TSLT_ERR_UNSUPPORTED, "%s: k_cap must be in 1..%d", name, TSLT_MAX_K_CAP);
  if (B == 0) return TSLT_OK;
  if (!target_logits || !q_idx || !q_logit || !q_count || !draft_tokens || !u_accept || !u_resample ||
      !out_accept_len || !out_tokens)
    return fail(TSLT_ERR_INVALID_ARG, "%s: null pointer", name);
  if (reinterpret_cast<uintptr_t>(target_logits) % elem_bytes(dt)) return fail(TSLT_ERR_INVALID_ARG, "%s: logits not aligned to their element type", name);
  const size_t need = tslt::verify_least_workspace_bytes(B, gamma);
  if (!ws || ws_bytes < need || reinterpret_cast<uintptr_t>(ws) % 256)
    return fail(TSLT_ERR_WORKSPACE, "%s: workspace of %zu bytes, 256-byte aligned, required", name, need);

  tslt::VerifyParams p{};
  p.target = target_logits; p.B = B; p.gamma = gamma; p.V = V; p.row_stride = row_stride;
  p.rT = reciprocal_temperature(target_temperature);
  p.k2 = log2e_over_T(p.rT);
  p.q_idx = q_idx; p.q_logit = q_logit; p.q_count = q_count; p.k_cap = k_cap;
  p.draft_tokens = draft_tokens; p.u_accept = u_accept; p.u_resample = u_resample;
  p.out_accept_len = out_accept_len; p.out_tokens = out_tokens; p.out_ratio = out_ratio; p.out_beta = out_beta;
  p.status = status;
  p.stage0 = stage0 >= gamma ? 0 : stage0;
  tslt::verify_carve_workspace(p, ws, ws_bytes, 16 / elem_bytes(dt));
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  hipError_t e = dt == TSLT_BF16 ? tslt::launch_verify<tslt::Bf16>(p, s, phases)
                 : dt == TSLT_F16 ? tslt::launch_verify<tslt::F16>(p, s, phases) : tslt::launch_verify<float>(p, s, phases);
  if (e != hipSuccess) return hip_fail(e, name);
  return TSLT_OK;
}

#define TSLT_VERIFY_ARGS                                                                                          \
  const void *target_logits, tslt_dtype dt, int64_t B, int32_t gamma, int64_t V, int64_t row_stride,             \
      float target_temperature, const int32_t *q_idx, const float *q_logit, const int32_t *q_count, int32_t k_cap, \
      const int32_t *draft_tokens, const float *u_accept, const float *u_resample, int32_t *out_accept_len,       \
      int32_t *out_tokens, float *out_ratio, float *out_beta, int32_t *status, void *ws, size_t ws_bytes, void *stream
#define TSLT_VERIFY_PASS                                                                                           \
  target_logits, dt, B, gamma, V, row_stride, target_temperature, q_idx, q_logit, q_count, k_cap, draft_tokens,   \
      u_accept, u_resample, out_accept_len, out_tokens, out_ratio, out_beta, status, ws, ws_bytes, stream

int tslt_verify(TSLT_VERIFY_ARGS) { return verify_impl(3, 0, "tslt_verify", TSLT_VERIFY_PASS); }
int tslt_verify_accept(TSLT_VERIFY_ARGS) { return verify_impl(1, 0, "tslt_verify_accept", TSLT_VERIFY_PASS); }
int tslt_verify_resample(TSLT_VERIFY_ARGS) { return verify_impl(2, 0, "tslt_verify_resample", TSLT_VERIFY_PASS); }
int tslt_verify_staged(TSLT_VERIFY_ARGS, int32_t first_stage) {
  return verify_impl(3, first_stage, "tslt_verify_staged", TSLT_VERIFY_PASS);
}
int tslt_verify_accept_staged(TSLT_VERIFY_ARGS, int32_t first_stage) {
  return verify_impl(1, first_stage, "tslt_verify_accept_staged", TSLT_VERIFY_PASS);
}

int tslt_verify_static(const void* target_logits, tslt_dtype dt, int64_t B, int32_t gamma, int64_t V, int64_t row_stride,
                       float target_temperature, const int32_t* q_idx, const float* q_logit, const int32_t* q_count,
                       int32_t k_cap, const int32_t* draft_tokens, const float* u_accept, const float* u_resample,
                       int32_t* out_accept_len, int32_t* out_tokens, float* out_ratio, float* out_beta, int32_t* status,
                       void* stream) {
  const char* name = "tslt_verify_static";
  if (B < 0 || gamma < 1) return fail(TSLT_ERR_INVALID_ARG, "%s: bad shape", name);
  if (B > TSLT_STATIC_MAX_POSITIONS || B * int64_t(gamma) > TSLT_STATIC_MAX_POSITIONS)
    return fail(TSLT_ERR_UNSUPPORTED, "%s: B * gamma = %lld positions, the static scratch array holds %d; use tslt_verify "
                "with a workspace", name, (long long)(B * int64_t(gamma)), TSLT_STATIC_MAX_POSITIONS);
  if (tslt::verify_least_workspace_bytes(B, gamma) > size_t(TSLT_STATIC_SCRATCH_BYTES))
    return fail(TSLT_ERR_UNSUPPORTED, "%s: the static scratch array is too small for this call", name);
  void* ptr = nullptr;
  const hipError_t e = scratch_on_current_device(&ptr);
  if (e != hipSuccess) return hip_fail(e, "tslt_verify_static: address of the scratch array");
  // every position's decision and status word is written by the acceptance kernel before the resampling
  // kernel reads it, so nothing in the array has to start at zero
  return verify_impl(3, 0, name, target_logits, dt, B, gamma, V, row_stride, target_temperature, q_idx, q_logit, q_count,
                     k_cap, draft_tokens, u_accept, u_resample, out_accept_len, out_tokens, out_ratio, out_beta, status, ptr,
                     size_t(TSLT_STATIC_SCRATCH_BYTES), stream);
}

int tslt_calibrate_read(const void* src, size_t bytes, int32_t n_blocks, uint32_t* sink, void* stream) {
  const char* name = "tslt_calibrate_read";
  if (!src || !sink) return fail(TSLT_ERR_INVALID_ARG, "%s: null pointer", name);
  if (reinterpret_cast<uintptr_t>(src) % 16) return fail(TSLT_ERR_INVALID_ARG, "%s: the buffer must be 16-byte aligned", name);
  if (n_blocks < 1) return fail(TSLT_ERR_INVALID_ARG, "%s: n_blocks must be >= 1", name);
  const size_t chunk = size_t(16) * tslt::kCalibUnroll * tslt::kBlock;       // bytes one workgroup reads per round
  if (bytes == 0 || bytes % (chunk * size_t(n_blocks)) != 0)
    return fail(TSLT_ERR_INVALID_ARG, "%s: bytes must be a positive multiple of n_blocks * %zu", name, chunk);
  const uint64_t vecs_per_block = bytes / 16 / size_t(n_blocks);
  hipLaunchKernelGGL(tslt::calibrate_read_kernel, dim3(unsigned(n_blocks)), dim3(tslt::kBlock), 0,
                     reinterpret_cast<hipStream_t>(stream), reinterpret_cast<const uint4*>(src), vecs_per_block, sink);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, name);
  return TSLT_OK;
}

int tslt_truncation_stats(const void* target_logits, tslt_dtype dt, int64_t rows, int64_t V, int64_t row_stride,
                          float target_temperature, const int32_t* q_idx, const float* q_logit, const int32_t* q_count,
                          int32_t k_cap, const int32_t* k_list, int32_t n_k, float* out_keep, float* out_beta,
                          int32_t* status, void* stream) {
  const char* name = "tslt_truncation_stats";
  if (!valid_dtype(dt)) return fail(TSLT_ERR_INVALID_ARG, "%s: unknown dtype %d", name, int(dt));
  if (rows < 0 || V <= 0 || row_stride < V) return fail(TSLT_ERR_INVALID_ARG, "%s: bad shape", name);
  if (row_too_long(V, dt) || rows > 0x7FFFFFFF) return fail(TSLT_ERR_UNSUPPORTED, "%s: rows must fit 31 bits, a row 4 GiB", name);
  if (!(target_temperature > 0.0f) || !std::isfinite(target_temperature)) return fail(TSLT_ERR_INVALID_ARG, "%s: temperature must be > 0", name);
  if (k_cap < 1 || k_cap > TSLT_MAX_K_CAP) return fail(TSLT_ERR_UNSUPPORTED, "%s: k_cap must be in 1..%d", name, TSLT_MAX_K_CAP);
  if (n_k < 1 || n_k > tslt::kMaxStatK) return fail(TSLT_ERR_UNSUPPORTED, "%s: between 1 and %d values of K", name, tslt::kMaxStatK);
  if (!k_list) return fail(TSLT_ERR_INVALID_ARG, "%s: null pointer", name);
  if (rows == 0) return TSLT_OK;
  if (!target_logits || !q_idx || !q_logit || !q_count || !out_keep || !out_beta) return fail(TSLT_ERR_INVALID_ARG, "%s: null pointer", name);
  if (reinterpret_cast<uintptr_t>(target_logits) % elem_bytes(dt)) return fail(TSLT_ERR_INVALID_ARG, "%s: logits not aligned to their element type", name);
  tslt::StatsParams p{};
  p.target = target_logits; p.rows = rows; p.V = V; p.row_stride = row_stride;
  p.rT = reciprocal_temperature(target_temperature);
  p.k2 = log2e_over_T(p.rT);
  p.q_idx = q_idx; p.q_logit = q_logit; p.q_count = q_count; p.k_cap = k_cap;
  p.n_k = n_k;
  for (int j = 0; j < n_k; ++j) p.k_list[j] = k_list[j];
  p.out_keep = out_keep; p.out_beta = out_beta; p.status = status;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const dim3 grid{unsigned(rows)}, block{unsigned(tslt::kBlock)};
  if (dt == TSLT_BF16) hipLaunchKernelGGL(tslt::truncation_stats_kernel<tslt::Bf16>, grid, block, 0, s, p);
  else if (dt == TSLT_F16) hipLaunchKernelGGL(tslt::truncation_stats_kernel<tslt::F16>, grid, block, 0, s, p);
  else hipLaunchKernelGGL(tslt::truncation_stats_kernel<float>, grid, block, 0, s, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, name);
  return TSLT_OK;
}

int tslt_multicandidate_stats(const void* target_logits, tslt_dtype dt, int64_t rows, int64_t V, int64_t row_stride,
                              float target_temperature, const int32_t* q_idx, const float* q_logit, const int32_t* q_count,
                              int32_t k_cap, int32_t k, float* out_beta, float* out_theta, int32_t* status, void* stream) {
  const char* name = "tslt_multicandidate_stats";
  if (!valid_dtype(dt)) return fail(TSLT_ERR_INVALID_ARG, "%s: unknown dtype %d", name, int(dt));
  if (rows < 0 || V <= 0 || row_stride < V) return fail(TSLT_ERR_INVALID_ARG, "%s: bad shape", name);
  if (row_too_long(V, dt) || rows > 0x7FFFFFFF) return fail(TSLT_ERR_UNSUPPORTED, "%s: rows must fit 31 bits, a row 4 GiB", name);
  if (!(target_temperature > 0.0f) || !std::isfinite(target_temperature)) return fail(TSLT_ERR_INVALID_ARG, "%s: temperature must be > 0", name);
  if (k_cap < 1 || k_cap > TSLT_MAX_K_CAP) return fail(TSLT_ERR_UNSUPPORTED, "%s: k_cap must be in 1..%d", name, TSLT_MAX_K_CAP);
  if (k < 1 || k > TSLT_MAX_BRANCH) return fail(TSLT_ERR_UNSUPPORTED, "%s: between 1 and %d candidates", name, TSLT_MAX_BRANCH);
  if (rows == 0) return TSLT_OK;
  if (!target_logits || !q_idx || !q_logit || !q_count || !out_beta || !out_theta) return fail(TSLT_ERR_INVALID_ARG, "%s: null pointer", name);
  if (reinterpret_cast<uintptr_t>(target_logits) % elem_bytes(dt)) return fail(TSLT_ERR_INVALID_ARG, "%s: logits not aligned to their element type", name);
  tslt::McStatsParams p{};
  p.target = target_logits; p.rows = rows; p.V = V; p.row_stride = row_stride;
  p.rT = reciprocal_temperature(target_temperature);
  p.k2 = log2e_over_T(p.rT);
  p.q_idx = q_idx; p.q_logit = q_logit; p.q_count = q_count; p.k_cap = k_cap; p.k = k;
  p.out_beta = out_beta; p.out_theta = out_theta; p.status = status;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const dim3 grid{unsigned(rows)}, block{unsigned(tslt::kBlock)};
  if (dt == TSLT_BF16) hipLaunchKernelGGL(tslt::multicandidate_stats_kernel<tslt::Bf16>, grid, block, 0, s, p);
  else if (dt == TSLT_F16) hipLaunchKernelGGL(tslt::multicandidate_stats_kernel<tslt::F16>, grid, block, 0, s, p);
  else hipLaunchKernelGGL(tslt::multicandidate_stats_kernel<float>, grid, block, 0, s, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, name);
  return TSLT_OK;
}

int tslt_verify_tree(const void* target_logits, tslt_dtype dt, int64_t B, int64_t V, int64_t row_stride,
                     float target_temperature, int32_t depth, const int32_t* expansion, const int32_t* q_idx,
                     const float* q_logit, const int32_t* q_count, int32_t k_cap, const int32_t* cand_tokens,
                     const float* u_accept, const float* u_resample, int32_t without_replacement,
                     int32_t* out_node_token, int32_t* out_node_slot, int32_t* out_seq, int32_t* out_len,
                     float* out_ratio, float* out_beta, int32_t* status, void* ws, size_t ws_bytes, void* stream) {
  const char* name = "tslt_verify_tree";
  if (!valid_dtype(dt)) return fail(TSLT_ERR_INVALID_ARG, "%s: unknown dtype %d", name, int(dt));
  if (B < 0 || V <= 0 || row_stride < V) return fail(TSLT_ERR_INVALID_ARG, "%s: bad shape", name);
  if (depth < 1 || !expansion) return fail(TSLT_ERR_INVALID_ARG, "%s: depth must be >= 1 and expansion given", name);
  if (depth > TSLT_MAX_TREE_DEPTH) return fail(TSLT_ERR_UNSUPPORTED, "%s: depth > %d", name, TSLT_MAX_TREE_DEPTH);
  if (!(target_temperature > 0.0f) || !std::isfinite(target_temperature)) return fail(TSLT_ERR_INVALID_ARG, "%s: temperature must be > 0", name);
  if (k_cap < 1 || k_cap > TSLT_MAX_K_CAP) return fail(TSLT_ERR_UNSUPPORTED, "%s: k_cap must be in 1..%d", name, TSLT_MAX_K_CAP);
  if (tslt::row_segments(V, 16 / elem_bytes(dt)) + 2 > tslt::kBlock || V > 0x7FFFFFFF) return fail(TSLT_ERR_UNSUPPORTED, "%s: V too large", name);
  tslt::TreeParams p{};
  int64_t width = 1, n_nodes = 1;
  p.offsets[0] = 0;
  for (int l = 0; l < depth; ++l) {
    if (expansion[l] < 1 || expansion[l] > TSLT_MAX_BRANCH)
      return fail(TSLT_ERR_UNSUPPORTED, "%s: expansion[%d] must be in 1..%d", name, l, TSLT_MAX_BRANCH);
    p.expansion[l] = expansion[l];
    p.offsets[l + 1] = int(n_nodes);
    width *= expansion[l];
    n_nodes += width;
    if (n_nodes > (1 << 24)) return fail(TSLT_ERR_UNSUPPORTED, "%s: tree too large", name);
  }
  p.offsets[depth + 1] = int(n_nodes);
  p.n_nodes = int(n_nodes);
  p.n_int = int(n_nodes - width);
  p.depth = depth;
  const bool all_nodes = out_node_token != nullptr || out_node_slot != nullptr;
  p.all_nodes = all_nodes ? 1 : 0;
  if (B * (all_nodes ? n_nodes : 1) * tslt::row_segments(V) > 0x7FFFFFFF || B * n_nodes > 0x7FFFFFFF)
    return fail(TSLT_ERR_UNSUPPORTED, "%s: B * nodes too large", name);
  if (B == 0) return TSLT_OK;
  if (!target_logits || !q_idx || !q_logit || !q_count || !cand_tokens || !u_accept || !u_resample || !out_seq || !out_len)
    return fail(TSLT_ERR_INVALID_ARG, "%s: null pointer", name);
  if (reinterpret_cast<uintptr_t>(target_logits) % elem_bytes(dt)) return fail(TSLT_ERR_INVALID_ARG, "%s: logits not aligned to their element type", name);
  const size_t need = tslt::tree_least_workspace_bytes(B, n_nodes, V, all_nodes);
  if (!ws || ws_bytes < need || reinterpret_cast<uintptr_t>(ws) % 256)
    return fail(TSLT_ERR_WORKSPACE, "%s: workspace of %zu bytes, 256-byte aligned, required", name, need);
  p.target = target_logits; p.B = B; p.V = V; p.row_stride = row_stride;
  p.rT = reciprocal_temperature(target_temperature);
  p.k2 = log2e_over_T(p.rT);
  p.q_idx = q_idx; p.q_logit = q_logit; p.q_count = q_count; p.k_cap = k_cap;
  p.cand_tokens = cand_tokens; p.u_accept = u_accept; p.u_resample = u_resample;
  p.wor = without_replacement ? 1 : 0;
  p.out_node_token = out_node_token; p.out_node_slot = out_node_slot; p.out_seq = out_seq; p.out_len = out_len;
  p.out_ratio = out_ratio; p.out_beta = out_beta; p.status = status;
  tslt::tree_carve_workspace(p, ws, ws_bytes, 16 / elem_bytes(dt));
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  hipError_t e = dt == TSLT_BF16 ? tslt::launch_verify_tree<tslt::Bf16>(p, s)
                 : dt == TSLT_F16 ? tslt::launch_verify_tree<tslt::F16>(p, s) : tslt::launch_verify_tree<float>(p, s);
  if (e != hipSuccess) return hip_fail(e, name);
  return TSLT_OK;
}

}  // extern "C"
