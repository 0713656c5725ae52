// Device-side helpers shared by the TSLT kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "bins.h"

namespace tslt {

// ---- host side: what is looked up or set once per device, so that a call after the first on a device is
// nothing but argument checks and launches ----------------------------------------------------------------
constexpr int kMaxDevices = 64;
inline int current_device_slot() {
  int d = 0;
  if (hipGetDevice(&d) != hipSuccess || d < 0 || d >= kMaxDevices) d = 0;
  return d;
}
// Lets `Kernel` be launched with up to `bytes` of dynamic LDS on the current device (needed above 48 KB).
template <auto Kernel> inline hipError_t allow_dynamic_lds(int bytes) {
  static std::atomic<int> granted[kMaxDevices];
  const int d = current_device_slot();
  if (granted[d].load(std::memory_order_relaxed) >= bytes) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(Kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) granted[d].store(bytes, std::memory_order_relaxed);
  return e;
}
template <auto Kernel> struct KernelTag { static constexpr auto value = Kernel; };      // names a kernel in an argument
// Compute units of the current device (256 if the query fails).
inline int compute_units() {
  static std::atomic<int> cus[kMaxDevices];
  const int d = current_device_slot();
  int n = cus[d].load(std::memory_order_relaxed);
  if (n > 0) return n;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
    n = 256;
  cus[d].store(n, std::memory_order_relaxed);
  return n;
}

constexpr int kBlock = 256;            // threads per workgroup of the streaming kernels
constexpr int kWaves = kBlock / 64;
constexpr uint32_t kNegInfBits = 0xFF800000u;

struct Bf16 { uint16_t bits; };        // storage tag for bf16 rows
struct F16 { uint16_t bits; };         // storage tag for binary16 rows

template <typename T> struct ElemTraits;
template <> struct ElemTraits<float> {
  static constexpr int kPerVec = 4;    // elements per 16-byte vector
  static constexpr int kBytes = 4;
};
template <> struct ElemTraits<Bf16> {
  static constexpr int kPerVec = 8;
  static constexpr int kBytes = 2;
};
template <> struct ElemTraits<F16> {
  static constexpr int kPerVec = 8;
  static constexpr int kBytes = 2;
};

__device__ __forceinline__ float as_f32(uint32_t b) { return __uint_as_float(b); }
__device__ __forceinline__ uint32_t as_u32(float f) { return __float_as_uint(f); }

// A pointer into device memory, typed as such.  Where the compiler cannot prove that a pointer is global
// it emits flat loads; those also count against the LDS counter, so that every wait for an LDS access
// waits for them too and a kernel that prefetches rows while it works in LDS loses the overlap.
template <typename U> __device__ __forceinline__ const U __attribute__((address_space(1)))* as_global(const U* p) {
  return (const U __attribute__((address_space(1)))*)p;
}

// Element i of a 16-byte vector, widened exactly to fp32.
template <typename T> __device__ __forceinline__ void unpack(const uint4& w, float (&v)[ElemTraits<T>::kPerVec]);
template <> __device__ __forceinline__ void unpack<float>(const uint4& w, float (&v)[4]) {
  v[0] = as_f32(w.x); v[1] = as_f32(w.y); v[2] = as_f32(w.z); v[3] = as_f32(w.w);
}
template <> __device__ __forceinline__ void unpack<Bf16>(const uint4& w, float (&v)[8]) {
  v[0] = as_f32(w.x << 16); v[1] = as_f32(w.x & 0xFFFF0000u);
  v[2] = as_f32(w.y << 16); v[3] = as_f32(w.y & 0xFFFF0000u);
  v[4] = as_f32(w.z << 16); v[5] = as_f32(w.z & 0xFFFF0000u);
  v[6] = as_f32(w.w << 16); v[7] = as_f32(w.w & 0xFFFF0000u);
}

__device__ __forceinline__ float f16_lo(uint32_t w) { return float(__builtin_bit_cast(_Float16, uint16_t(w))); }
__device__ __forceinline__ float f16_hi(uint32_t w) { return float(__builtin_bit_cast(_Float16, uint16_t(w >> 16))); }
template <> __device__ __forceinline__ void unpack<F16>(const uint4& w, float (&v)[8]) {
  v[0] = f16_lo(w.x); v[1] = f16_hi(w.x);
  v[2] = f16_lo(w.y); v[3] = f16_hi(w.y);
  v[4] = f16_lo(w.z); v[5] = f16_hi(w.z);
  v[6] = f16_lo(w.w); v[7] = f16_hi(w.w);
}

// The scaled logits s = fl32(z * rT) of a vector (binary16: widened and multiplied by one instruction; adding -0 to
// the product keeps it as it is).
template <typename T> __device__ __forceinline__ void unpack_scaled(const uint4& w, float rT, float (&s)[ElemTraits<T>::kPerVec]) {
  unpack<T>(w, s);
#pragma unroll
  for (int e = 0; e < ElemTraits<T>::kPerVec; ++e) s[e] = __fmul_rn(s[e], rT);
}
template <> __device__ __forceinline__ void unpack_scaled<F16>(const uint4& w, float rT, float (&s)[8]) {
  const uint32_t x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    s[2 * k] = __builtin_fmaf(f16_lo(x[k]), rT, -0.0f);
    s[2 * k + 1] = __builtin_fmaf(f16_hi(x[k]), rT, -0.0f);
  }
}

template <typename T> __device__ __forceinline__ uint4 neg_inf_vec();
template <> __device__ __forceinline__ uint4 neg_inf_vec<float>() {
  return make_uint4(kNegInfBits, kNegInfBits, kNegInfBits, kNegInfBits);
}
template <> __device__ __forceinline__ uint4 neg_inf_vec<Bf16>() {
  return make_uint4(0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u);
}

template <> __device__ __forceinline__ uint4 neg_inf_vec<F16>() {
  return make_uint4(0xFC00FC00u, 0xFC00FC00u, 0xFC00FC00u, 0xFC00FC00u);
}

// Scalar load of element i of a row, any alignment of the element type.
template <typename T> __device__ __forceinline__ float load_elem(const void* row, int64_t i);
template <> __device__ __forceinline__ float load_elem<float>(const void* row, int64_t i) {
  return as_global(reinterpret_cast<const float*>(row))[i];
}
template <> __device__ __forceinline__ float load_elem<Bf16>(const void* row, int64_t i) {
  return as_f32(uint32_t(as_global(reinterpret_cast<const uint16_t*>(row))[i]) << 16);
}

template <> __device__ __forceinline__ float load_elem<F16>(const void* row, int64_t i) {
  return f16_lo(as_global(reinterpret_cast<const uint16_t*>(row))[i]);
}

// Order-preserving map fp32 -> uint32 (larger value, larger key).  -0.0 must be folded into +0.0 by
// the caller (add 0.0f) when the two have to compare equal.
__device__ __forceinline__ uint32_t mono_key(float v) {
  uint32_t b = as_u32(v);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key_to_f32(uint32_t k) {
  return as_f32((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}
constexpr uint32_t kKeyNegInf = 0x007FFFFFu;   // mono_key(-inf)
constexpr uint32_t kKeyPosInf = 0xFF800000u;   // mono_key(+inf)

// Candidate record: value key in the high word, inverted index in the low word, so that a plain
// descending sort of the 64-bit word gives "value descending, index ascending".
__device__ __forceinline__ uint64_t make_cand(float v, uint32_t idx) {
  return (uint64_t(mono_key(v + 0.0f)) << 32) | uint64_t(0xFFFFFFFFu - idx);
}
__device__ __forceinline__ float cand_value(uint64_t c) { return key_to_f32(uint32_t(c >> 32)); }
__device__ __forceinline__ uint32_t cand_index(uint64_t c) { return 0xFFFFFFFFu - uint32_t(c); }

// 16-byte streaming load (read-once data: do not keep it in the caches longer than needed).
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_vec_stream(const uint4* p) {
  u32x4_t r = __builtin_nontemporal_load(as_global(reinterpret_cast<const u32x4_t*>(p)));
  return make_uint4(r.x, r.y, r.z, r.w);
}
__device__ __forceinline__ uint4 load_vec(const uint4* p) {
  u32x4_t r = *as_global(reinterpret_cast<const u32x4_t*>(p));
  return make_uint4(r.x, r.y, r.z, r.w);
}

// A row's aligned body as a buffer: 16-byte loads through a resource descriptor take the row's base and size
// from scalar registers, a per-thread byte offset that never changes (lane * 16) from a vector register and
// the moving part of the address from a scalar one, so that a streaming loop spends no vector instruction on
// addresses; a load that reaches past the body's end returns zeros instead of faulting (the hardware checks
// the range of the whole offset, also where the scalar part alone lies far beyond the size: measured on gfx950), and the
// loops give such vectors the value they need afterwards.  The body must be below 4 GiB.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_buffer(const uint4* body, uint32_t nvec) {
  // (third dword: raw buffer of 32-bit data, the setting of the GFX9 family)
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(body), 0, int(nvec * 16u), 0x00020000);
}
__device__ __forceinline__ uint4 buffer_load_vec_stream(__amdgpu_buffer_rsrc_t r, uint32_t lane_bytes, uint32_t wave_bytes) {
  u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(r, int(lane_bytes), int(wave_bytes), 2);      // 2: nontemporal
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint4 buffer_load_vec(__amdgpu_buffer_rsrc_t r, uint32_t lane_bytes, uint32_t wave_bytes) {
  u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(r, int(lane_bytes), int(wave_bytes), 0);
  return make_uint4(v.x, v.y, v.z, v.w);
}
// max of three without the NaN-quieting moves the compiler adds around fmaxf (NaNs are found by other means)
__device__ __forceinline__ float max3f(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }
__device__ __forceinline__ int wave_id() { return threadIdx.x >> 6; }

__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ int lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi(uint32_t(mask >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(mask), 0));
}

// A condition that is the same in all lanes of a wave, as such: the compiler branches on it without masking lanes.
__device__ __forceinline__ bool same_in_wave(bool b) { return __builtin_amdgcn_readfirstlane(int(b)) != 0; }

// The value of one lane, named by a wave-uniform number, in all lanes (no LDS round trip).
__device__ __forceinline__ double lane_f64(double v, int src) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), src), __builtin_amdgcn_readlane(__double2loint(v), src));
}

// Cross-lane moves on the VALU's data-parallel-primitive path (no LDS round trip).  A lane whose source lies
// outside its row of 16, or that the row / bank mask leaves out, gets `old`.  Controls used here:
// row_shr:n = 0x110 + n (lane i reads lane i - n of its row), row_bcast:15 = 0x142 (lane 15 of every row to
// the whole next row), row_bcast:31 = 0x143 (lane 31 to rows 2 and 3).
template <int CTRL, int ROW_MASK = 0xF, int BANK_MASK = 0xF>
__device__ __forceinline__ int dpp_i32(int old, int v) {
  return __builtin_amdgcn_update_dpp(old, v, CTRL, ROW_MASK, BANK_MASK, false);
}
template <int CTRL, int ROW_MASK = 0xF, int BANK_MASK = 0xF>
__device__ __forceinline__ double dpp_f64(double old, double v) {
  const int lo = dpp_i32<CTRL, ROW_MASK, BANK_MASK>(__double2loint(old), __double2loint(v));
  const int hi = dpp_i32<CTRL, ROW_MASK, BANK_MASK>(__double2hiint(old), __double2hiint(v));
  return __hiloint2double(hi, lo);
}
// (a lane without a source gets 0 and nothing has to be prepared for it)
template <int CTRL> __device__ __forceinline__ double dpp_or_zero_f64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
// Inclusive scan over the 64 lanes of a wave with an associative operation `op` whose identity is `id`:
// four steps inside every row of 16, then the row totals are carried into the later rows.  Lane 63 ends up
// with the reduction over the wave.
template <typename Op> __device__ __forceinline__ int wave_scan_i32(int v, int id, Op op) {
  v = op(v, dpp_i32<0x111>(id, v));
  v = op(v, dpp_i32<0x112>(id, v));
  v = op(v, dpp_i32<0x114>(id, v));
  v = op(v, dpp_i32<0x118>(id, v));
  v = op(v, dpp_i32<0x142, 0xA>(id, v));
  v = op(v, dpp_i32<0x143, 0xC>(id, v));
  return v;
}
__device__ __forceinline__ int last_lane_i32(int v) { return __builtin_amdgcn_readlane(v, 63); }
__device__ __forceinline__ double last_lane_f64(double v) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63), __builtin_amdgcn_readlane(__double2loint(v), 63));
}

__device__ __forceinline__ int wave_incl_scan_i32(int v) { return wave_scan_i32(v, 0, [](int a, int b) { return a + b; }); }
// N sums at once: the steps of one fill the latencies of the others.
template <int N> __device__ __forceinline__ void wave_incl_scan_f64(double (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_or_zero_f64<0x111>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_or_zero_f64<0x112>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_or_zero_f64<0x114>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_or_zero_f64<0x118>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_f64<0x142, 0xA>(0.0, v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_f64<0x143, 0xC>(0.0, v[i]);
}
// Inclusive scan within each row of 16 lanes.
__device__ __forceinline__ double scan16_f64(double v) {
  v += dpp_or_zero_f64<0x111>(v);
  v += dpp_or_zero_f64<0x112>(v);
  v += dpp_or_zero_f64<0x114>(v);
  v += dpp_or_zero_f64<0x118>(v);
  return v;
}
__device__ __forceinline__ double wave_incl_scan_f64(double v) {
  double t[1] = {v};
  wave_incl_scan_f64<1>(t);
  return t[0];
}
template <int N> __device__ __forceinline__ void wave_sums_f64(double (&v)[N]) {
  wave_incl_scan_f64<N>(v);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = last_lane_f64(v[i]);
}
// Reductions over a wave; every lane gets the result.
__device__ __forceinline__ double wave_sum_f64(double v) { return last_lane_f64(wave_incl_scan_f64(v)); }
__device__ __forceinline__ int wave_sum_i32(int v) { return last_lane_i32(wave_incl_scan_i32(v)); }
__device__ __forceinline__ float wave_max_f32(float v) {
  // on the bit patterns: the maximum of NaN-free floats through fmaxf, carried as ints by the moves
  const int r = wave_scan_i32(__float_as_int(v), __float_as_int(-INFINITY),
                              [](int a, int b) { return __float_as_int(fmaxf(__int_as_float(a), __int_as_float(b))); });
  return __int_as_float(last_lane_i32(r));
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  return uint32_t(last_lane_i32(wave_scan_i32(int(v), 0, [](int a, int b) { return int(uint32_t(a) > uint32_t(b) ? uint32_t(a) : uint32_t(b)); })));
}
__device__ __forceinline__ int wave_max_i32(int v) {
  return last_lane_i32(wave_scan_i32(v, int(0x80000000), [](int a, int b) { return a > b ? a : b; }));
}
__device__ __forceinline__ int wave_or_i32(int v) { return last_lane_i32(wave_scan_i32(v, 0, [](int a, int b) { return a | b; })); }

// Small per-block scratch for reductions and scans; one instance lives in static LDS.
// `NW` is the number of waves of the workgroup that calls the helpers.
struct BlockScratch {
  double d[24];
  float f[16];
  int i[16];
};

// Block-wide reductions.  Every thread of the block must call; the result is returned to all.
template <int NW> __device__ __forceinline__ double block_sum_f64(double v, BlockScratch& s) {
  v = wave_sum_f64(v);
  __syncthreads();
  if (lane_id() == 0) s.d[wave_id()] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w) t += s.d[w];
  return t;
}
template <int NW> __device__ __forceinline__ float block_max_f32(float v, BlockScratch& s) {
  v = wave_max_f32(v);
  __syncthreads();
  if (lane_id() == 0) s.f[wave_id()] = v;
  __syncthreads();
  float t = s.f[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) t = fmaxf(t, s.f[w]);
  return t;
}
template <int NW> __device__ __forceinline__ int block_sum_i32(int v, BlockScratch& s) {
  v = wave_sum_i32(v);
  __syncthreads();
  if (lane_id() == 0) s.i[wave_id()] = v;
  __syncthreads();
  int t = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) t += s.i[w];
  return t;
}

template <int NW> __device__ __forceinline__ int block_max_i32(int v, BlockScratch& s) {
  v = wave_max_i32(v);
  __syncthreads();
  if (lane_id() == 0) s.i[wave_id()] = v;
  __syncthreads();
  int t = s.i[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) t = s.i[w] > t ? s.i[w] : t;
  return t;
}

template <int NW> __device__ __forceinline__ int block_or_i32(int v, BlockScratch& s) {
  v = wave_or_i32(v);
  __syncthreads();
  if (lane_id() == 0) s.i[wave_id()] = v;
  __syncthreads();
  int t = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) t |= s.i[w];
  return t;
}

// Block-wide exclusive scan in thread order; `total` receives the sum over the block.
template <int NW> __device__ __forceinline__ int block_excl_scan_i32(int v, BlockScratch& s, int& total) {
  const int inc = wave_incl_scan_i32(v);
  __syncthreads();
  if (lane_id() == 63) s.i[wave_id()] = inc;
  __syncthreads();
  int base = 0, t = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    if (w < wave_id()) base += s.i[w];
    t += s.i[w];
  }
  total = t;
  return base + inc - v;
}

// Sort of n candidate records held in LDS, descending, by a counting sort over NT linear value bins (they
// divide the interval [min, max] of the values present evenly; any monotone binning keeps the result exact)
// followed by an exact rank inside each bin.  The largest min(n, k_keep) records end up in out[0..) in order.  Only
// the bins that can reach the first k_keep places are moved: `tmp` needs room for k_keep records plus the population
// of the bin that straddles that boundary; the function returns false, leaving `in` intact, when tmp_cap is too small
// for that (kRankAhead records more behind tmp_cap are written and read).  `in` and `out` may be the same array; `tmp`
// must be distinct from both.  `bins` holds NT words of LDS, NT = threads of the workgroup.
// Bound by latencies: six barriers, and in the rank the population of a bin (tens of records where bfloat16 leaves few
// values apart), which is therefore read kRankAhead records at a time.
constexpr int kRankAhead = 4;
template <int kBins> __device__ __forceinline__ int value_bin(uint64_t c, float vmin, float scale) {
  return value_bin_of(cand_value(c) - vmin, scale, kBins);
}
// kRange: the bins divide [lo, hi] instead, whatever lies outside in the first and the last of them, and `bins` has been set to zero:
// the step that looks for the extremes, a third of the whole, and its barrier fall away.  (False where that makes a bin too
// crowded; nothing has been moved then.)
template <int NT, bool kRange = false>
__device__ __forceinline__ bool bucket_sort_desc(const uint64_t* in, int n, uint64_t* tmp, int tmp_cap, uint64_t* out,
                                                 int k_keep, uint32_t* bins, BlockScratch& red, float lo = 0.0f, float hi = 0.0f) {
  constexpr int NW = NT / 64;
  static_assert(NW + 2 <= 16, "room in the scratch");
  if (n <= 0) return true;
  const int tid = threadIdx.x;
  float vmin = lo, span = hi - lo;                       // may overflow to +inf: then one bin
  if constexpr (!kRange) {
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
    const uint32_t* key = reinterpret_cast<const uint32_t*>(in) + 1;      // the high word of a record
#pragma unroll 4
    for (int i = tid; i < n; i += NT) {
      const uint32_t k = key[2 * i];
      kmin = k < kmin ? k : kmin;
      kmax = k > kmax ? k : kmax;
    }
    kmax = wave_max_u32(kmax);
    kmin = ~wave_max_u32(~kmin);
    bins[tid] = 0;
    if (lane_id() == 0) { red.i[wave_id()] = int(kmin); red.f[wave_id()] = as_f32(kmax); }
    __syncthreads();
    kmin = uint32_t(red.i[0]); kmax = as_u32(red.f[0]);
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      kmin = uint32_t(red.i[w]) < kmin ? uint32_t(red.i[w]) : kmin;
      kmax = as_u32(red.f[w]) > kmax ? as_u32(red.f[w]) : kmax;
    }
    vmin = key_to_f32(kmin);
    span = key_to_f32(kmax) - vmin;
  }
  const float scale = (span > 0.0f && span < 3.0e38f) ? float(NT - 1) / span : 0.0f;
  if constexpr (kRange) {
    if (scale == 0.0f) return false;
  }
  for (int i = tid; i < n; i += NT) atomicAdd(&bins[value_bin<NT>(in[i], vmin, scale)], 1u);
  __syncthreads();
  // where each bin begins, in descending order; the one that holds place k_keep (the last, if there are fewer records)
  const int b_mine = NT - 1 - tid, mine = int(bins[b_mine]);
  const int inc = wave_incl_scan_i32(mine);
  if (lane_id() == 63) red.i[wave_id()] = inc;
  __syncthreads();
  int run = inc - mine;
#pragma unroll
  for (int w = 0; w < NW; ++w) run += w < wave_id() ? red.i[w] : 0;
  const int place = n < k_keep ? n : k_keep;
  bins[b_mine] = uint32_t(run);
  if (run < place && run + mine >= place) { red.f[0] = __int_as_float(run + mine); red.f[1] = __int_as_float(b_mine); }
  __syncthreads();
  const int n_moved = __float_as_int(red.f[0]), last_bin = __float_as_int(red.f[1]);
  if (n_moved > tmp_cap) return false;
  for (int i = tid; i < n; i += NT) {
    const uint64_t c = in[i];
    const int b = value_bin<NT>(c, vmin, scale);
    if (b >= last_bin) tmp[atomicAdd(&bins[b], 1u)] = c;
  }
  if (tid < kRankAhead) tmp[n_moved + tid] = 0;          // smaller than every record
  __syncthreads();
  // (a bin's word is now where it ends.  Records behind a bin are smaller, so that a step past its end counts nothing.)
  for (int i = tid; i < n_moved; i += NT) {
    const uint64_t c = tmp[i];
    const int b = value_bin<NT>(c, vmin, scale);
    const int s0 = b == NT - 1 ? 0 : int(bins[b + 1]), s1 = int(bins[b]);
    int r = s0;
    for (int j = s1 - s0 > 1 ? s0 : s1; j < s1; j += kRankAhead) {      // (alone in its bin: nothing to look at)
      uint64_t t[kRankAhead];
#pragma unroll
      for (int u = 0; u < kRankAhead; ++u) t[u] = tmp[j + u];
#pragma unroll
      for (int u = 0; u < kRankAhead; ++u) r += t[u] > c ? 1 : 0;
    }
    if (r < k_keep) out[r] = c;
  }
  __syncthreads();
  return true;
}

// The same for a few records, a quarter of the workgroup's threads at most: four lanes count the larger ones for each.  out is
// another array; behind a barrier on both sides.
template <int NT>
__device__ __forceinline__ void rank_sort_desc(const uint64_t* in, int n, uint64_t* out, int k_keep) {
  const int c = threadIdx.x >> 2, q = threadIdx.x & 3;
  if (__builtin_amdgcn_readfirstlane(wave_id() * 16) < n) {      // whole waves
    const uint64_t mine = in[c < n ? c : n - 1];
    int r = 0;
    for (int j = q; j < n; j += 16) {
      uint64_t t[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) t[u] = in[j + 4 * u < n ? j + 4 * u : n - 1];
#pragma unroll
      for (int u = 0; u < 4; ++u) r += t[u] > mine && j + 4 * u < n ? 1 : 0;
    }
    r += dpp_i32<0xB1>(0, r);                                    // quad_perm 1 0 3 2, then 2 3 0 1
    r += dpp_i32<0x4E>(0, r);
    if (q == 0 && c < n && r < k_keep) out[r] = mine;
  }
  __syncthreads();
}

// How a row of V elements splits into a 16-byte aligned body of whole vectors plus at most
// 2*(kPerVec-1) edge elements in front of and behind it.
struct RowSplit {
  int head;        // elements before the aligned body
  int64_t nvec;    // whole 16-byte vectors in the body
  int tail;        // elements after the body
  const uint4* body;
};
template <typename T> __device__ __forceinline__ RowSplit split_row(const void* row, int64_t V) {
  constexpr int E = ElemTraits<T>::kPerVec;
  RowSplit r;
  uintptr_t a = reinterpret_cast<uintptr_t>(row);
  int mis = int((a & 15u) / ElemTraits<T>::kBytes);
  int head = mis ? (E - mis) : 0;
  if (head > V) head = int(V);
  r.head = head;
  r.nvec = (V - head) / E;
  r.tail = int(V - head - r.nvec * E);
  r.body = reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(row) + size_t(head) * ElemTraits<T>::kBytes);
  return r;
}
// Index (within the row) and value of edge element e in 0 .. head+tail-1.
template <typename T> __device__ __forceinline__ int64_t edge_index(const RowSplit& r, int e) {
  return e < r.head ? int64_t(e) : int64_t(r.head) + r.nvec * ElemTraits<T>::kPerVec + (e - r.head);
}

}  // namespace tslt
