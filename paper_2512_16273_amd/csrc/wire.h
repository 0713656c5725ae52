// tslt_pack / tslt_unpack: the wire format of a batch of truncated sets (Section 2.2 fixes its size, K pairs
// of a b_idx-bit token id and a b_prob-bit value per position; the layout is defined here).
//
// The stream of one row, least significant bit first: 16 bits count, then per kept entry, in canonical
// order, b_idx = ceil(log2 V) bits of token id followed by the 16 bits of the value (binary16 or bfloat16).
// Rows are padded with zero bits to whole 32-bit words and concatenated; row_offset[r] is the first word of
// row r, row_offset[rows] the total.  Bit p of a row's stream is bit p % 32 of its word p / 32.
#pragma once
#include <hip/hip_fp16.h>
#include "common.h"

namespace tslt {

constexpr int kPayloadF32 = 0, kPayloadBf16 = 1, kPayloadF16 = 2;    // numbered as tslt_dtype

// A scaled logit as it travels: rounded to nearest-even to the 16-bit format, clamped to its finite range,
// and returned as the fp32 value the receiver decodes.
__device__ __forceinline__ float round_payload(float x, int payload) {
  if (payload == kPayloadBf16) {
    const float big = 3.3895313892515355e38f;                 // largest finite bfloat16
    x = fminf(fmaxf(x, -big), big);
    uint32_t b = __float_as_uint(x);
    b = (b + 0x7FFFu + ((b >> 16) & 1u)) & 0xFFFF0000u;
    return __uint_as_float(b);
  }
  if (payload == kPayloadF16) {
    x = fminf(fmaxf(x, -65504.0f), 65504.0f);
    return __half2float(__float2half_rn(x));
  }
  return x;
}
__device__ __forceinline__ uint32_t payload_bits16(float x, int payload) {
  x = round_payload(x, payload);
  if (payload == kPayloadF16) return uint32_t(__half_as_ushort(__float2half_rn(x)));
  return __float_as_uint(x) >> 16;
}
__device__ __forceinline__ float payload_from_bits16(uint32_t b, int payload) {
  if (payload == kPayloadF16) return __half2float(__ushort_as_half(static_cast<unsigned short>(b)));
  return __uint_as_float(b << 16);
}

inline int wire_index_bits(int64_t V) {
  int b = 0;
  while ((int64_t(1) << b) < V) ++b;
  return b;
}
inline int64_t wire_row_words(int64_t count, int b_idx) { return (16 + count * (b_idx + 16) + 31) / 32; }

struct WireParams {
  const int32_t* idx;
  const float* logit;
  const int32_t* count;
  int64_t rows;
  int k_cap;
  int b_idx;
  int payload;
  uint32_t* words;
  int64_t* row_offset;
  int64_t rows_per;      // of one workgroup
  int clear;             // the words behind the stream, up to the bound, are set to 0
  // unpack
  const uint32_t* in_words;
  const int64_t* in_row_offset;
  int32_t* out_idx;
  float* out_logit;
  int32_t* out_count;
};

__device__ __forceinline__ int wire_clamped_count(int c, int k_cap) { return c < 0 ? 0 : (c > k_cap ? k_cap : c); }

// Packing in one launch: a workgroup of four waves takes rows_per consecutive rows, adds up the words of all rows before
// them (their counts come out of the L2: 4 bytes a row), scans its own and packs a row per wave at a time.  A lane makes
// a whole word out of the entries that lie in it (three at most, two from 31 bits an entry on), so that nothing is assembled in LDS and
// every store is a full line.  With `clear`, a row zeroes as many words as it falls short of a full row's, counted from
// the end of out_words: together all those behind the stream.  Bound by its launch at the sizes of a round (2048 rows of k_cap 256: 6.4 us
// the kernel, 4.7 unpacking, beside 11 of the host's), by trips to memory one after the other in wide rows: us of the kernel a word at a
// time / four, 16384 rows of k_cap 1024 76.3 / 52.4, 8192 of 1000 28.6 / 25.8, 2048 of 256 6.5 / 6.1.  A row that has no more than a word a lane
// takes them one at a time: 16384 of 16 16.8, by four 17.3.
constexpr int kPackThreads = 256, kPackWaves = kPackThreads / 64;
// Workgroups beyond which they take more than one row per wave: what fills the chip (each adds up all counts before its
// rows, so that more cost: 4 million rows of 2 entries 5.2 ms, 7.8 with 4096).  With 1024 and three entries to every word
// wide rows were slower than by the launch for offsets and a row assembled in LDS: 16384 rows of k_cap 1024, packed
// and unpacked, 106 us so, 135 by 1024, 104 now; 8192 rows 56, 60, 46; 16384 of 256 52, 46, 39.
constexpr int kPackGroups = 2048;
inline int64_t wire_rows_per_group(int64_t rows) {
  const int64_t r = (rows + kPackGroups - 1) / kPackGroups;
  return r > kPackWaves ? r : kPackWaves;
}
__device__ __forceinline__ int wire_words_of(int count, const WireParams& p) {
  return (16 + wire_clamped_count(count, p.k_cap) * (p.b_idx + 16) + 31) >> 5;
}
template <int kAt>
__global__ __launch_bounds__(kPackThreads) void wire_pack_kernel(const WireParams p) {
  __shared__ long long before_s[kPackWaves];
  __shared__ int wave_tot[kPackWaves], count_s[kPackThreads], off_s[kPackThreads];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t r0 = int64_t(blockIdx.x) * p.rows_per;
  const int64_t r1 = r0 + p.rows_per < p.rows ? r0 + p.rows_per : p.rows;
  if (p.rows == 0 && tid == 0) p.row_offset[0] = 0;
  const int E = p.b_idx + 16;
  const int row_max = (16 + p.k_cap * E + 31) >> 5;
  long long base = 0;
  // (eight counts at a time, as many in flight; a row beyond the group's first reads row 0's and counts as nothing)
  for (int64_t r = tid; r < r0; r += 8 * kPackThreads) {
    int c[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) c[u] = p.count[r + u * kPackThreads < r0 ? r + u * kPackThreads : 0];
#pragma unroll
    for (int u = 0; u < 8; ++u) base += r + u * kPackThreads < r0 ? wire_words_of(c[u], p) : 0;
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) base += __shfl_xor(base, d, 64);
  if (lane == 0) before_s[wave] = base;
  __syncthreads();
  base = 0;
#pragma unroll
  for (int w = 0; w < kPackWaves; ++w) base += before_s[w];
  const uint32_t inv_E = uint32_t(0xFFFFFFFFu / uint32_t(E)) + 1u;      // x / E = umulhi(x, inv_E) for x < 2^16
  for (int64_t c0 = r0; c0 < r1; c0 += kPackThreads) {
    const int64_t mine = c0 + tid;
    const int my_count = mine < r1 ? wire_clamped_count(p.count[mine], p.k_cap) : 0;
    const int my_words = mine < r1 ? wire_words_of(my_count, p) : 0;
    const int inc = wave_incl_scan_i32(my_words);
    __syncthreads();                                                    // the last chunk's rows are packed
    if (lane == 63) wave_tot[wave] = inc;
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kPackWaves; ++w) {
      before += w < wave ? wave_tot[w] : 0;
      total += wave_tot[w];
    }
    count_s[tid] = my_count;
    off_s[tid] = before + inc - my_words;
    if (mine < r1) {
      p.row_offset[mine] = base + before + inc - my_words;
      if (mine == p.rows - 1) p.row_offset[p.rows] = base + before + inc;
    }
    __syncthreads();
    const int n = int(r1 - c0 < kPackThreads ? r1 - c0 : kPackThreads);
    for (int k = wave; k < n; k += kPackWaves) {
      const int64_t r = c0 + k;
      const int c = count_s[k];
      const int n_words = (16 + c * E + 31) >> 5;
      const long long off = base + off_s[k];
      const int32_t* ix = p.idx + size_t(r) * p.k_cap;
      const float* lg = p.logit + size_t(r) * p.k_cap;
      uint32_t* out = p.words + off;
      // (kAt words a lane at a time: what they are made of is requested for all of them first)
      for (int w0 = 0; w0 < n_words; w0 += kAt * 64) {
        int id[kAt][3];
        float value[kAt][3];
        auto first_of = [&](int w) {                                    // the first entry that reaches into word w
          const int b0 = w * 32 - 16;                                   // of the entries' own bit stream
          return b0 > 0 ? int(__umulhi(uint32_t(b0), inv_E)) : 0;
        };
#pragma unroll
        for (int u = 0; u < kAt; ++u) {
          if (w0 + 64 * u >= n_words) break;
          const int first = first_of(w0 + 64 * u + lane);
#pragma unroll
          for (int t = 0; t < 3; ++t) {
            if (t == 2 && E >= 31) break;                               // two cover 32 bits wherever they begin
            const int at = first + t < c ? first + t : 0;
            id[u][t] = ix[at];
            value[u][t] = lg[at];
          }
        }
#pragma unroll
        for (int u = 0; u < kAt; ++u) {
          if (w0 + 64 * u >= n_words) break;
          const int w = w0 + 64 * u + lane, b0 = w * 32 - 16, first = first_of(w);
          uint32_t word = w == 0 ? uint32_t(c) : 0u;
#pragma unroll
          for (int t = 0; t < 3; ++t) {
            if (t == 2 && E >= 31) break;
            const int i = first + t;
            const uint64_t entry = (uint64_t(uint32_t(id[u][t])) & ((uint64_t(1) << p.b_idx) - 1)) |
                                   (uint64_t(payload_bits16(value[u][t], p.payload)) << p.b_idx);
            const int sh = i * E - b0;                                  // where the entry begins in the word
            const uint32_t piece = sh >= 0 ? uint32_t(entry << (sh & 31)) : uint32_t(entry >> (-sh & 63));
            word |= i < c && sh < 32 ? piece : 0u;
          }
          if (w < n_words) out[w] = word;
        }
      }
      if (p.clear) {
        uint32_t* tail = p.words + (p.rows * row_max - ((r + 1) * row_max - (off + n_words)));
        for (int w = lane; w < row_max - n_words; w += 64) tail[w] = 0u;
      }
    }
    base += total;
  }
}

// One wave per row, an entry a lane at a time.  (Four entries a lane, their words requested before the count is known, take a trip to
// memory less and more instructions: 14 rows of k_cap 256 4.1 us the kernel so, 3.8 by four, beside 11 of the host's; 16384 of 16 5.7 / 6.0, of 64
// 6.4 / 7.0, of 1024 29.2 / 30.2, 4000 of 40 3.7 / 4.0, 2048 of 256 4.7 / 4.6.)
__global__ __launch_bounds__(64) void wire_unpack_kernel(const WireParams p) {
  const int64_t r = blockIdx.x;
  const int lane = threadIdx.x;
  const uint32_t* in = p.in_words + p.in_row_offset[r];
  const int64_t n_words = p.in_row_offset[r + 1] - p.in_row_offset[r];
  const int E = p.b_idx + 16;
  int c = n_words > 0 ? int(in[0] & 0xFFFFu) : 0;
  // a count that its row's words cannot hold is cut to what they do hold
  const long long fits = n_words > 0 ? (n_words * 32 - 16) / E : 0;
  if (c > fits) c = int(fits);
  c = wire_clamped_count(c, p.k_cap);
  int32_t* ix = p.out_idx + size_t(r) * p.k_cap;
  float* lg = p.out_logit + size_t(r) * p.k_cap;
  for (int i = lane; i < p.k_cap; i += 64) {
    int id = -1;
    float v = -INFINITY;
    if (i < c) {
      const long long bit = 16 + (long long)i * E;
      const int64_t w = bit >> 5;
      const int sh = int(bit & 31);
      uint64_t lo = uint64_t(in[w]) | (w + 1 < n_words ? uint64_t(in[w + 1]) << 32 : 0);
      uint64_t entry = lo >> sh;
      if (sh + E > 64 && w + 2 < n_words) entry |= uint64_t(in[w + 2]) << (64 - sh);
      entry &= (uint64_t(1) << E) - 1;
      id = int(entry & ((uint64_t(1) << p.b_idx) - 1));
      v = payload_from_bits16(uint32_t(entry >> p.b_idx) & 0xFFFFu, p.payload);
    }
    ix[i] = id;
    lg[i] = v;
  }
  if (lane == 0) p.out_count[r] = c;
}

}  // namespace tslt
