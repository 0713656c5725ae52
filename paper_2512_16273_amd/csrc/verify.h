// tslt_verify: token-sequence verification (Algorithm 3) against sparse draft distributions.
//
// Batches up to round_rows(): verify_round_kernel, one workgroup of 1024 threads per (sequence, row), makes the
// acceptance test and the draw from one fp64 pass over the row, and the last workgroup of a sequence keeps the draw that
// counts.  Larger ones, which fill the chip, in two halves:
// Kernel A, one workgroup of 256 threads per (sequence, draft position): eval_row_on_set over the target row in
// fp32 terms, at the memory's pace, then the ratio p(x)/q_hat(x) of the draft token, the acceptance decision
// u < min(1, ratio) and Lemma 1's sum min(p, q_hat).
// Kernel B, one workgroup of 1024 threads per sequence: finds the first rejected position j (or the bonus row) from
// kernel A's decisions, sweeps that one target row in fp64, draws from norm(max(0, p - q_hat)) (or from p for
// the bonus row) by inverse CDF and writes the sequence's outputs.
// Where a few long rows leave compute units idle, several workgroups of the same kernels sweep each (rowsample.h).
#pragma once
#include "rowops.h"
#include "rowsample.h"

namespace tslt {

struct VerifyParams {
  const void* target;
  int64_t B, V, row_stride;
  int gamma;
  float rT, k2;
  const int32_t* q_idx;
  const float* q_logit;
  const int32_t* q_count;
  int k_cap;
  const int32_t* draft_tokens;
  const float* u_accept;
  const float* u_resample;
  int32_t* out_accept_len;
  int32_t* out_tokens;
  float* out_ratio;
  float* out_beta;
  int32_t* status;
  // workspace
  int32_t* flags;        // [B, gamma] 1 accepted, 0 rejected, 2 row unusable, 3 not examined (staged mode)
  int32_t* row_status;   // [B, gamma]
  int stage0;            // staged mode: positions in the first stage (0 = all positions in one launch)
  int j_begin, j_count;  // the positions one launch covers (verify_round_kernel with draws: the bonus row too)
  int draws;             // verify_round_kernel draws as well
  double* items;         // masses of shared rows' items
  int64_t items_stride;
  int64_t items_rows;    // there is room for (read on the host)
  int parts;             // workgroups that share a row
  uint64_t* part_words;  // [rows, parts]: theirs (handover.h)
  uint64_t* words;       // [B, gamma + 1, 2]: what a round's workgroups leave (null: the workspace has no room; its rows are not shared)
  Tag tag;
};
constexpr int kFlagSkipped = 3;

// Rows that may be shared by workgroups (row_parts): those of a small round, or one for each sequence.
inline int64_t verify_rows_to_share(int64_t B, int64_t gamma, int64_t V) {
  if (B <= 0 || gamma <= 0 || V < kShareLeastV) return 0;
  return B * (gamma + 1) <= kShareRows ? B * (gamma + 1) : (B <= kShareRows ? B : 0);
}
// Rows of a round whose workgroups leave their results in memory for the last of each sequence (more than a round has: round_rows).  (Rows
// shorter than kHandLeastV would gain as much, 16 x 8 binary16 rows of 1000 11.0 us by a launch more, 9.5 so; their callers are told the
// size that they have always been told, and no call is refused what it was given before.)
constexpr int64_t kHandRows = 1024, kHandLeastV = 2048;
inline int64_t verify_rows_handed(int64_t B, int64_t gamma, int64_t V) {
  return V >= kHandLeastV && B * (gamma + 1) <= kHandRows ? B * (gamma + 1) : 0;
}
// What a call has to be given: a decision and a status word for every position.  With room behind them for what workgroups
// hand over, the size that callers are told, rows are shared and a round takes one launch.
inline size_t verify_least_workspace_bytes(int64_t B, int64_t gamma) { return align256(size_t(B) * gamma * 4) * 2; }
inline size_t verify_words_bytes(int64_t B, int64_t gamma, int64_t V) { return align256(size_t(verify_rows_handed(B, gamma, V)) * 16); }
inline size_t verify_part_words_bytes(int64_t B, int64_t gamma, int64_t V) {
  return verify_rows_to_share(B, gamma, V) > 0 ? align256(size_t(kShareWords) * 8) : 0;
}
inline size_t verify_workspace_bytes(int64_t B, int64_t gamma, int64_t V, int k_cap) {
  (void)k_cap;
  return verify_least_workspace_bytes(B, gamma) + verify_words_bytes(B, gamma, V) + verify_part_words_bytes(B, gamma, V) +
         align256(size_t(verify_rows_to_share(B, gamma, V) * items_stride(V)) * sizeof(double));
}
// (Of less than that, an earlier version's size say, what fits: that version's has room for the masses alone, of which a 16-bit row has half
// as many as it is asked for.  per_vec: the type's elements in a vector.)
inline void verify_carve_workspace(VerifyParams& p, void* ws, size_t ws_bytes, int per_vec) {
  char* w = reinterpret_cast<char*>(ws);
  p.flags = reinterpret_cast<int32_t*>(w); w += align256(size_t(p.B) * p.gamma * 4);
  p.row_status = reinterpret_cast<int32_t*>(w); w += align256(size_t(p.B) * p.gamma * 4);
  p.items_stride = items_stride(p.V, per_vec);
  p.words = p.part_words = nullptr;
  p.items = nullptr;
  p.items_rows = 0;
  int64_t left = int64_t(ws_bytes) - int64_t(w - reinterpret_cast<char*>(ws));
  const int64_t handed = int64_t(verify_words_bytes(p.B, p.gamma, p.V)), parts = int64_t(verify_part_words_bytes(p.B, p.gamma, p.V));
  if (handed > 0 && left >= handed) {
    p.words = reinterpret_cast<uint64_t*>(w);
    w += handed;
    left -= handed;
  }
  if (parts > 0 && left > parts) {
    p.part_words = reinterpret_cast<uint64_t*>(w);
    p.items = reinterpret_cast<double*>(w + parts);
    p.items_rows = (left - parts) / (p.items_stride * int64_t(sizeof(double)));
  }
}

template <typename T> __device__ __forceinline__ const void* target_row(const VerifyParams& p, int64_t b, int j) {
  return reinterpret_cast<const char*>(p.target) +
         (size_t(b) * (p.gamma + 1) + j) * size_t(p.row_stride) * ElemTraits<T>::kBytes;
}

// A later stage: nothing to do for a sequence that an earlier stage has rejected (all threads of a workgroup).
__device__ __forceinline__ bool skip_position(const VerifyParams& p, int64_t b, int64_t r) {
  int dead = 0;
  for (int i = threadIdx.x; i < p.j_begin; i += blockDim.x) dead |= p.flags[b * p.gamma + i] != 1 ? 1 : 0;
  if (!__syncthreads_or(dead)) return false;
  if (threadIdx.x == 0) {
    p.flags[r] = kFlagSkipped;
    p.row_status[r] = 0;
    if (p.out_ratio) p.out_ratio[r] = NAN;
    if (p.out_beta) p.out_beta[r] = NAN;
  }
  return true;
}

// ---------------------------------------------------------------------------------------------
// Kernel A
// ---------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kBlock, kAccWavesPerSimd) void verify_accept_kernel(const VerifyParams p) {
  __shared__ VerifyShared sh;
  const int tid = threadIdx.x;
  const int64_t b = blockIdx.x / p.j_count;
  const int j = p.j_begin + int(blockIdx.x - b * p.j_count);
  const int64_t r = b * p.gamma + j;       // row index in [0, B*gamma)
  if (p.j_begin > 0 && skip_position(p, b, r)) return;
  const void* row = target_row<T>(p, b, j);
  const RowSplit rs = split_row<T>(row, p.V);
  int count = p.q_count[r];
  count = count < 0 ? 0 : (count > p.k_cap ? p.k_cap : count);
  double p_s[kSetPer], q_s[kSetPer], p_out;
  int yi[kSetPer], st;
  bool ok;
  eval_row_on_set<T>(row, rs, p.V, p.rT, p.k2, p.q_idx + size_t(r) * p.k_cap, p.q_logit + size_t(r) * p.k_cap, count, sh,
                     p_s, q_s, yi, p_out, ok, st);
  const int x = p.draft_tokens[r];
  double beta = 0.0;
  if (tid == 0) { sh.bcast_d[0] = -1.0; sh.bcast_i[0] = 0; }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSetPer; ++k) {
    if (tid + k * kBlock < count && ok) {
      beta += p_s[k] < q_s[k] ? p_s[k] : q_s[k];
      if (yi[k] == x && q_s[k] > 0.0) {
        // the first matching entry decides (sets have distinct indices)
        if (atomicCAS(&sh.bcast_i[0], 0, 1) == 0) sh.bcast_d[0] = p_s[k] / q_s[k];
      }
    }
  }
  beta = block_sum_f64<kWaves>(beta, sh.red);
  if (tid == 0) {
    const double ratio = sh.bcast_d[0];
    int flag;
    if (!ok) flag = 2;
    else {
      if (sh.bcast_i[0] == 0) { st |= 4; flag = 0; }
      else {
        const double bound = ratio < 1.0 ? ratio : 1.0;
        flag = double(p.u_accept[r]) < bound ? 1 : 0;
      }
    }
    p.flags[r] = flag;
    p.row_status[r] = st;
    if (p.out_ratio) p.out_ratio[r] = ok ? float(ratio) : NAN;
    if (p.out_beta) p.out_beta[r] = ok ? float(beta) : NAN;
  }
}

// ---------------------------------------------------------------------------------------------
// Kernel B: one workgroup of 1024 threads per sequence, or p.parts of them (kParts), sweeps the row to be sampled and writes
// the sequence's outputs.
// ---------------------------------------------------------------------------------------------
template <typename T, typename Terms, int kWavesPerSimd, bool kParts = false, int kLoads = kStreamed>
__global__ __launch_bounds__(kRowThreads, kWavesPerSimd) void verify_resample_kernel(const VerifyParams p) {
  __shared__ RowShared sh;
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  double* table = reinterpret_cast<double*>(dyn_lds);
  const int tid = threadIdx.x, lane = lane_id();
  const uint32_t at = kParts ? blockIdx.x / uint32_t(p.parts) : blockIdx.x;      // (a division by 64 bits takes half a microsecond)
  const int64_t b = at;
  const int part = kParts ? int(blockIdx.x - at * p.parts) : 0;
  // The decisions of the sequence's first 64 positions are requested first, and with them the table where it is copied (asked for with
  // the row, behind them: 48 x 5 fp32 rows of 151936 43.6 us, 43.1 so; 128 x 4 binary16 rows of 32000 24.7 and 23.8; 400 x 4 of 60000 66.4 and 64.9;
  // not in fp32's form of 64 registers, which then spills), else half of it is built while they
  // travel.  Every wave then finds the first rejected position by itself (gamma when every draft token was
  // accepted): the words are few and nothing has to be handed round.
  const int32_t* fl_b = p.flags + b * p.gamma;
  const int f0 = lane < p.gamma ? fl_b[lane] : 1;
  const auto asked = [] {
    if constexpr (kWavesPerSimd == kShared && ElemTraits<T>::kBytes == 4) return AskWithRow{};
    else return Terms::begin();
  }();
  if constexpr (!kParts) Terms::first_half(table, p.rT);
  int j0 = f0 != 1 ? lane : p.gamma;
  if (p.gamma > 64 && ballot(f0 != 1) == 0) {
    for (int j = lane + 64; j < p.gamma; j += 64)
      if (fl_b[j] != 1) { j0 = j; break; }
  }
  const int jstar = -wave_max_i32(-j0);        // the smallest over the wave
  const bool residual = jstar < p.gamma;
  // the decision at that position, from the lane that holds it (a position beyond the first 64 is read again)
  const bool unusable = residual && (jstar < 64 ? __shfl(f0, jstar, 64) : fl_b[jstar]) == 2;
  const int64_t r = b * p.gamma + (residual ? jstar : 0);
  const float u_res = p.u_resample[b * (p.gamma + 1) + jstar];
  // (what the end needs is requested behind the sweep, whose registers are short, and travels during the search)
  const int j_lane = lane < p.gamma ? lane : p.gamma - 1;
  int st_first, x_first;
  auto request_end = [&]() { st_first = p.row_status[b * p.gamma + j_lane]; x_first = p.draft_tokens[b * p.gamma + j_lane]; };
  RowWork<T> w;
  int token = -1;
  if (tid == 0) sh.cmd = 0;                    // read behind a barrier: 1 when there is something to draw from
  if (!unusable) {
    row_open<T>(w, target_row<T>(p, b, jstar), p.V, p.rT, sh);
    row_take_set(w, p.q_idx + size_t(r) * p.k_cap, p.q_logit + size_t(r) * p.k_cap, residual ? p.q_count[r] : 0, p.k_cap);
    if constexpr (kParts) {
      if (!row_shared<T, Terms, kLoads>(w, table, asked, part, p.parts, p.items + b * p.items_stride, p.part_words + b * p.parts, p.tag, sh)) return;
    } else {
      row_sweep<T, Terms, kWavesPerSimd == kAlone, kLoads>(w, table, 1, asked, sh);
    }
    request_end();
    row_clear<T>(table);
    const int waves = row_set_waves(w), wave = __builtin_amdgcn_readfirstlane(wave_id());
    RowState rst;
    double left = 0.0;                             // max(0, p - q) at this thread's entry
    if (wave < waves) {
      row_eval(w, rst, sh);
      if (residual && rst.ok) left = row_test(w, rst, -1, 0, sh);
    }
    __syncthreads();
    if (wave < waves && residual && rst.ok) row_set_mass(w, left * rst.zp, sh);
    __syncthreads();
    if (wave == 0) {
      if (rst.ok) row_locate(w, rst, u_res, residual, residual ? row_tested(waves, 0, sh).part * rst.zp - rst.sum_e : 0.0, sh);
      if (lane == 0) { sh.cmd = rst.ok ? 1 : 0; sh.st = rst.st; }      // (another wave may still look at sh.flags)
    }
    __syncthreads();
    if (sh.cmd) token = row_pick(w, table, sh);
  } else {
    if (part != 0) return;
    request_end();
    if (tid == 0) sh.st = 0;
    __syncthreads();
  }
  if (wave_id() != 0) return;
  // status bits of the positions up to the one that decided
  int st = residual ? 0 : sh.st;
  for (int j = lane; j <= jstar && j < p.gamma; j += 64) st |= j == lane ? st_first : p.row_status[b * p.gamma + j];
  st = wave_or_i32(st);
  int32_t* ot = p.out_tokens + size_t(b) * (p.gamma + 1);
  for (int j = lane; j <= p.gamma; j += 64) {
    int v = -1;
    if (j < jstar) v = j == lane ? x_first : p.draft_tokens[b * p.gamma + j];
    else if (j == jstar) v = token;
    ot[j] = v;
  }
  if (lane == 0) {
    p.out_accept_len[b] = jstar;
    if (p.status) p.status[b] = st;
  }
}

// ---------------------------------------------------------------------------------------------
// A round in one pass over the rows, for batches that do not fill the chip (bound there by one row's own latency: the
// sweep by sixteen waves, then the chain of steps after it): one workgroup of 1024 threads per (sequence, row), or p.parts of them
// (kParts), sweeps its row once, takes the acceptance test from the sums and, if the token is rejected (or
// the row is the bonus row), draws the replacement at once, whether or not an earlier position will turn out to
// have been rejected (one sequence x 4, binary16 V = 32000: 26 us by kernels A and B, 14.1 by a round's kernel and a second launch, 12.2 so;
// 8 x 8 bfloat16, V = 128256: 30.6, 17.9 by three launches, 15.8).  What a position came to it leaves in memory (handover.h); the workgroup that finds those of all its
// sequence keeps the draw of the first rejected position and writes the sequence's outputs.  With a workspace that has no room
// for that a second launch does, one wave per sequence; until then a position's draw waits in its place in out_tokens, and
// the bonus row's status in out_accept_len.
// Without draws it is kernel A for such batches: the decisions of a batch are made in the same way whether it is
// verified by one call, by two halves or in stages.
// ---------------------------------------------------------------------------------------------
// One wave: the outputs of a sequence, from position j's decision, status bits and draw on: at(j) gives them for the positions of a
// lane, four words of gamma + 1 of them.  x_first: the lane's draft token.
template <typename F>
__device__ __forceinline__ void write_sequence(const VerifyParams& p, int64_t b, int x_first, F at) {
  const int lane = lane_id();
  int jstar = p.gamma, st = 0, token = -1;
  for (int j0 = 0; j0 <= p.gamma; j0 += 64) {
    const int j = j0 + lane;
    int flag = 1, s = 0, t = -1;
    if (j <= p.gamma) at(j, flag, s, t);
    const uint64_t stop = ballot(j == p.gamma || (j < p.gamma && flag != 1));
    st |= stop == 0 || lane <= __ffsll((long long)stop) - 1 ? s : 0;
    if (stop != 0) {
      const int src = __ffsll((long long)stop) - 1;
      jstar = j0 + src;
      token = __builtin_amdgcn_readlane(t, src);
      break;
    }
  }
  st = wave_or_i32(st);
  int32_t* ot = p.out_tokens + size_t(b) * (p.gamma + 1);
  for (int j = lane; j <= p.gamma; j += 64) {
    int v = -1;
    if (j < jstar) v = j == lane ? x_first : p.draft_tokens[b * p.gamma + j];
    else if (j == jstar) v = token;
    ot[j] = v;
  }
  if (lane == 0) {
    p.out_accept_len[b] = jstar;
    if (p.status) p.status[b] = st;
  }
}
template <typename T, typename Terms, int kWavesPerSimd, bool kParts = false>
__global__ __launch_bounds__(kRowThreads, kWavesPerSimd) void verify_round_kernel(const VerifyParams p) {
  __shared__ RowShared sh;
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  double* table = reinterpret_cast<double*>(dyn_lds);
  const uint32_t at = kParts ? blockIdx.x / uint32_t(p.parts) : blockIdx.x;      // (a division by 64 bits takes half a microsecond)
  const int64_t b = at / uint32_t(p.j_count);
  const int j = p.j_begin + int(at - uint32_t(b) * p.j_count);
  const bool bonus = j == p.gamma;
  const int64_t r = b * p.gamma + (bonus ? 0 : j);
  if (p.j_begin > 0 && skip_position(p, b, r)) return;
  RowWork<T> w;
  row_open<T>(w, target_row<T>(p, b, j), p.V, p.rT, sh);
  const int count = p.q_count[r], x = p.draft_tokens[r];
  const float u_acc = p.u_accept[r], u_res = p.u_resample[b * (p.gamma + 1) + j];
  row_take_set(w, p.q_idx + size_t(r) * p.k_cap, p.q_logit + size_t(r) * p.k_cap, bonus ? 0 : count, p.k_cap);
  if constexpr (kParts) {
    const int part = int(blockIdx.x - at * p.parts);
    if (!row_shared<T, Terms>(w, table, AskWithRow{}, part, p.parts, p.items + at * p.items_stride, p.part_words + at * p.parts, p.tag, sh)) return;
  } else {
    row_sweep<T, Terms, kWavesPerSimd == kAlone>(w, table, -1, AskWithRow{}, sh);
  }
  // (nothing is stored to memory before the last barrier, which would wait for it)
  row_clear<T>(table);
  const int waves = row_set_waves(w), wave = __builtin_amdgcn_readfirstlane(wave_id());
  int st = 0, flag = 0;
  float ratio = NAN, beta = NAN;
  RowState rst;
  double left = 0.0;                               // max(0, p - q) at this thread's entry
  if (wave < waves) {
    row_eval(w, rst, sh);
    if (!bonus && rst.ok) left = row_test(w, rst, x, 0, sh);
  }
  __syncthreads();
  double corr = 0.0;
  if (wave < waves) {
    flag = rst.ok ? 0 : 2;
    if (!bonus && rst.ok) {
      const RowTest t = row_tested(waves, 0, sh);
      ratio = float(t.ratio);
      beta = float(t.shared);
      if (!t.found) rst.st |= 4;
      const double bound = t.ratio < 1.0 ? t.ratio : 1.0;
      flag = t.found && double(u_acc) < bound ? 1 : 0;
      corr = t.part * rst.zp - rst.sum_e;
      if (flag == 0 && p.draws) row_set_mass(w, left * rst.zp, sh);
    }
  }
  __syncthreads();
  if (wave == 0) {
    if (flag == 0 && p.draws) row_locate(w, rst, u_res, !bonus, corr, sh);
    st = rst.st;
    if (lane_id() == 0) sh.cmd = flag;
  }
  __syncthreads();
  const int token = sh.cmd == 0 && p.draws ? row_pick(w, table, sh) : -1;
  if (threadIdx.x == 0 && !bonus) {
    if (p.out_ratio) p.out_ratio[r] = ratio;
    if (p.out_beta) p.out_beta[r] = beta;
  }
  if (p.words == nullptr || !p.draws) {
    if (threadIdx.x != 0) return;
    if (!bonus) {
      p.flags[r] = flag;
      p.row_status[r] = st;
    } else {
      p.out_accept_len[b] = st;
    }
    if (p.draws) p.out_tokens[size_t(b) * (p.gamma + 1) + j] = token;
    return;
  }
  if (wave_id() != 0) return;
  const int lane = lane_id();
  const int x_first = p.draft_tokens[b * p.gamma + (lane < p.gamma ? lane : p.gamma - 1)];      // (travels meanwhile)
  // (nothing in LDS is needed any more)
  int* tokens = sh.set_y;
  int* state = reinterpret_cast<int*>(sh.set_e);
  if (!hand_over(p.words + 2 * size_t(b) * (p.gamma + 1), j, p.gamma + 1, uint32_t(token), uint32_t(flag | st << 8), p.tag, tokens, state)) return;
  write_sequence(p, b, x_first, [&](int i, int& f, int& s, int& t) {
    t = tokens[i];
    f = state[i] & 255;
    s = state[i] >> 8;
  });
}
__global__ __launch_bounds__(64) void verify_select_kernel(const VerifyParams p) {
  const int64_t b = blockIdx.x;
  const int lane = threadIdx.x;
  const int x_first = p.draft_tokens[b * p.gamma + (lane < p.gamma ? lane : p.gamma - 1)];
  write_sequence(p, b, x_first, [&](int j, int& flag, int& s, int& t) {
    t = p.out_tokens[size_t(b) * (p.gamma + 1) + j];
    if (j < p.gamma) { flag = p.flags[b * p.gamma + j]; s = p.row_status[b * p.gamma + j]; }
    else s = p.out_accept_len[b];
  });
}

// Largest batch, in rows B * (gamma + 1), that is verified by verify_round_kernel: one row per compute unit, and two
// through bfloat16's bit table, whose sweep is bound by the LDS and leaves the vector units to the other row's steps.
// Measured, us a round, this way / by kernels A and B (V = 128256, k_cap 256): bfloat16 384 rows 33.3 / 38.2, 512 36.2 /
// 40.2, 896 65.6 / 59.3; binary16 384 55.5 / 45.4; fp32 384 55.7 / 58.3, 512 63.8 / 62.8 (fp32 keeps binary16's line: 4 %
// in a narrow range).
template <typename Terms> inline int64_t round_rows() { return int64_t(compute_units()) * (Terms::kBits && !kLargeTable<Terms> ? 2 : 1); }

// phases: bit 0 = acceptance decisions (kernel A), bit 1 = resampling and outputs (kernel B)
template <typename T, typename Terms> hipError_t launch_verify_with(VerifyParams p, hipStream_t s, int phases) {
  hipError_t e = hipSuccess;
  const int64_t cus = compute_units();
  auto by_rows = [&](auto alone, auto shared, int64_t rows) -> hipError_t {      // one workgroup per row
    // (binary16's table leaves a compute unit to one workgroup in any case)
    if constexpr (kLargeTable<Terms>) {
      if ((e = allow_dynamic_lds<decltype(alone)::value>(int(Terms::kBytes))) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kLargeTable<Terms> || rows <= cus ? alone.value : shared.value, dim3(unsigned(rows)), dim3(kRowThreads),
                       Terms::kBytes, s, p);
    return hipGetLastError();
  };
  auto round = [&]() {
    return by_rows(KernelTag<&verify_round_kernel<T, Terms, kAlone>>{}, KernelTag<&verify_round_kernel<T, Terms, kShared>>{},
                   p.B * p.j_count);
  };
  auto share = [&](auto fn, int64_t rows) -> hipError_t {                        // p.parts workgroups per row
    if constexpr (kLargeTable<Terms>) {
      if ((e = allow_dynamic_lds<decltype(fn)::value>(int(Terms::kBytes))) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(fn.value, dim3(unsigned(rows * p.parts)), dim3(kRowThreads), Terms::kBytes, s, p);
    return hipGetLastError();
  };
  const bool by_row = p.B * (p.gamma + 1) <= round_rows<Terms>();
  if (by_row && phases == 3 && p.stage0 == 0) {
    p.j_begin = 0;
    p.j_count = p.gamma + 1;
    p.draws = 1;
    p.parts = p.words != nullptr && p.B * p.j_count <= p.items_rows ? row_parts<T, Terms>(p.V, p.B * p.j_count) : 1;
    // (a sequence of more positions than a wave has lanes: more words than one trip to memory brings.  1 x 200 bfloat16 rows of 8000 11.3 us by a
    // launch more, 12.4 so; 2 x 100 11.3 / 12.3, 1 x 127 11.2 / 10.6, 2 x 63 11.2 / 10.1)
    if (p.gamma >= 64 && p.parts == 1) p.words = nullptr;
    if (p.words != nullptr) p.tag = next_tag();
    e = p.parts > 1 ? share(KernelTag<&verify_round_kernel<T, Terms, kAlone, true>>{}, p.B * p.j_count) : round();
    if (e != hipSuccess || p.words != nullptr) return e;
    hipLaunchKernelGGL(verify_select_kernel, dim3(unsigned(p.B)), dim3(64), 0, s, p);
    return hipGetLastError();
  }
  if (phases & 1) {
    // stages of stage0, stage0, 2 * stage0, 4 * stage0, ... positions; one stage if stage0 is 0
    int len = p.stage0 > 0 ? p.stage0 : p.gamma;
    p.draws = 0;
    for (int j0 = 0, k = 0; j0 < p.gamma; ++k) {
      p.j_begin = j0;
      p.j_count = p.gamma - j0 < len ? p.gamma - j0 : len;
      if (by_row) {
        e = round();
      } else {
        hipLaunchKernelGGL(verify_accept_kernel<T>, dim3(unsigned(p.B * p.j_count)), dim3(kBlock), 0, s, p);
        e = hipGetLastError();
      }
      if (e != hipSuccess) return e;
      j0 += p.j_count;
      if (k > 0) len *= 2;
    }
  }
  if (phases & 2) {
    p.parts = p.B <= p.items_rows ? row_parts<T, Terms>(p.V, p.B) : 1;
    auto resample = [&](auto loads) -> hipError_t {
      constexpr int kLoads = decltype(loads)::value;
      if (p.parts > 1) {
        p.tag = next_tag();
        return share(KernelTag<&verify_resample_kernel<T, Terms, kAlone, true, kLoads>>{}, p.B);
      }
      return by_rows(KernelTag<&verify_resample_kernel<T, Terms, kAlone, false, kLoads>>{},
                     KernelTag<&verify_resample_kernel<T, Terms, kShared, false, kLoads>>{}, p.B);
    };
    if constexpr (ElemTraits<T>::kBytes == 4) {
      if (p.B * (p.gamma + 1) * p.V * 4 > kStreamBytes && p.B * p.V * 4 <= kCachedBytes) return resample(std::integral_constant<int, kCached>{});
    }
    return resample(std::integral_constant<int, kStreamed>{});
  }
  return e;
}
// Binary16 batches beyond round_rows() of rows this long: the bit table (128 x 5 by PowTerms / by it, V = 152064 63.4 / 60.2
// us, 256000 95.5 / 86.2; 100000 47.9 either way), at the price of rows centred on 0, outside its range (63.3 / 91.9, 95.6 / 139.2).
constexpr int64_t kBitMinV16 = 147456;
template <typename T> hipError_t launch_verify(VerifyParams p, hipStream_t s, int phases) {
  if constexpr (ExpTab<T>::kHas) {
    const bool chosen = !std::is_same<T, F16>::value || (p.V >= kBitMinV16 && p.B * (p.gamma + 1) > round_rows<PowTerms<T>>());
    if (chosen && exp_table_usable<T>(p.rT)) return launch_verify_with<T, BitTerms<T>>(p, s, phases);
  }
  return launch_verify_with<T, PowTerms<T>>(p, s, phases);
}

}  // namespace tslt
