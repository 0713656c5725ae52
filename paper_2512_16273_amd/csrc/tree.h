// tslt_verify_tree: token-tree verification (Algorithm 8) with multi-candidate verification
// (Algorithm 5) at every non-leaf node.  Nodes are stored breadth-first (Section 4.1).
//
// With a sparse q_hat the distribution p^(i) is a vector a on the set and a scalar multiple c of p outside it,
// and the update p^(i+1) = norm(max(0, p^(i) - q_hat)) is a <- max(0, a - q_hat) / Z, c <- c / Z with
// Z = sum(max(0, a - q_hat)) + c * p_out: one dense pass per node, O(k * K) work for the k candidates, and the
// sums of that pass serve the draw as well (rowsample.h).  Bound by the vector units (fp32: 19 instructions an element,
// 5.5 TB/s) or the LDS (bfloat16).  Two fp32 trees of 1365 nodes, V = 151936, every node: 546 us as a pass for the
// tests, a sweep, a finish and two more launches, 302 so; the path of 64 binary16 trees <2,2,2>, V = 32000: 52 and 39.5.
// Paths over long rows take the tests on the way from an fp32 pass (rowops.h) and sweep the last node alone.
#pragma once
#include "rowops.h"
#include "rowsample.h"

namespace tslt {

constexpr int kMaxTreeDepth = 16;
constexpr int kMaxBranch = 16;
constexpr int64_t kXcds = 8;             // consecutive workgroups go to one after the other of them
static_assert(kMaxBranch <= kMaxStages, "a stage to a candidate");

struct TreeParams {
  const void* target;
  int64_t B, V, row_stride;
  int n_nodes, n_int, depth;
  int expansion[kMaxTreeDepth];
  int offsets[kMaxTreeDepth + 2];     // first node of every layer; offsets[depth + 1] = n_nodes
  float rT, k2;
  const int32_t* q_idx;
  const float* q_logit;
  const int32_t* q_count;
  int k_cap;
  int wor;                // candidates were drawn without replacement: stage proposals are renormalised
  const int32_t* cand_tokens;
  const float* u_accept;
  const float* u_resample;
  int32_t* out_node_token;
  int32_t* out_node_slot;
  int32_t* out_seq;
  int32_t* out_len;
  float* out_ratio;
  float* out_beta;        // [B, n_nodes - 1] stage acceptance rate sum_x min(q^(i), p^(i)) of every tested candidate
  int32_t* status;
  // workspace
  // (every node evaluated only)
  int32_t* node_slot;     // [B, n_nodes] accepted child number or -1
  int32_t* node_token;    // [B, n_nodes] the node's output
  int32_t* node_status;   // [B, n_nodes]
  // (path only, tree_quick_kernel first)
  int32_t* walk_node;     // [B] where the quick walk stopped
  int32_t* walk_status;   // [B] status bits of the nodes before it
  // masses of shared rows' items: of the node where the quick walk stopped [B, items_stride], or of every node evaluated at
  // once [B, n_eval, items_stride]
  double* items;
  int64_t items_stride;
  int parts;              // workgroups that share a row
  int turn;               // a path's workgroups are this many apart
  uint64_t* part_words;   // [rows, parts]: theirs (handover.h)
  uint64_t* words;        // [B, n_nodes, 2]: what the workgroups of a tree's nodes leave, in place of the node arrays (else null)
  Tag tag;
  int all_nodes;
  int n_eval;             // nodes of a tree that tree_node_kernel evaluates: whole layers from the root
  int n_eval_layers;
  int64_t items_rows;     // there is room for (read on the host)
};

// (Evaluating every node uses three of the four node arrays and, where the rows of few nodes are shared by workgroups, the masses of
// their items; the two words a tree are for the path.  With node outputs masses are asked for once a node: the size that
// callers have been told all along, so that a workspace kept from an earlier version and one sized by this one are the same.
// For the path a call may be given less than it is told to bring: the rows of a small tree's nodes are then not shared.)
inline size_t tree_least_workspace_bytes(int64_t B, int64_t n_nodes, int64_t V, bool all_nodes) {
  const size_t n_seg = size_t(row_segments(V));
  const size_t tasks = all_nodes ? size_t(n_nodes) : 1;
  return align256(size_t(B) * n_nodes * 4) * 4 + align256(size_t(B) * 4) * 2 +
         align256(size_t(B) * tasks * (n_seg + 2) * 16) +
         align256(size_t(B) * tasks * n_seg * kSubChunks * sizeof(double));
}
inline size_t tree_workspace_bytes(int64_t B, int64_t n_nodes, int64_t V, bool all_nodes) {
  const size_t least = tree_least_workspace_bytes(B, n_nodes, V, all_nodes);
  if (V < kShareLeastV) return least;
  const size_t arrays = align256(size_t(B) * n_nodes * 4) * 4 + align256(size_t(B) * 4) * 2;
  const size_t rows = arrays + size_t(kShareWords) * 8 + align256(size_t(std::min(B * n_nodes, kShareRows) * items_stride(V)) * sizeof(double));
  return std::max(least, rows);
}
inline void tree_carve_workspace(TreeParams& p, void* ws, size_t ws_bytes, int per_vec) {
  const size_t per = align256(size_t(p.B) * p.n_nodes * 4);
  char* w = reinterpret_cast<char*>(ws) + per;       // (the first of the four node arrays that are asked for is not used ...)
  p.words = reinterpret_cast<uint64_t*>(ws);         // (... but where these words take their place, 16 bytes a node)
  p.node_slot = reinterpret_cast<int32_t*>(w); w += per;
  p.node_token = reinterpret_cast<int32_t*>(w); w += per;
  p.node_status = reinterpret_cast<int32_t*>(w); w += per;
  p.walk_node = reinterpret_cast<int32_t*>(w); w += align256(size_t(p.B) * 4);
  p.walk_status = reinterpret_cast<int32_t*>(w); w += align256(size_t(p.B) * 4);
  p.part_words = reinterpret_cast<uint64_t*>(w); w += size_t(kShareWords) * 8;
  p.items = reinterpret_cast<double*>(w);
  p.items_stride = items_stride(p.V, per_vec);
  const int64_t left = int64_t(ws_bytes) - int64_t(w - reinterpret_cast<char*>(ws));
  p.items_rows = left > 0 ? left / (p.items_stride * int64_t(sizeof(double))) : 0;
}

template <typename T> __device__ __forceinline__ const void* tree_row(const TreeParams& p, int64_t b, int node) {
  return reinterpret_cast<const char*>(p.target) +
         (size_t(b) * p.n_nodes + node) * size_t(p.row_stride) * ElemTraits<T>::kBytes;
}
__device__ __forceinline__ int tree_layer(const TreeParams& p, int node) {
  int l = 0;
  while (l < p.depth && node >= p.offsets[l + 1]) ++l;
  return l;
}
// first child of a non-leaf node: the i-th node of layer l owns nodes i*k .. i*k + k-1 of layer l+1
__device__ __forceinline__ int tree_first_child(const TreeParams& p, int node, int layer) {
  return p.offsets[layer + 1] + (node - p.offsets[layer]) * p.expansion[layer];
}

// ---------------------------------------------------------------------------------------------
// One node of tree b, by all threads of a workgroup: Algorithm 5 at a non-leaf node, then, unless a child was
// accepted, the draw of its output (a leaf: of its target distribution).  Writes the ratios and rates of the
// candidates it tested; returns the state (0 sampled, 1 a child accepted, 2 row unusable), the accepted child in
// `slot`, the output in `token` and the status bits in `st` (both as the first wave has them).  Unless a child was
// accepted the terms' table is used up.  kParts: p.parts workgroups share the row, `row_at` in order, of which this one is
// `part`; state 3 where it leaves the node to another.  kOnce: the workgroup has no other row to sweep.
// ---------------------------------------------------------------------------------------------
// (A candidate's ratio and rate go straight to memory where another workgroup may write over them.)
__device__ __forceinline__ void store_rate(float* to, float v, bool through) {
  if (through) __hip_atomic_store(to, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *to = v;
}
template <typename T, typename Terms, bool kOneCopy = false, int kLoads = kStreamed, bool kParts = false, bool kOnce = false>
__device__ __forceinline__ int tree_node(const TreeParams& p, int64_t b, int node, double* table, bool build, RowShared& sh,
                                         int& slot, int& token, int& st, int64_t row_at = 0, int part = 0) {
  const int lane = lane_id();
  const bool leaf = node >= p.n_int;
  const int64_t row = b * p.n_int + (leaf ? 0 : node);
  RowWork<T> w;
  row_open<T>(w, tree_row<T>(p, b, node), p.V, p.rT, sh);
  row_take_set(w, p.q_idx + size_t(row) * p.k_cap, p.q_logit + size_t(row) * p.k_cap, leaf ? 0 : p.q_count[row], p.k_cap);
  const float u_res = p.u_resample[size_t(b) * p.n_nodes + node];
  // candidate `lane` of a non-leaf node
  const int layer = tree_layer(p, node);
  const int k = leaf ? 0 : p.expansion[layer];
  const int64_t c0 = leaf ? 0 : b * (p.n_nodes - 1) + tree_first_child(p, node, layer) - 1;
  const int my_cand = p.cand_tokens[c0 + (lane < k ? lane : 0)];
  const float my_u = p.u_accept[c0 + (lane < k ? lane : 0)];
  if constexpr (kParts) {
    if (!row_shared<T, Terms, kLoads>(w, table, AskWithRow{}, part, p.parts, p.items + row_at * p.items_stride, p.part_words + row_at * p.parts, p.tag, sh))
      return 3;
  } else {
    row_sweep<T, Terms, kOneCopy, kLoads>(w, table, build ? -1 : -2, AskWithRow{}, sh);
  }
  if (kOnce) row_clear<T>(table);                                   // (the table is not needed for another row)
  token = -1;
  st = 0;
  float my_ratio = NAN, my_beta = NAN;                              // NaN if the candidate is never tested
  const int waves = row_set_waves(w), wave = __builtin_amdgcn_readfirstlane(wave_id());
  if (wave < waves) {
    RowState r;
    row_eval(w, r, sh);
    int accepted = -1, barriers = 0;
    double part = -1.0;                                             // of the last rejection, whose update is still to be made
    if (!leaf) {
      int gone = -1;
      if (r.ok) {
        for (int i = 0; i < k; ++i) {
          const int x = __builtin_amdgcn_readlane(my_cand, i);
          if (x < 0) continue;                                      // absent candidate
          if (part >= 0.0) {                                        // the candidate before was rejected
            row_update(w, r, part, gone);
            if (p.wor) {
              const double rest = 1.0 - r.removed;
              r.qscale = rest > 0.0 ? 1.0 / rest : 0.0;
            }
          }
          row_test(w, r, x, barriers, sh);
          __syncthreads();
          const RowTest t = row_tested(waves, barriers, sh);
          ++barriers;
          if (!t.found) r.st |= 4;
          if (lane == i) { my_ratio = float(t.ratio); my_beta = float(t.shared); }   // Section 4.3's beta^(i)
          const double bound = t.ratio < 1.0 ? t.ratio : 1.0;
          const float u = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_u), i));
          if (same_in_wave(t.found && double(u) < bound)) { accepted = i; token = x; break; }
          part = t.part;
          // drawn without replacement: x leaves the urn and what is left is renormalised
          gone = p.wor && t.found ? x : -1;
          if (gone >= 0) r.removed += t.q_x;
        }
      }
    }
    const bool draw = accepted < 0 && r.ok;
    const bool pending = draw && part >= 0.0 && row_has_residual(r, part);
    const bool updated = draw && (r.stages > 0 || pending);         // not at a leaf or where every candidate is absent
    // (where there is an update there has been a test, and a barrier behind every wave's look at the masses)
    const double corr = updated ? row_correct(w, r, pending, part, sh) : 0.0;
    if (wave == 0 && lane == 0) sh.stop_at = barriers + 1;
    __syncthreads();
    if (wave == 0) {
      if (draw) row_locate(w, r, u_res, updated, corr, sh);
      st = r.st;
      if (lane == 0) sh.cmd = accepted >= 0 ? accepted : (r.ok ? -1 : -2);
    }
  } else {
    // the others pass as many barriers, whose number they learn at the last of them
    int barriers = 0;
    do {
      __syncthreads();
      ++barriers;
    } while (__builtin_amdgcn_readfirstlane(sh.stop_at) != barriers);
  }
  __syncthreads();
  slot = sh.cmd;
  if (threadIdx.x < k) {
    const bool through = p.words != nullptr && !p.all_nodes;
    if (p.out_ratio) store_rate(&p.out_ratio[c0 + lane], my_ratio, through);
    if (p.out_beta) store_rate(&p.out_beta[c0 + lane], my_beta, through);
  }
  if (slot >= 0) return 1;
  const int state = slot == -1 ? 0 : 2;
  slot = -1;
  if (state == 0) {
    if (!kOnce) {
      row_clear<T>(table);
      __syncthreads();
    }
    token = row_pick(w, table, sh);
  }
  return state;
}

// The new-sequence search through the layers that have been evaluated: all threads of the calling workgroup; the first
// appends the outputs to out_seq and notes the candidates that were tested.  The nodes' accepted children, outputs and
// status words are brought into LDS first, all at once, where they fit (`room` words at `nodes`): one memory latency in
// place of one for every layer (two trees of 1365 nodes in six layers: 12 us by one thread out of memory, 5 so).
struct TreeWalk {
  int first_cand[kMaxTreeDepth + 1], n_cand[kMaxTreeDepth + 1];      // of every node passed
  int n_passed, node, layer, len, status, done;
  int all_status;                                                    // of every node evaluated (if they were looked at)
};
// One thread: at(node) gives a node's accepted child (-1: none), output and status bits.
template <typename F> __device__ __forceinline__ void tree_search(const TreeParams& p, int64_t b, TreeWalk& w, F at) {
  int32_t* seq = p.out_seq + size_t(b) * (p.depth + 1);
  int node = 0, layer = 0, len = 0, st = 0, done = 0;
  while (!done && layer < p.n_eval_layers) {
    int slot, token, status;
    at(node, slot, token, status);
    st |= status;
    seq[len++] = token;
    done = 1;
    if (node >= p.n_int) break;
    const int child = tree_first_child(p, node, layer);
    w.first_cand[layer] = child - 1;
    w.n_cand[layer] = p.expansion[layer];
    ++layer;
    if (slot >= 0) {
      node = child + slot;
      done = 0;
    }
  }
  w.n_passed = layer;
  w.node = node;
  w.layer = layer;
  w.len = len;
  w.status = st;
  w.done = done;
}
__device__ __forceinline__ void tree_walk(const TreeParams& p, int64_t b, TreeWalk& w, int32_t* nodes, int room) {
  const int tid = threadIdx.x, n = p.n_eval;
  const bool here = 3 * n <= room;
  if (tid == 0) w.all_status = 0;
  __syncthreads();
  if (here || p.all_nodes) {
    int st = 0;
    for (int i = tid; i < n; i += blockDim.x) {
      const int64_t at = b * p.n_nodes + i;
      const int status = p.node_status[at];
      st |= status;
      if (here) {
        nodes[i] = p.node_slot[at];
        nodes[n + i] = p.node_token[at];
        nodes[2 * n + i] = status;
      }
    }
    st = wave_or_i32(st);
    if (lane_id() == 0 && st) atomicOr(&w.all_status, st);
  }
  __syncthreads();
  if (tid == 0) {
    tree_search(p, b, w, [&](int node, int& slot, int& token, int& status) {
      const int64_t at = b * p.n_nodes + node;
      slot = here ? nodes[node] : p.node_slot[at];
      token = here ? nodes[n + node] : p.node_token[at];
      status = here ? nodes[2 * n + node] : p.node_status[at];
    });
  }
  __syncthreads();
}
// The ratios and rates of the candidates of all other nodes: NaN.
__device__ __forceinline__ void tree_clear_others(const TreeParams& p, int64_t b, const TreeWalk& w, int threads) {
  for (int i = threadIdx.x; i < p.n_nodes - 1; i += threads) {
    bool tested = false;
    for (int l = 0; l < w.n_passed; ++l) tested |= i >= w.first_cand[l] && i < w.first_cand[l] + w.n_cand[l];
    if (tested) continue;
    if (p.out_ratio) p.out_ratio[size_t(b) * (p.n_nodes - 1) + i] = NAN;
    if (p.out_beta) p.out_beta[size_t(b) * (p.n_nodes - 1) + i] = NAN;
  }
}

// What every node evaluated gives as a tree's outputs.
__device__ __forceinline__ void tree_write(const TreeParams& p, int64_t b, const TreeWalk& w, int threads) {
  if (threadIdx.x == 0) {
    p.out_len[b] = w.len;
    for (int i = w.len; i <= p.depth; ++i) p.out_seq[size_t(b) * (p.depth + 1) + i] = -1;
    if (p.status) p.status[b] = p.all_nodes ? w.all_status : w.status;
  }
  if (!p.all_nodes) tree_clear_others(p, b, w, threads);
}

// ---------------------------------------------------------------------------------------------
// Every node of the layers wanted: one workgroup per node, or p.parts of them (kParts).  Where those are the whole of a tree of no
// more than kHandNodes, what a node came to is left in memory (handover.h) and the workgroup that finds all of its tree's
// searches the new sequence at once; else tree_walk_kernel or tree_path_kernel does, from the node arrays.
// ---------------------------------------------------------------------------------------------
constexpr int kHandNodes = 256;
template <typename T, typename Terms, int kWavesPerSimd, bool kParts = false>
__global__ __launch_bounds__(kRowThreads, kWavesPerSimd) void tree_node_kernel(const TreeParams p) {
  __shared__ RowShared sh;
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  const uint32_t at = kParts ? blockIdx.x / uint32_t(p.parts) : blockIdx.x;      // (a division by 64 bits takes half a microsecond)
  const int64_t b = at / uint32_t(p.n_eval);
  const int node = int(at - uint32_t(b) * p.n_eval);
  int slot, token, st;
  if (tree_node<T, Terms, kWavesPerSimd == kAlone, kStreamed, kParts, true>(p, b, node, reinterpret_cast<double*>(dyn_lds), true, sh, slot, token, st,
                                                                      at, int(blockIdx.x - at * p.parts)) == 3) return;
  if (wave_id() != 0) return;
  const int64_t n = b * p.n_nodes + node;
  auto node_outputs = [&]() {
    if (p.out_node_token) p.out_node_token[n] = token;
    if (p.out_node_slot) p.out_node_slot[n] = slot;
  };
  if (p.words == nullptr) {
    if (threadIdx.x == 0) {
      node_outputs();
      p.node_slot[n] = slot;
      p.node_token[n] = token;
      p.node_status[n] = st;
    }
    return;
  }
  // The candidates' ratios and rates are at memory before the words, for whoever finds these may write NaN over them.  (A node that
  // draws has had them there since its search.)
  stores_arrived();
  if (threadIdx.x == 0) node_outputs();
  // (nothing of the row is needed any more)
  int* tokens = sh.set_y;
  int* state = reinterpret_cast<int*>(sh.set_e);
  TreeWalk& walk = *reinterpret_cast<TreeWalk*>(sh.set_a);
  static_assert(sizeof(TreeWalk) <= sizeof(sh.set_a) && kHandNodes <= kRowThreads, "room in LDS");
  if (!hand_over(p.words + 2 * size_t(b) * p.n_nodes, node, p.n_nodes, uint32_t(token), uint32_t((slot + 1) | st << 8), p.tag, tokens, state)) return;
  int all = 0;
  for (int i = lane_id(); i < p.n_nodes; i += 64) all |= state[i] >> 8;
  all = wave_or_i32(all);
  if (threadIdx.x == 0) {
    walk.all_status = all;
    tree_search(p, b, walk, [&](int i, int& s, int& t, int& status) {
      s = (state[i] & 255) - 1;
      t = tokens[i];
      status = state[i] >> 8;
    });
  }
  wave_sync();
  tree_write(p, b, walk, 64);
}

// One workgroup per tree, after every node has been evaluated.
constexpr int kWalkNodes = 3 * 4000;                                 // words: 47 KB
__global__ __launch_bounds__(1024) void tree_walk_kernel(const TreeParams p) {
  __shared__ TreeWalk w;
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  const int64_t b = blockIdx.x;
  tree_walk(p, b, w, reinterpret_cast<int32_t*>(dyn_lds), 3 * p.n_eval <= kWalkNodes ? kWalkNodes : 0);
  tree_write(p, b, w, blockDim.x);
}

// ---------------------------------------------------------------------------------------------
// The quick walk, for paths only: one workgroup per tree (of 512 threads, or 256 where trees outnumber compute units) runs
// Algorithm 5 from the root on as long as a candidate is accepted, on rowops.h's pass of fp32 terms.  It stops at a leaf,
// at a node that accepts none (whose output has to be drawn) and wherever the fp32 terms have nothing to say: an unusable
// row or set, or a rejection that leaves less than kQuickResidual.  From there on the fp64 kernels decide for themselves.
// ---------------------------------------------------------------------------------------------
constexpr double kQuickResidual = 0x1p-10;
template <typename T, int NT>
__device__ __forceinline__ int tree_quick_node(const TreeParams& p, int64_t b, int node, int layer, VerifyShared& sh, int& st) {
  constexpr int kPer = 1024 / NT;
  const int tid = threadIdx.x;
  const int k = p.expansion[layer];
  const int64_t c0 = b * (p.n_nodes - 1) + tree_first_child(p, node, layer) - 1;
  const void* row = tree_row<T>(p, b, node);
  const RowSplit rs = split_row<T>(row, p.V);
  const int64_t r = b * p.n_int + node;
  int count = p.q_count[r];
  count = count < 0 ? 0 : (count > p.k_cap ? p.k_cap : count);
  double a_s[kPer], q_s[kPer], p_out;
  int yi[kPer];
  bool ok;
  eval_row_on_set<T, true, NT>(row, rs, p.V, p.rT, p.k2, p.q_idx + size_t(r) * p.k_cap, p.q_logit + size_t(r) * p.k_cap, count, sh,
                           a_s, q_s, yi, p_out, ok, st);
  if (!ok) return -1;
  double c = 1.0, qscale = 1.0, removed = 0.0;       // the stage's proposal is q_s * qscale
  for (int i = 0; i < k; ++i) {
    const int x = p.cand_tokens[c0 + i];
    if (x < 0) continue;                             // absent candidate (block-uniform)
    if (tid == 0) { sh.bcast_d[0] = -1.0; sh.bcast_d[1] = 0.0; sh.bcast_i[0] = 0; }
    __syncthreads();
    double shared = 0.0, part = 0.0;
    int mine = -1;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const double qq = q_s[q] * qscale, d = a_s[q] - qq > 0.0 ? a_s[q] - qq : 0.0;
      shared += yi[q] >= 0 ? a_s[q] - d : 0.0;       // min(a, q)
      part += yi[q] >= 0 ? d : 0.0;
      if (yi[q] == x && q_s[q] > 0.0 && atomicCAS(&sh.bcast_i[0], 0, 1) == 0) {
        sh.bcast_d[0] = a_s[q] / qq;
        sh.bcast_d[1] = q_s[q];
        mine = q;
      }
    }
    double none = 0.0;
    block_sum3_f64<NT / 64>(shared, part, none, sh.red);      // (and its barriers)
    const double ratio = sh.bcast_d[0], q_x = sh.bcast_d[1];
    const bool found = sh.bcast_i[0] != 0;
    __syncthreads();
    if (!found) st |= 4;
    if (tid == 0) {
      if (p.out_ratio) p.out_ratio[c0 + i] = float(ratio);
      if (p.out_beta) p.out_beta[c0 + i] = float(shared);    // Section 4.3's beta^(i)
    }
    const double bound = ratio < 1.0 ? ratio : 1.0;
    if (found && double(p.u_accept[c0 + i]) < bound) return i;
    const double Z = part + c * p_out;
    if (!(Z > kQuickResidual * c)) return -1;
    const double inv_Z = 1.0 / Z;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const double d = a_s[q] - q_s[q] * qscale;
      a_s[q] = yi[q] >= 0 && d > 0.0 ? d * inv_Z : 0.0;
      if (p.wor && found && q == mine) q_s[q] = 0.0;         // drawn without replacement: x leaves the urn
    }
    c *= inv_Z;
    if (p.wor && found) {
      removed += q_x;
      const double rest = 1.0 - removed;
      qscale = rest > 0.0 ? 1.0 / rest : 0.0;
    }
  }
  return -1;
}
template <typename T, int NT>
__global__ __launch_bounds__(NT) void tree_quick_kernel(const TreeParams p) {
  __shared__ VerifyShared sh;
  const int tid = threadIdx.x;
  const int64_t b = blockIdx.x;
  for (int i = tid; i < p.n_nodes - 1; i += NT) {
    if (p.out_ratio) p.out_ratio[size_t(b) * (p.n_nodes - 1) + i] = NAN;
    if (p.out_beta) p.out_beta[size_t(b) * (p.n_nodes - 1) + i] = NAN;
  }
  __syncthreads();
  int node = 0, layer = 0, st_all = 0;
  while (node < p.n_int) {
    int st;
    const int slot = tree_quick_node<T, NT>(p, b, node, layer, sh, st);
    if (slot < 0) break;                     // (its ratios are written again by the node's evaluation)
    st_all |= st;
    node = tree_first_child(p, node, layer) + slot;
    if (tid == 0) p.out_seq[size_t(b) * (p.depth + 1) + layer] = p.cand_tokens[b * (p.n_nodes - 1) + node - 1];
    ++layer;
  }
  if (tid == 0) {
    p.walk_node[b] = node;
    p.walk_status[b] = st_all;
  }
}

// ---------------------------------------------------------------------------------------------
// Only the verified path is wanted: one workgroup per tree takes up the walk where it has got to, then goes from node to
// node, running Algorithm 5 at each node it reaches, descending into the accepted child and drawing the output of the
// node it stops at, so that a target row is read only where it counts.  Uniforms are indexed by node, so the result is
// the one that evaluating every node gives.  The node at which the quick walk stopped may be shared by p.parts workgroups; the one that
// finds its masses complete goes on alone.  (The walk through evaluated layers is not compiled into the other forms,
// whose registers it costs.)
// ---------------------------------------------------------------------------------------------
enum { kFromRoot = 0, kFromHead = 1, kFromQuick = 2 };      // nothing done yet; the first layers evaluated; the quick walk
template <typename T, typename Terms, int kFrom, int kLoads = kStreamed, bool kParts = false>
__global__ __launch_bounds__(kRowThreads) void tree_path_kernel(const TreeParams p) {
  __shared__ RowShared sh;
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  const int tid = threadIdx.x;
  const uint32_t part = kParts ? blockIdx.x / uint32_t(p.turn) : 0u, tree = kParts ? blockIdx.x - part * uint32_t(p.turn) : blockIdx.x;
  if (kParts && tree >= uint32_t(p.B)) return;
  const int64_t b = tree;
  int node = 0, layer = 0, len = 0, st_all = 0, token = -1;
  bool done = false;
  if constexpr (kFrom == kFromHead) {
    __shared__ TreeWalk walk;
    tree_walk(p, b, walk, reinterpret_cast<int32_t*>(dyn_lds), int(Terms::kBytes / 4));      // (the terms' table comes later)
    tree_clear_others(p, b, walk, kRowThreads);
    node = walk.node;
    layer = walk.layer;
    len = walk.len;
    st_all = walk.status;
    done = walk.done;
  } else if constexpr (kFrom == kFromQuick) {
    node = p.walk_node[b];
    layer = len = tree_layer(p, node);
    st_all = p.walk_status[b];
  } else {
    for (int i = tid; i < p.n_nodes - 1; i += kRowThreads) {
      if (p.out_ratio) p.out_ratio[size_t(b) * (p.n_nodes - 1) + i] = NAN;
      if (p.out_beta) p.out_beta[size_t(b) * (p.n_nodes - 1) + i] = NAN;
    }
  }
  __syncthreads();
  int32_t* seq = p.out_seq + size_t(b) * (p.depth + 1);
  bool build = true;                         // the terms' table is still to be made
  bool shared = kParts;
  while (!done) {
    int slot, st, state;
    if (kParts && shared) {
      state = tree_node<T, Terms, false, kLoads, kParts>(p, b, node, reinterpret_cast<double*>(dyn_lds), true, sh, slot, token, st, b,
                                                         int(part));
      if (state == 3) return;
      shared = false;
    } else {
      state = tree_node<T, Terms, false, kLoads>(p, b, node, reinterpret_cast<double*>(dyn_lds), build, sh, slot, token, st);
      build = false;
    }
    st_all |= st;
    if (tid == 0) seq[len] = token;
    ++len;
    if (state != 1) break;
    node = tree_first_child(p, node, layer) + slot;
    ++layer;
  }
  if (tid == 0) {
    p.out_len[b] = len;
    for (int i = len; i <= p.depth; ++i) seq[i] = -1;
    if (p.status) p.status[b] = st_all;
  }
}

// How many layers of a tree whose path is wanted are evaluated at once, every node of them, before the path is walked:
// rows on the chip together take one row's time where the walk takes one for every layer.  The whole tree, where it
// comes to one row per compute unit, or two unless they are binary16 rows of two layers; else, for rows of 100000
// and more, the largest head of at least two layers that comes to one, where as many are left at most.  us a call,
// layers one by one / at once (V = 32000, then 152064): 8 trees <2,2,2>, all layers, binary16 35.9 / 22.7 and 94 / 32,
// fp32 36.4 / 19.4 and 94 / 34.6; 30 such trees, fp32 37.0 / 27.6 and 95 / 70, bfloat16 29 / 24.3 and 58 / 40; 34
// trees <4,2> binary16 29.4 / 34.2 and 55 / 58; two of the four layers of 64 trees <2,2,2>: binary16 39 / 45 and
// 100 / 95, fp32 36.8 / 37.8 and 96 / 84, bfloat16 28.6 / 33.2 and 59 / 56.
template <typename T> inline int layers_at_once(const TreeParams& p) {
  const int64_t cus = compute_units();
  const bool two = p.depth >= 3 || !std::is_same<T, F16>::value;
  if (p.B * p.n_nodes <= cus * (two ? 2 : 1)) return p.depth + 1;
  if (p.V < 100000) return 0;
  int l = p.depth;
  while (l > 0 && p.B * p.offsets[l] > cus) --l;
  return l >= 2 && 2 * l >= p.depth + 1 ? l : 0;
}

// Whether a path that does not fit the chip at once is walked quickly first.  With terms from the bit table a node's fp64
// sweep costs no more than the fp32 pass; the others' is bound by the vector units (19 instructions a term), and one
// compute unit to a tree takes them all.  So: long rows of several layers; where trees outnumber compute units, shorter
// ones too.  Where more than half of the layers fit the chip at once they are evaluated so (unless few layers of the
// longest 16-bit rows).  us a call, in fp64 node by node (head layers at once from 100000 on) / quick walk:
//   binary16  64 <4,2> 64000 41.7 / 43.4, 99968 57.4 / 47;  64 <2,2,2> 48000 45.7 / 43.4, 64000 54.5 / 48, 152064 81.9 / 68;
//             20 <4,2,2,1> 256000 179.8 / 102;  12 <4,4,4> 152064 65.3 / 71.4, 256000 103 / 84;  8 <2,2,2,2,2,2> 256000 107 / 139;
//             300 <2,2,2> 32000 56.6 / 58.6, 64000 84.3 / 82.9;  512 <1,1,1,1> 16000 63.4 / 56.5, 32000 84.9 / 69
//   fp32      64 <2,2,2> 64000 50.8 / 51.5, 99968 70.3 / 61;  128 <2,2,2> 99968 70.2 / 72.1;  128 <3,3> 152064 74.2 / 71.3;
//             512 <1,1,1,1> 16000 62.4 / 60.1, 32000 85.7 / 77.9;  400 <4,2> 64000 79.1 / 81.7, 99968 111.9 / 105.4
// Against the walk of fp64 sums the ratios' error stays what it was (2.4e-8 to 4.3e-8, the outputs' rounding).
template <typename T, typename Terms> inline bool quick_walk(const TreeParams& p, int layers_first) {
  if (Terms::kBits || p.depth < 2) return false;
  const int64_t cus = compute_units();
  if (ElemTraits<T>::kBytes == 2) {
    if (2 * layers_first > p.depth + 1) return p.V >= 200000 && p.depth <= 3;
    return p.V >= (p.B >= 2 * cus ? 12000 : (2 * p.B >= 3 * cus ? 32000 : (p.depth > 2 ? 64000 : 80000)));
  }
  if (2 * layers_first > p.depth + 1) return false;
  return p.V >= (p.B >= 2 * cus ? 32000 : (p.B > cus || 4 * p.B <= cus ? 96000 : 150000));
}
template <typename T, typename Terms> hipError_t launch_verify_tree_with(TreeParams p, hipStream_t s) {
  p.n_eval_layers = p.all_nodes ? p.depth + 1 : layers_at_once<T>(p);
  const bool quick = p.n_eval_layers <= p.depth && quick_walk<T, Terms>(p, p.n_eval_layers);
  if (quick) p.n_eval_layers = 0;
  p.n_eval = p.offsets[p.n_eval_layers];
  hipError_t e = hipSuccess;
  if (p.n_eval > 0) {
    // (one binary16 tree of 13 nodes, V = 9728: 18.3 us with 64 registers, 17.5 with 128)
    const int64_t rows = p.B * p.n_eval;
    const bool alone = rows <= compute_units();
    p.parts = rows <= p.items_rows ? row_parts<T, Terms>(p.V, rows) : 1;
    // (handing over keeps a workgroup a microsecond longer: of many times what the chip holds at once, more than the launch that it saves.
    // 117 trees <4,4,4> of fp32 rows of 17296, 9945 rows, 220 us by a second launch, 239 so; 14 such trees of bfloat16 9083 37.4 / 34.3.
    // And where each looks at many words: trees of 255 nodes, 3 binary16 of rows of 8000 26.3 / 27.6, 3 fp32 of 30000 34.0 / 36.8, 2 binary16 18.9 / 19.0,
    // 2 fp32 25.4 / 24.7; of 85, 12 binary16 of 8000 30.0 / 31.1, 9 fp32 35.8 / 35.8, 6 binary16 19.8 / 18.8; of 15, 50 binary16 26.3 / 25.6.)
    if (p.n_eval_layers <= p.depth || p.n_nodes > kHandNodes || rows > (p.n_nodes > 128 ? 2 : 4) * compute_units()) p.words = nullptr;
    p.tag = next_tag();
    hipLaunchKernelGGL((p.parts > 1 ? tree_node_kernel<T, Terms, kAlone, true> : alone ? tree_node_kernel<T, Terms, kAlone> : tree_node_kernel<T, Terms, kShared>),
                       dim3(unsigned(rows * p.parts)), dim3(kRowThreads), Terms::kBytes, s, p);
    if ((e = hipGetLastError()) != hipSuccess || p.words != nullptr) return e;
  }
  p.words = nullptr;
  auto walk = [&](auto fn) {
    hipLaunchKernelGGL(fn, dim3(unsigned(p.B)), dim3(kRowThreads), Terms::kBytes, s, p);
    return hipGetLastError();
  };
  if constexpr (!Terms::kBits) {
    if (quick) {
      if (p.B <= compute_units()) hipLaunchKernelGGL((tree_quick_kernel<T, 512>), dim3(unsigned(p.B)), dim3(512), 0, s, p);
      else hipLaunchKernelGGL((tree_quick_kernel<T, 256>), dim3(unsigned(p.B)), dim3(256), 0, s, p);
      if ((e = hipGetLastError()) != hipSuccess) return e;
      // as many workgroups to a row as fill the chip, a run for every wave at least
      const int64_t runs = p.V / (ElemTraits<T>::kPerVec * kRunVecs) + 1;
      p.parts = p.B <= p.items_rows ? int(std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(compute_units(), kShareWords) / p.B, (runs + kRowWaves - 1) / kRowWaves))) : 1;
      auto last_rows = [&](auto loads) -> hipError_t {
        constexpr int kLoads = decltype(loads)::value;
        if (p.parts == 1) return walk(tree_path_kernel<T, typename Terms::Walked, kFromQuick, kLoads>);
        p.tag = next_tag();
        // On the XCD on which the tree has been walked, where that leaves a compute unit to each: every part reads the set and gathers the row at
        // it, and eight L2s full of that had the quick walk fetch its sets again.  us in a launch each / side by side / so, 40 binary16 trees
        // <2,2,2> of 64000, sets of 16 49.3 / 49.2 / 49.5, of 400 52.5 / 51.8 / 51.7, of 1024 58.6 / 60.1 / 55.9; of 100000, sets of 400 59.4 / 60.3 /
        // 58.4; 64 fp32 of 151936, sets of 400 79.7 / 80.2 / 78.3.  50 fp32 of 151936, sets of 32, 7 trees of 5 parts on one XCD: 73.4 / 73.2 / 82.4.
        const int64_t per_xcd = (p.B + kXcds - 1) / kXcds;
        p.turn = int(per_xcd * p.parts * kXcds <= compute_units() ? per_xcd * kXcds : p.B);
        hipLaunchKernelGGL((tree_path_kernel<T, typename Terms::Walked, kFromQuick, kLoads, true>), dim3(unsigned(p.turn * p.parts)), dim3(kRowThreads), Terms::kBytes, s, p);
        return hipGetLastError();
      };
      if constexpr (ElemTraits<T>::kBytes == 4) {
        if (p.B * p.n_nodes * p.V * 4 > kStreamTreeBytes) return last_rows(std::integral_constant<int, kCached>{});
      }
      return last_rows(std::integral_constant<int, kStreamed>{});
    }
  }
  if (p.n_eval == 0) {
    if constexpr (ElemTraits<T>::kBytes == 4) {
      if (p.V < kByAddressV) return walk(tree_path_kernel<T, typename Terms::Walked, kFromRoot, kByAddress>);
    }
    return walk(tree_path_kernel<T, typename Terms::Walked, kFromRoot>);
  }
  if (p.n_eval_layers <= p.depth) return walk(tree_path_kernel<T, typename Terms::Walked, kFromHead>);
  const int threads = std::min(1024, (p.n_eval + 63) / 64 * 64);
  hipLaunchKernelGGL(tree_walk_kernel, dim3(unsigned(p.B)), dim3(threads), 3 * p.n_eval <= kWalkNodes ? 12 * p.n_eval : 0, s, p);
  return hipGetLastError();
}
template <typename T> hipError_t launch_verify_tree(const TreeParams& p, hipStream_t s) {
  if constexpr (std::is_same<T, Bf16>::value) {
    if (exp_table_usable<T>(p.rT)) return launch_verify_tree_with<T, BitTerms<T>>(p, s);
  }
  return launch_verify_tree_with<T, PowTerms<T>>(p, s);
}

}  // namespace tslt
