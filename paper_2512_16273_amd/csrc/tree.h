// tslt_verify_tree: token-tree verification (Algorithm 8) with multi-candidate verification
// (Algorithm 5) at every non-leaf node.  Nodes are stored breadth-first (Section 4.1).
//
// With a sparse q_hat the distribution p^(i) is a vector a on the set and a scalar multiple c of p outside it,
// and the update p^(i+1) = norm(max(0, p^(i) - q_hat)) is a <- max(0, a - q_hat) / Z, c <- c / Z with
// Z = sum(max(0, a - q_hat)) + c * p_out: one dense pass per node, O(k * K) work for the k candidates, and the
// sums of that pass serve the draw as well (rowsample.h).  Bound by the vector units (fp32: 19 instructions an element,
// 5.1 TB/s) or the LDS (bfloat16).  Two fp32 trees of 1365 nodes, V = 151936, every node: 546 us as a pass for the
// tests, a sweep, a finish and two more launches, 330 so; the path of 64 binary16 trees <2,2,2>, V = 32000: 52 and 39.7.
#pragma once
#include "rowsample.h"

namespace tslt {

constexpr int kMaxTreeDepth = 16;
constexpr int kMaxBranch = 16;

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
  int32_t* node_state;    // [B, n_nodes] 0 sampled, 1 a child accepted, 2 row unusable
  int32_t* node_slot;     // [B, n_nodes] accepted child number or -1
  int32_t* node_token;    // [B, n_nodes] the node's output
  int32_t* node_status;   // [B, n_nodes]
  int all_nodes;
};

// (More than the kernels use: the size that callers have been told all along, so that a workspace kept from an
// earlier version and one sized by this one are the same.)
inline size_t tree_workspace_bytes(int64_t B, int64_t n_nodes, int64_t V, bool all_nodes) {
  const size_t n_seg = size_t(row_segments(V));
  const size_t tasks = all_nodes ? size_t(n_nodes) : 1;
  return align256(size_t(B) * n_nodes * 4) * 4 + align256(size_t(B) * 4) * 2 +
         align256(size_t(B) * tasks * (n_seg + 2) * 16) +
         align256(size_t(B) * tasks * n_seg * kSubChunks * sizeof(double));
}
inline void tree_carve_workspace(TreeParams& p, void* ws) {
  char* w = reinterpret_cast<char*>(ws);
  const size_t per = align256(size_t(p.B) * p.n_nodes * 4);
  p.node_state = reinterpret_cast<int32_t*>(w); w += per;
  p.node_slot = reinterpret_cast<int32_t*>(w); w += per;
  p.node_token = reinterpret_cast<int32_t*>(w); w += per;
  p.node_status = reinterpret_cast<int32_t*>(w);
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
// accepted the terms' table is used up.
// ---------------------------------------------------------------------------------------------
template <typename T, typename Terms>
__device__ __forceinline__ int tree_node(const TreeParams& p, int64_t b, int node, double* table, bool build, RowShared& sh,
                                         int& slot, int& token, int& st) {
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
  row_sweep<T, Terms>(w, table, build ? -1 : -2, sh);
  token = -1;
  st = 0;
  float my_ratio = NAN, my_beta = NAN;                              // NaN if the candidate is never tested
  if (wave_id() == 0) {
    RowState r;
    row_eval(w, r, sh);
    int accepted = -1;
    double part = -1.0;                                             // of the last rejection, whose update is still to be made
    if (!leaf) {
      int gone = -1;
      double gone_q = 0.0;
      if (r.ok) {
        for (int i = 0; i < k; ++i) {
          const int x = __builtin_amdgcn_readlane(my_cand, i);
          if (x < 0) continue;                                      // absent candidate
          if (part >= 0.0) {                                        // the candidate before was rejected
            row_update(w, r, part, gone, sh);
            r.removed += gone_q;
            const double rest = 1.0 - r.removed;
            r.qscale = p.wor ? (rest > 0.0 ? 1.0 / rest : 0.0) : 1.0;
          }
          const RowTest t = row_test(w, r, x, sh);
          if (!t.found) r.st |= 4;
          if (lane == i) { my_ratio = float(t.ratio); my_beta = float(t.shared); }   // Section 4.3's beta^(i)
          const double bound = t.ratio < 1.0 ? t.ratio : 1.0;
          const float u = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_u), i));
          if (t.found && double(u) < bound) { accepted = i; token = x; break; }
          part = t.part;
          // drawn without replacement: x leaves the urn and what is left is renormalised
          gone = p.wor && t.found ? x : -1;
          gone_q = gone >= 0 ? t.q_x : 0.0;
        }
      }
    }
    if (accepted < 0 && r.ok) row_locate(w, r, u_res, r.stages > 0 || part >= 0.0 ? row_correct(w, r, part, sh) : 0.0, sh);
    st = r.st;
    if (lane == 0) sh.cmd = accepted >= 0 ? accepted : (r.ok ? -1 : -2);
  }
  __syncthreads();
  slot = sh.cmd;
  if (threadIdx.x < k) {
    if (p.out_ratio) p.out_ratio[c0 + lane] = my_ratio;
    if (p.out_beta) p.out_beta[c0 + lane] = my_beta;
  }
  if (slot >= 0) return 1;
  const int state = slot == -1 ? 0 : 2;
  slot = -1;
  if (state == 0) {
    row_clear<T>(table);
    __syncthreads();
    if (wave_id() < kPickWaves) token = row_pick(w, table, sh);     // (nothing follows for the other waves)
  }
  return state;
}

// ---------------------------------------------------------------------------------------------
// Every node: one workgroup per node.
// ---------------------------------------------------------------------------------------------
template <typename T, typename Terms>
__global__ __launch_bounds__(kRowThreads, kShared) void tree_node_kernel(const TreeParams p) {
  __shared__ RowShared sh;
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  const int64_t b = blockIdx.x / p.n_nodes;
  const int node = int(blockIdx.x - b * p.n_nodes);
  int slot, token, st;
  const int state = tree_node<T, Terms>(p, b, node, reinterpret_cast<double*>(dyn_lds), true, sh, slot, token, st);
  if (threadIdx.x == 0) {
    const int64_t n = b * p.n_nodes + node;
    p.node_state[n] = state;
    p.node_slot[n] = slot;
    p.node_token[n] = token;
    p.node_status[n] = st;
    if (p.out_node_token) p.out_node_token[n] = token;
    if (p.out_node_slot) p.out_node_slot[n] = slot;
  }
}

// The new-sequence search, one wave per tree.
__global__ __launch_bounds__(64) void tree_walk_kernel(const TreeParams p) {
  const int64_t b = blockIdx.x;
  const int lane = threadIdx.x;
  int st = 0;
  for (int n = lane; n < p.n_nodes; n += 64) st |= p.node_status[b * p.n_nodes + n];
  st = wave_or_i32(st);
  if (lane == 0) {
    int node = 0, layer = 0, len = 0;
    int32_t* seq = p.out_seq + size_t(b) * (p.depth + 1);
    while (node < p.n_int && p.node_state[b * p.n_nodes + node] == 1) {
      const int child = tree_first_child(p, node, layer) + p.node_slot[b * p.n_nodes + node];
      seq[len++] = p.node_token[b * p.n_nodes + node];
      node = child;
      ++layer;
    }
    seq[len] = p.node_token[b * p.n_nodes + node];
    p.out_len[b] = len + 1;
    for (int i = len + 1; i <= p.depth; ++i) seq[i] = -1;
    if (p.status) p.status[b] = st;
  }
}

// ---------------------------------------------------------------------------------------------
// Only the verified path is wanted: one workgroup per tree walks from the root, running Algorithm 5 at each node
// it reaches, descending into the accepted child and drawing the output of the node it stops at, so that at most
// depth + 1 target rows are read per tree, each once.  Uniforms are indexed by node, so the result is the one the
// all-nodes kernel gives.
// ---------------------------------------------------------------------------------------------
template <typename T, typename Terms>
__global__ __launch_bounds__(kRowThreads) void tree_path_kernel(const TreeParams p) {
  __shared__ RowShared sh;
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  const int tid = threadIdx.x;
  const int64_t b = blockIdx.x;
  for (int i = tid; i < p.n_nodes - 1; i += kRowThreads) {
    if (p.out_ratio) p.out_ratio[size_t(b) * (p.n_nodes - 1) + i] = NAN;
    if (p.out_beta) p.out_beta[size_t(b) * (p.n_nodes - 1) + i] = NAN;
  }
  __syncthreads();
  int32_t* seq = p.out_seq + size_t(b) * (p.depth + 1);
  int node = 0, layer = 0, len = 0, st_all = 0, token = -1;
  for (;;) {
    int slot, st;
    const int state = tree_node<T, Terms>(p, b, node, reinterpret_cast<double*>(dyn_lds), node == 0, sh, slot, token, st);
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

template <typename T, typename Terms> hipError_t launch_verify_tree_with(const TreeParams& p, hipStream_t s) {
  if (!p.all_nodes) {
    hipLaunchKernelGGL((tree_path_kernel<T, Terms>), dim3(unsigned(p.B)), dim3(kRowThreads), Terms::kBytes, s, p);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((tree_node_kernel<T, Terms>), dim3(unsigned(p.B * p.n_nodes)), dim3(kRowThreads), Terms::kBytes, s, p);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(tree_walk_kernel, dim3(unsigned(p.B)), dim3(64), 0, s, p);
  return hipGetLastError();
}
template <typename T> hipError_t launch_verify_tree(const TreeParams& p, hipStream_t s) {
  if constexpr (ExpTab<T>::kHas) {
    if (exp_table_usable<T>(p.rT)) return launch_verify_tree_with<T, BitTerms<T>>(p, s);
  }
  return launch_verify_tree_with<T, PowTerms<T>>(p, s);
}

}  // namespace tslt
