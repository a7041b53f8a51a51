// Internal declarations shared by the translation units of libspectree (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#ifdef __HIPCC__
#include <hip/hip_bf16.h>
#endif
#include <stdint.h>

#include <algorithm>

#include "spec_tree.h"

namespace spec {

// ---------------------------------------------------------------------------------------------
// Launch plan of one tree-attention call: how the key range [0, prefix_len + N) of every
// (request, head) is cut into chunks (one workgroup each) and where the partial results live.
// ---------------------------------------------------------------------------------------------
struct AttnPlan {
  int chunk_keys;   // fixed chunks: keys per workgroup (multiple of 32)
  int n_splits;     // chunks covering max_prefix_len + N; balanced plan: partial slots per (request, head)
  int balanced_wgs; // > 0: balanced plan that aims at this many chunks (see balanced_deal), chunk_keys is 0
  bool contiguous;  // balanced plan as equal contiguous shares of all tiles (see contiguous_deal), few-query kernel only
  bool wide;        // bf16: the wide kernel runs the plan (several query tiles per K/V head, or k_new not laid out like q)
  int heads_per_wg; // wide kernel, whole key ranges: consecutive K/V heads of a request served by one workgroup
  bool m32;         // 5..8 query tiles, D = 128: the kernel of tree_attention_bf16_wide32.hip (four wavefronts of 32
                    // queries, two workgroups per compute unit) instead of the wide kernel's eight wavefronts of 16
  // Partials, addressed through partial_row(): [B][H][n_splits][N] rows under fixed chunks, [n_splits][B][H][N] under the
  // balanced deal, which sizes n_splits for one request holding all the tiles: a pair's slots are filled from 0, so the
  // slots in use are one compact piece of the workspace.
  size_t ws_o_off;  // float [rows][D]   un-normalised partial outputs
  size_t ws_ml_off; // float [rows][2]   running max (log2 domain) and partial sum
  size_t ws_bytes;
};

// Block table of a paged cache as the kernels take it (by value). table == nullptr: the cache is contiguous,
// [B, H_kv, S_cap, D]. Otherwise the cache is [n_blocks, H_kv, 2^log2_tokens, D] and the descriptor's
// kv_stride_b is the stride between blocks.
struct Pages {
  const int32_t* table;   // [B, max_blocks]
  int max_blocks;
  int log2_tokens;
  int n_blocks;
};
inline Pages no_pages() { return Pages{nullptr, 0, 0, 0}; }

// Rotary position embedding applied inside the fused append + attention call (cos == nullptr: none): the caller's
// float32 device tables [len, D/2]. Token i of request b sits at position prefix_len[b] + tree_depth[b, i].
struct Rope {
  const float* cos;
  const float* sin;
  int len;
};
inline Rope no_rope() { return Rope{nullptr, nullptr, 0}; }

int compute_units();   // of the current device
AttnPlan make_attn_plan(const spec_attn_desc_t& d, bool paged = false);

#define SPEC_SMALL_TILE_KEYS 32   // keys per wavefront tile of the few-query bf16 kernel (N <= 16)
#define SPEC_WIDE_TILE_KEYS 64    // keys per workgroup tile of the wide bf16 kernel (N > 16)

// Workgroups of a balanced launch: the chunks the deal aims at, or one per (request, virtual head) pair.
inline unsigned balanced_grid(const AttnPlan& p, int B, int virtual_heads) {
  const long pairs = (long)B * virtual_heads;
  return (unsigned)(pairs > p.balanced_wgs ? pairs : p.balanced_wgs);
}

// Query heads per key/value head, and how the bf16 kernels split them. Every query head of a group brings
// ceil(N / 16) 16-query MFMA tiles; a workgroup holds at most 8 tiles, i.e. `heads_per_wg` whole heads, so a
// (request, K/V head) pair is served by `n_qgroups` workgroups ("virtual heads" hv = h_kv * n_qgroups + qg),
// each streaming the pair's K/V for its own heads (the repeats are served by the caches).
struct QueryGroups {
  int group;          // query heads per K/V head
  int tiles_per_head; // ceil(N / 16)
  int heads_per_wg;   // query heads one workgroup serves
  int n_qgroups;      // workgroups per (request, K/V head) pair
  int tiles_per_wg;   // heads_per_wg * tiles_per_head, 1..8
};
inline QueryGroups attn_query_groups(const spec_attn_desc_t& d) {
  QueryGroups g;
  g.group = d.H / d.H_kv;
  g.tiles_per_head = (d.N + 15) / 16;
  const int fit = 8 / g.tiles_per_head > 0 ? 8 / g.tiles_per_head : 1;
  g.heads_per_wg = g.group < fit ? g.group : fit;
  g.n_qgroups = (g.group + g.heads_per_wg - 1) / g.heads_per_wg;
  g.tiles_per_wg = g.heads_per_wg * g.tiles_per_head;
  return g;
}

// float32 kernel: a workgroup serves one or two 16-query tiles of the group * N queries of a K/V head (more would not fit
// its registers beside a K/V tile), further tiles go to further workgroups.
inline int f32_query_tiles(const spec_attn_desc_t& d) { return (long)(d.H / d.H_kv) * d.N <= 16 ? 1 : 2; }
inline int f32_query_groups(const spec_attn_desc_t& d) {
  const int per_wg = 16 * f32_query_tiles(d);
  return (int)(((long)(d.H / d.H_kv) * d.N + per_wg - 1) / per_wg);
}

// Arithmetic of the balanced deal (see balanced_deal), shared by the kernels and by a host test.
// Tiles of a request; none if it does not fit the capacity.
__host__ __device__ inline int request_tiles(int P, int N, int S_cap, int tile) {
  return (P >= 0 && P <= S_cap - N) ? (P + N + tile - 1) / tile : 0;
}
// a / b for 0 <= a, 0 < b < 2^30 and a quotient below 2^22: the deal divides a dozen times in a row before a workgroup's first
// load, and an integer division is some thirty instructions on the vector unit. The reciprocal is good to 2^-22, so that the
// quotient is off by one at most, which the remainder shows.
__host__ __device__ inline int deal_quotient(int a, int b) {
#ifdef __HIP_DEVICE_COMPILE__
  const int q = (int)((float)a * __builtin_amdgcn_rcpf((float)b));
  const int rest = a - q * b;
  return q + (rest >= b) - (rest < 0);
#else
  return a / b;
#endif
}
// Chunks of a request with tb tiles: their number, and the tiles of each but the last.
__host__ __device__ inline int deal_chunks(int tb, int share) { return deal_quotient(tb + share - 1, share); }
__host__ __device__ inline int deal_chunk_tiles(int tb, int chunks) { return deal_quotient(tb + chunks - 1, chunks); }
// Number r of a request's chunks (over all virtual heads): its (K/V head, chunk) unit and its query group. The query groups
// of a unit read the same keys: whole blocks of eight units are numbered so that a unit's groups are eight apart, which puts
// them on one XCD; what is left over takes them in a row.
struct DealUnit { int unit, qg; };
__host__ __device__ inline DealUnit deal_unit(int r, int n_qg, int units) {
  if (n_qg == 1) return {r, 0};
  const int blk = deal_quotient(r, 8 * n_qg), rr = r - blk * 8 * n_qg;
  if ((blk + 1) * 8 <= units) return {blk * 8 + rr % 8, rr / 8};
  const int unit = deal_quotient(r, n_qg);
  return {unit, r - unit * n_qg};
}
// Whether the chunks of request i, of size_i tiles each, come before those of request j in descending order of size.
__host__ __device__ inline bool deal_before(int size_i, int i, int size_j, int j) {
  return size_i > size_j || (size_i == size_j && i < j);
}
// Place of workgroup id among the `count` chunks in descending order of size. A compute unit takes workgroups id and id + compute_units
// when two fit it, and they share its rate: the longest chunk goes with the shortest, the second longest with the second shortest and
// so on (32 requests x 64 / 8 heads of 900 to 4100 keys: 93.1 -> 89.9 us with the merge; the tiles of a compute unit were 28 to 52, are 38 to
// 41 now). With more chunks than fit at once the longest start first.
__host__ __device__ inline long deal_place(long id, long count, int compute_units) {
  return id < compute_units || count > 2l * compute_units ? id : count - 1 - (id - compute_units);
}

// Strides of k_new / v_new (all zero in the descriptor: laid out like q).
struct NewStrides { long b, n, h; };
inline NewStrides attn_new_strides(const spec_attn_desc_t& d) {
  if (d.new_stride_b == 0 && d.new_stride_n == 0 && d.new_stride_h == 0)
    return {(long)d.q_stride_b, (long)d.q_stride_n, (long)d.q_stride_h};
  return {(long)d.new_stride_b, (long)d.new_stride_n, (long)d.new_stride_h};
}

// Kernel launchers (defined in the .hip files). All return hipError_t of the launch.
hipError_t launch_kv_append(const spec_attn_desc_t& d, const Pages& pg, const void* k_new, const void* v_new,
                            void* k_cache, void* v_cache, const int32_t* prefix_len, int32_t* status, hipStream_t s);
hipError_t launch_kv_append_rope(const spec_attn_desc_t& d, const Pages& pg, const void* k_new, const void* v_new,
                                 void* k_cache, void* v_cache, const int32_t* tree_depth, const int32_t* prefix_len,
                                 const float* rope_cos, const float* rope_sin, int rope_len, int32_t* status,
                                 hipStream_t s, void* q = nullptr);
hipError_t launch_kv_commit(const spec_attn_desc_t& d, const Pages& pg, int n_layers, void* const* k_caches,
                            void* const* v_caches,
                            const int32_t* path, int Lmax, const int32_t* len, const int32_t* prefix_len,
                            int32_t* prefix_len_out, int32_t* status, hipStream_t s);
// k_new / v_new non-null (either dtype): the kernel also appends the tree rows to the cache (fused KV append).
hipError_t launch_tree_attention_f32(const spec_attn_desc_t& d, const AttnPlan& plan, const Pages& pg, const float* q,
                                     float* k_cache, float* v_cache, const float* k_new, const float* v_new,
                                     const int32_t* parent, const int32_t* depth, const int32_t* prefix_len, float* out,
                                     void* ws, int32_t* status, hipStream_t s);
// rope.cos non-null (with k_new / v_new): the queries (in registers) and the new K rows (before they are used and
// stored) are rotated by their positions' angles.
hipError_t launch_tree_attention_bf16(const spec_attn_desc_t& d, const AttnPlan& plan, const Pages& pg, const void* q, void* k_cache,
                                      void* v_cache, const void* k_new, const void* v_new, const int32_t* parent,
                                      const int32_t* depth, const int32_t* prefix_len, void* out, void* ws,
                                      int32_t* status, hipStream_t s, const Rope& rope = no_rope());
// Several query tiles per K/V head, or k_new / v_new not laid out like q: the workgroup's wavefronts split the queries and share the
// K/V stream through LDS.
hipError_t launch_tree_attention_bf16_wide(const spec_attn_desc_t& d, const AttnPlan& plan, const Pages& pg, const void* q, void* k_cache,
                                           void* v_cache, const void* k_new, const void* v_new, const int32_t* parent,
                                           const int32_t* depth, const int32_t* prefix_len, void* out, void* ws,
                                           int32_t* status, hipStream_t s, const Rope& rope = no_rope());
// Five to eight query tiles per K/V head, D = 128: 32-query MFMA tiles, K/V loaded straight into an LDS ring.
hipError_t launch_tree_attention_bf16_wide32(const spec_attn_desc_t& d, const AttnPlan& plan, const Pages& pg, const void* q,
                                             void* k_cache, void* v_cache, const void* k_new, const void* v_new,
                                             const int32_t* parent, const int32_t* depth, const int32_t* prefix_len,
                                             void* out, void* ws, int32_t* status, hipStream_t s,
                                             const Rope& rope = no_rope());
hipError_t launch_attn_combine(const spec_attn_desc_t& d, const AttnPlan& plan, const int32_t* prefix_len, const void* ws,
                               void* out, int32_t* status, hipStream_t s);
hipError_t launch_expand_topk(int B, int F, int V, int logits_dtype, const void* logits, int k, const int32_t* child_slot,
                              int N, int32_t* tree_token, int32_t* status, hipStream_t s);
hipError_t launch_tree_merge(int B, int M, int Nin, const int32_t* in_parent, const int32_t* in_token,
                             const int32_t* in_size, int Nout, int32_t* out_parent, int32_t* out_depth,
                             int32_t* out_token, int32_t* out_ssm, int32_t* out_size, int32_t* node_map, int32_t* status,
                             hipStream_t s);
// LM head + arg-max (lm_head.hip). Workspace: per row one (max, arg-max) pair per vocabulary tile.
#define SPEC_LM_HEAD_VOCAB_TILE 64   // the smaller of the two workgroup shapes: sizes the partials
inline size_t lm_head_partials_bytes(int M, int V) {
  const size_t n_vtiles = ((size_t)V + SPEC_LM_HEAD_VOCAB_TILE - 1) / SPEC_LM_HEAD_VOCAB_TILE;
  return 2 * (((size_t)M * n_vtiles * 4 + 255) / 256 * 256);
}
hipError_t launch_lm_head_argmax(int M, int K, int V, const void* hidden, const void* weight, int32_t* node_argmax,
                                 float* node_max, void* ws, hipStream_t s);
// The same pass over the weights that also writes bf16 logits and their softmax statistics; the workspace holds
// three partial arrays (lm_head_partials_bytes(M, V) / 2 each).
hipError_t launch_lm_head(int M, int K, int V, const void* hidden, const void* weight, void* logits_out, float inv_temp,
                          int32_t* node_argmax, float* node_max, float* node_sumexp, void* ws, hipStream_t s);
hipError_t launch_node_stats(int B, int N, int V, int logits_dtype, const void* logits, float inv_temp,
                             int32_t* node_argmax, float* node_max, float* node_sumexp, hipStream_t s,
                             const int32_t* parent = nullptr, int own_levels = 0);
hipError_t launch_node_sample(int B, int N, int V, int logits_dtype, const void* logits, float inv_temp,
                              const float* node_max, const float* u_sample, int32_t* node_sample, hipStream_t s);
hipError_t launch_greedy_walk(int B, int N, const int32_t* node_argmax, const int32_t* token, const int32_t* parent,
                              int Lmax, int32_t* path, int32_t* len, int32_t* out_tokens, int32_t* status,
                              hipStream_t s);
// Vocabularies whose distribution the stochastic walk keeps in its workgroup's registers: 32 floats per thread. With 64 the
// kernel spills and the buffer form is the faster one (8 trees of 16, 50000 float32: 67 us against 59).
inline bool stochastic_walk_in_registers(int V) { return V <= 32768; }
// Levels up to which a tree's nodes get their statistics from the walk itself (0: none); those of deeper trees come from the
// pass over all nodes. A walk visits at most as many nodes as its tree has levels, and each node costs it about 1e-4 V us more
// than a walk over given statistics (96 accepted nodes in a row, us, own / given: 8192 float32 144 / 58, 16384: 220 / 59, 32000:
// 350 / 61, 32003: 358 / 66; 32000 bfloat16 296 / 61, 31999: 362 / 68; 0.5 us more at least, 2048: 112 / 58); the pass costs its
// bytes at 5.5 TB/s and a launch. The line is drawn at 0.9e-4 V, a little past the level where the two are equal, as the usual path has a few
// nodes and not all its levels: 16 x 128 nodes of 32000 float32, 16 levels, three drafts, 44.6 us, and a path accepted to the end of such
// a tree 5 us more than behind a pass (10 us more at worst: 33 levels of 2048). All 128 nodes of chains accepted: 130 us
// (96 of them 100, 350 by their own statistics). Looking at the trees makes a pass 2 us longer, and one that leaves them all out
// takes 4.5: only from 8 levels on, which fewer trees of a batch exceed. Where Lmax or N are no more than the levels, no tree
// has to be looked at.
inline int stochastic_own_levels(int B, int N, int V, int logits_dtype, int Lmax) {
  if (!stochastic_walk_in_registers(V)) return 0;
  const double pass_us = (double)B * N * V * (logits_dtype == SPEC_BF16 ? 2 : 4) / 5.5e6;
  const double node_us = V * 0.9e-4;
  const int levels = (int)std::min(pass_us / node_us, (double)SPEC_MAX_TREE_NODES);
  return levels >= 8 || levels >= std::min(Lmax, N) ? levels : 0;
}
hipError_t launch_stochastic_walk(int B, int N, int V, int logits_dtype, const void* logits, const float* probs_ssm,
                                  int R, const int32_t* ssm_row, const int32_t* token, const int32_t* parent,
                                  const float* u_accept, const float* u_order, const float* u_final, float inv_temp,
                                  const float* node_max, const float* node_sumexp, float* resid, int Lmax,
                                  int32_t* path, int32_t* len, int32_t* out_tokens, int32_t* status, hipStream_t s,
                                  int own_levels = 0);

// ---------------------------------------------------------------------------------------------
// Device helpers
// ---------------------------------------------------------------------------------------------
#ifdef __HIPCC__

// Row of node 0 of a (request, head) pair's slot in the partials.
template <bool BALANCED>
__device__ __forceinline__ long partial_row(int b, int h, int slot, int B, int H, int N, int n_splits) {
  return BALANCED ? (((long)slot * B + b) * H + h) * N : (((long)b * H + h) * n_splits + slot) * N;
}

// What a partial says of itself, so that the merge needs neither the tree nor the deal: the sum of the chunk that ends its request
// carries a sign (sums have none), which tells how many slots are filled, and a maximum of NaN (never a maximum: fmaxf drops NaN)
// stands for a row with nothing to merge, whose "sum" says why.
constexpr float PARTIAL_BAD_TREE = -0.f, PARTIAL_FINAL = -1.f;   // malformed tree; the only chunk, whose workgroup wrote the output
__device__ __forceinline__ float partial_sum(float l, bool last) { return __builtin_copysignf(l, last ? -1.f : 1.f); }
__device__ __forceinline__ bool partial_ends(float m, float l) { return m != m || (__float_as_int(l) < 0); }
__device__ __forceinline__ void mark_partial(float* __restrict__ ws_ml, long row, float why) {
  ws_ml[row * 2 + 0] = __int_as_float(0x7fc00000);
  ws_ml[row * 2 + 1] = why;
}

// A workgroup-uniform value back in a scalar register. The compiler divides on the vector unit and leaves the quotient
// there, and with it every address and loop bound derived from it: the balanced launches lost 8 to 15 us of 100 to that.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
// a / b of workgroup-uniform numbers; without the division, which stands before a kernel's first load, where b is 1
__device__ __forceinline__ int uniform_div(int a, int b) { return b == 1 ? a : uniform(a / b); }

// Checks one request's parents with the threads of a workgroup (blockDim.x >= N): true for every thread iff parent[0] == -1 and
// 0 <= parent[i] < i. `flag` is one int of LDS. Contains two __syncthreads().
__device__ inline bool tree_is_valid(const int32_t* __restrict__ parent, int N, int* flag) {
  const int t = threadIdx.x;
  if (t == 0) *flag = 0;
  __syncthreads();
  if (t < N) {
    const int p = parent[t];
    const bool ok = t == 0 ? p == -1 : p >= 0 && p < t;
    if (!ok) atomicOr(flag, 1);
  }
  __syncthreads();
  return *flag == 0;
}

// A tree's ancestor-or-self masks, from the parents and depths in LDS. A lane has a node; its mask and the node after it reach
// twice as far up after every exchange within the wavefront: two or three exchanges for the usual tree, where a walk up the
// parent chain is a dependent LDS read per level, after two barriers more (chains of 64 and 128
// nodes: 32 heads of 1024 keys 19.6 -> 15.9 us, 16 requests of 512 keys 53.9 -> 45.0; random trees of 24 11.4 -> 11.2).
struct TreeLds {
  unsigned long long anc[SPEC_MAX_TREE_NODES][2];
  int parent[SPEC_MAX_TREE_NODES], depth[SPEC_MAX_TREE_NODES], up[SPEC_MAX_TREE_NODES];
  int bad[2];
};
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
// By one whole wavefront, with nodes `lane` and (above 64 nodes) `lane + 64`; returns, to all its lanes, whether the tree is
// malformed (the masks then mean nothing).
template <int NODES>   // per lane
__device__ __forceinline__ bool tree_masks_of(TreeLds& s, int N, int lane, int par0, int dep0) {
  unsigned long long lo[NODES], hi[NODES];
  int up[NODES];
  bool ok = true;
#pragma unroll
  for (int i = 0; i < NODES; ++i) {
    const int v = lane + 64 * i;
    up[i] = -1;
    lo[i] = i == 0 ? 1ull << lane : 0ull;
    hi[i] = i == 0 ? 0ull : 1ull << lane;
    if (v < N) {
      const int p = i == 0 ? par0 : s.parent[v], d = i == 0 ? dep0 : s.depth[v], q = min(max(p, 0), N - 1);
      ok = ok && (v == 0 ? p == -1 && d == 0 : p >= 0 && p < v && d == s.depth[q] + 1);
      if (p >= 0) {
        if (q < 64) lo[i] |= 1ull << q; else hi[i] |= 1ull << (q - 64);
        up[i] = s.parent[q];
      }
    }
  }
  if (__any(!ok)) return true;
  bool more = __any(up[0] >= 0 || up[NODES - 1] >= 0);
  while (true) {
#pragma unroll
    for (int i = 0; i < NODES; ++i)
      if (lane + 64 * i < N) {
        s.anc[lane + 64 * i][0] = lo[i];
        s.anc[lane + 64 * i][1] = hi[i];
        if (more) s.up[lane + 64 * i] = up[i];
      }
    if (!more) return false;
    wave_lds_fence();
    int next[NODES];
#pragma unroll
    for (int i = 0; i < NODES; ++i) {
      next[i] = -1;
      if (up[i] >= 0) {
        lo[i] |= s.anc[up[i]][0];
        if (NODES > 1) hi[i] |= s.anc[up[i]][1];
        next[i] = s.up[up[i]];
      }
    }
    wave_lds_fence();
#pragma unroll
    for (int i = 0; i < NODES; ++i) up[i] = next[i];
    more = __any(up[0] >= 0 || up[NODES - 1] >= 0);
  }
}
__device__ __forceinline__ bool tree_masks_by_wave(TreeLds& s, int N, int lane, int par0, int dep0) {   // par0, dep0: of node `lane`
  return N <= 64 ? tree_masks_of<1>(s, N, lane, par0, dep0) : tree_masks_of<2>(s, N, lane, par0, dep0);
}
// By two wavefronts, of which `half` has nodes 64 half and up: each follows its nodes' ancestors within its half, and `up` ends as
// the first one below it, whose mask is the rest. Above 64 nodes that is one node per lane instead of two (us, one wavefront /
// two: 32 heads of 1000 keys, trees of 128, 22.0 / 21.5, chains 22.7 / 21.7; 3 x 64 heads of 150 keys 18.1 / 17.7, chains 18.8 /
// 17.8; 16 x 32 of 512, 43.9 / 43.7). Not in the kernel for fewer queries, where nothing but D = 64 has as many nodes and the
// longer code costs trees of up to 64 about 1 % (32 heads of 1024 keys, trees of 64, 15.6 / 15.8).
__device__ __forceinline__ bool tree_masks_of_half(TreeLds& s, int N, int half, int lane, int par, int dep) {
  const int base = 64 * half, v = base + lane;
  unsigned long long own = 1ull << lane;
  int up = -1;
  bool ok = true;
  if (v < N) {
    const int q = min(max(par, 0), N - 1);
    ok = v == 0 ? par == -1 && dep == 0 : par >= 0 && par < v && dep == s.depth[q] + 1;
    up = par;
    if (par >= base) {
      own |= 1ull << (q - base);
      up = s.parent[q];
    }
  }
  if (__any(!ok)) return true;
  while (true) {
    if (v < N) {
      s.anc[v][half] = own;
      s.up[v] = up;
    }
    if (!__any(up >= base)) return false;
    wave_lds_fence();
    int next = up;
    if (up >= base) {
      own |= s.anc[up][half];
      next = s.up[up];
    }
    wave_lds_fence();
    up = next;
  }
}
// Called by every thread, behind a barrier after the words were stored; false: malformed, with nothing left to wait for.
template <class Barrier>
__device__ __forceinline__ bool tree_masks_by_two_waves(TreeLds& s, int N, int wave, int lane, int par, int dep, Barrier&& barrier) {
  if (wave < 2) {
    const bool bad = tree_masks_of_half(s, N, wave, lane, par, dep);
    if (lane == 0) s.bad[wave] = bad;
    if (wave == 0) s.anc[lane][1] = 0;
  }
  barrier();
  if (s.bad[0] | s.bad[1]) return false;
  if (N > 64) {
    if (wave == 1 && lane + 64 < N) s.anc[lane + 64][0] = s.anc[s.up[lane + 64]][0];
    barrier();
  }
  return true;
}

// Balanced plan: every (request, head) pair's key tiles (`tile` keys each) are cut into equal chunks of at most `share`
// tiles, as many for each request as its length asks for, and workgroup id has chunk number id. `share` is (nearly) the
// smallest for which the chunks of all pairs are at most n_wg (or one per pair, if there are more pairs; the grid has room
// for either, see balanced_grid()). A workgroup has one chunk of one pair: a share that crossed from one pair into the next would pay a second prologue and
// epilogue (measured against a deal of equal contiguous shares over the same 512 workgroups, which also spilled registers in its
// loop over segments: 32 requests x 64 / 8 heads, 900-4100 keys: 123 -> 103 us; 4 x 32 heads, 8192-16384: 147 -> 139 us). A request that does not fit
// the cache capacity has no tiles.
//
// All functions read prefix_len[] with the 64 lanes of a wavefront at once, as a workgroup has its first key only behind them (a
// scalar walk is one dependent load per request: 40 us for 32 requests). Every lane must be active; results are uniform.
// a / b of non-negative numbers, in 32 bits where they fit (a 64-bit division is some hundred instructions)
__device__ inline long deal_div(long a, long b) {
  return ((a | b) >> 30) == 0 && (a >> 21) < b ? (long)deal_quotient((int)a, (int)b) : a / b;
}
// Inclusive sum over the lanes of a wavefront (lane 63 holds the total), in register moves: row shifts, then the last lane
// of each row of 16 into the rows after it.
__device__ inline int wave_inclusive_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return v;
}
__device__ inline int wave_sum_uniform(int v) { return __builtin_amdgcn_readlane(wave_inclusive_sum(v), 63); }

struct BalancedDeal {
  int share;    // most tiles of a chunk (>= 1)
  long count;   // chunks over all requests and heads
};
__device__ inline BalancedDeal balanced_deal(const int32_t* __restrict__ prefix_len, int B, int N, int H, int S_cap, int tile,
                                             int n_wg) {
  const int lane = threadIdx.x & 63;
  const int first = lane < B ? request_tiles(prefix_len[lane], N, S_cap, tile) : 0;
  auto tiles_of = [&](int b0) {
    return b0 == 0 ? first : b0 + lane < B ? request_tiles(prefix_len[b0 + lane], N, S_cap, tile) : 0;
  };
  long tiles = 0, pairs = 0;
  for (int b0 = 0; b0 < B; b0 += 64) {
    const int v = tiles_of(b0);
    tiles += wave_sum_uniform(v);
    pairs += __popcll(__ballot(v > 0));
  }
  pairs *= H;
  const long cap = max((long)n_wg, pairs);
  long share = max(1l, deal_div(tiles * H + cap - 1, cap));
  BalancedDeal d;
  for (int i = 0;; ++i) {   // the share grows by the factor that is missing, from below; the last step always fits
    if (i == 12) share = 0x3fffffff;
    d.share = (int)min(share, 0x3fffffffl);
    d.count = 0;
    for (int b0 = 0; b0 < B; b0 += 64) {
      const int v = tiles_of(b0);
      d.count += wave_sum_uniform(deal_chunks(v, d.share));
    }
    d.count *= H;
    if (d.count <= cap || i == 12) return d;
    share = max(share + 1, deal_div(share * d.count, cap));
  }
}
// Chunk `id` (< count) of the deal: request, head, tiles [tile0, tile0 + n_tiles) (none if rounding leaves the request
// fewer chunks than it was counted with) and the request's chunks per head. `sorted` (B <= 64): chunk number `id` where the requests
// stand in descending order of their chunks' sizes.
struct DealChunk {
  int b, h, chunk, tile0, n_tiles, chunks;
};
__device__ inline DealChunk deal_find(const int32_t* __restrict__ prefix_len, int B, int N, int H, int n_qg, int S_cap,
                                      int tile, const BalancedDeal& d, long id, bool sorted = false) {
  const int lane = threadIdx.x & 63;
  DealChunk c = {0, 0, 0, 0, 0, 1};
  long acc = 0;   // chunks per head over the requests below b0
  for (int b0 = 0; b0 < B; b0 += 64) {
    const int tb_lane = b0 + lane < B ? request_tiles(prefix_len[b0 + lane], N, S_cap, tile) : 0;
    const int v = deal_chunks(tb_lane, d.share);
    int incl;   // chunks per head of the requests up to this lane's
    const int size = sorted && v > 0 ? deal_chunk_tiles(tb_lane, v) : 0;
    const int some_size = __builtin_amdgcn_readlane(size, __ffsll((long long)__ballot(v > 0)) - 1);   // (id < count: some lane has chunks)
    // Equal sizes stand in their order already: the loop of 16 to 32 requests takes 1 us, in front of the first key (us, with it always /
    // where sizes differ: 16 x 32 / 8 heads of 9000 keys, trees of 16, 110.1 / 109.1; 32 x 32 / 8 of 4200, 10, 99.4 / 97.5).
    if (sorted && __any(v > 0 && size != some_size)) {
      incl = v;
      for (int i = 0; i < B; ++i) {
        const int s_i = __builtin_amdgcn_readlane(size, i), v_i = __builtin_amdgcn_readlane(v, i);
        incl += deal_before(s_i, i, size, lane) ? v_i : 0;
      }
    } else {
      incl = wave_inclusive_sum(v);
    }
    const unsigned long long hit = __ballot((acc + incl) * H > id && (!sorted || (long)(incl - v) * H <= id));
    if (hit != 0) {
      const int f = __ffsll((long long)hit) - 1;
      const int tb = __builtin_amdgcn_readlane(tb_lane, f);
      c.chunks = __builtin_amdgcn_readlane(v, f);
      c.b = b0 + f;
      const int r = (int)(id - (acc + __builtin_amdgcn_readlane(incl, f) - c.chunks) * H);   // < H * chunks
      const DealUnit u = deal_unit(r, n_qg, deal_quotient(H, n_qg) * c.chunks);
      const int kv_head = deal_quotient(u.unit, c.chunks);
      c.chunk = u.unit - kv_head * c.chunks;
      c.h = kv_head * n_qg + u.qg;
      const int per = deal_chunk_tiles(tb, c.chunks);
      c.tile0 = c.chunk * per;
      c.n_tiles = max(0, min(per, tb - c.tile0));
      return {c.b, uniform(c.h), uniform(c.chunk), uniform(c.tile0), uniform(c.n_tiles), c.chunks};
    }
    acc += __builtin_amdgcn_readlane(incl, 63);
  }
  return c;
}

// Contiguous form of the balanced plan: the key tiles of all pairs, ordered by (request, head, key), are dealt to n_wg
// workgroups in equal contiguous shares; a share that crosses from one pair into the next is two segments in a row. For the
// few-query kernel, which runs one workgroup per compute unit, where there are fewer than two chunks per pair: whole
// fractions of a pair would leave compute units idle (6 requests x 32 heads x 64 of 4500 keys, 192 pairs on 256 compute
// units: 45.6 us, 51.3 in halves).
struct ContiguousDeal {
  long total;   // tiles over all requests and heads
  long share;   // tiles per workgroup (>= 1)
};
__device__ inline ContiguousDeal contiguous_deal(const int32_t* __restrict__ prefix_len, int B, int N, int H, int S_cap,
                                                 int tile, int n_wg) {
  const int lane = threadIdx.x & 63;
  long tiles = 0;
  for (int b0 = 0; b0 < B; b0 += 64) {
    const int v = b0 + lane < B ? request_tiles(prefix_len[b0 + lane], N, S_cap, tile) : 0;
    tiles += wave_sum_uniform(v);
  }
  ContiguousDeal r;
  r.total = tiles * H;
  r.share = max(1l, deal_div(r.total + n_wg - 1, n_wg));
  return r;
}
// The request that holds tile `pos` (< total) of the contiguous deal: its index, first tile and tiles per head.
struct DealRequest {
  int b;
  long start;
  int tiles;
};
__device__ inline DealRequest contiguous_find(const int32_t* __restrict__ prefix_len, int B, int N, int H, int S_cap, int tile,
                                              long pos) {
  const int lane = threadIdx.x & 63;
  long acc = 0;   // tiles per head over the requests below b0
  for (int b0 = 0; b0 < B; b0 += 64) {
    const int v = b0 + lane < B ? request_tiles(prefix_len[b0 + lane], N, S_cap, tile) : 0;
    const int incl = wave_inclusive_sum(v);
    const unsigned long long hit = __ballot((acc + incl) * H > pos);
    if (hit != 0) {
      const int f = __ffsll((long long)hit) - 1;
      const int tb = __builtin_amdgcn_readlane(v, f);
      return {b0 + f, (acc + __builtin_amdgcn_readlane(incl, f) - tb) * H, tb};
    }
    acc += __builtin_amdgcn_readlane(incl, 63);
  }
  return {0, 0, 1};   // not reached for pos < total
}

// Rotation of the two 16-byte pieces of a row that pair up under the half-split rotary embedding (piece `lo`
// holds dimensions c .. c + EPV, `hi` the same dimensions + D/2), by the angles whose cosines / sines are cs / sn.
// float32 arithmetic in one fixed order (product, then fused multiply-add: the product is kept out of the
// compiler's contraction so that every kernel that rotates a row produces the same bits), rounded to the storage
// type.
template <bool BF16>
__device__ __forceinline__ void rope_pair(const uint4 lo, const uint4 hi, const float* __restrict__ cs,
                                          const float* __restrict__ sn, uint4* olo, uint4* ohi) {
  constexpr int EPV = BF16 ? 8 : 4;   // elements per 16-byte piece
  float x1[EPV], x2[EPV];
  if (BF16) {
    const unsigned a[4] = {lo.x, lo.y, lo.z, lo.w}, bb[4] = {hi.x, hi.y, hi.z, hi.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      x1[2 * j] = __uint_as_float(a[j] << 16);
      x1[2 * j + 1] = __uint_as_float(a[j] & 0xffff0000u);
      x2[2 * j] = __uint_as_float(bb[j] << 16);
      x2[2 * j + 1] = __uint_as_float(bb[j] & 0xffff0000u);
    }
  } else {
    x1[0] = __uint_as_float(lo.x); x1[1] = __uint_as_float(lo.y); x1[2] = __uint_as_float(lo.z); x1[3] = __uint_as_float(lo.w);
    x2[0] = __uint_as_float(hi.x); x2[1] = __uint_as_float(hi.y); x2[2] = __uint_as_float(hi.z); x2[3] = __uint_as_float(hi.w);
  }
  float y1[EPV], y2[EPV];
#pragma unroll
  for (int j = 0; j < EPV; ++j) {
    const float co = cs[j], si = sn[j];
    float p1 = x2[j] * si, p2 = x1[j] * si;
    asm("" : "+v"(p1), "+v"(p2));
    y1[j] = fmaf(x1[j], co, -p1);
    y2[j] = fmaf(x2[j], co, p2);
  }
  if (BF16) {
    unsigned o1[4], o2[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      union { __hip_bfloat16 h; unsigned short u; } a0, a1, b0, b1;
      a0.h = __float2bfloat16(y1[2 * j]); a1.h = __float2bfloat16(y1[2 * j + 1]);
      b0.h = __float2bfloat16(y2[2 * j]); b1.h = __float2bfloat16(y2[2 * j + 1]);
      o1[j] = (unsigned)a0.u | ((unsigned)a1.u << 16);
      o2[j] = (unsigned)b0.u | ((unsigned)b1.u << 16);
    }
    *olo = make_uint4(o1[0], o1[1], o1[2], o1[3]);
    *ohi = make_uint4(o2[0], o2[1], o2[2], o2[3]);
  } else {
    *olo = make_uint4(__float_as_uint(y1[0]), __float_as_uint(y1[1]), __float_as_uint(y1[2]), __float_as_uint(y1[3]));
    *ohi = make_uint4(__float_as_uint(y2[0]), __float_as_uint(y2[1]), __float_as_uint(y2[2]), __float_as_uint(y2[3]));
  }
}

__device__ inline void set_status(int32_t* status, int b, int bit) {
  if (status != nullptr) atomicOr(&status[b], bit);
}

// Offset, in the units of the two strides, of logical cache row `row` of request b before the head and
// column terms. Paged: `ok` tells whether the table entry lies inside the pool; an entry outside is
// replaced by one inside (block 0 or the last), so the offset always stays within the cache.
__device__ inline long cache_row_offset(const Pages& pg, int b, int row, long kv_sb, long kv_ss, bool* ok) {
  *ok = true;
  if (pg.table == nullptr) return b * kv_sb + (long)row * kv_ss;
  const int e = pg.table[(long)b * pg.max_blocks + (row >> pg.log2_tokens)];
  *ok = e >= 0 && e < pg.n_blocks;
  const int blk = min(max(e, 0), pg.n_blocks - 1);
  return blk * kv_sb + (long)(row & ((1 << pg.log2_tokens) - 1)) * kv_ss;
}

// The block numbers of a paged request in the lanes of a wavefront: lane i has logical block first + i. A tile's block then
// costs a register move, where an entry read from the table for every tile is a scalar load and a wait for it in front of the
// tile's requests (us, before / now: 24 requests x 32 / 8 heads of 900 to 3100 keys, trees of 30, 83.2 / 68.8; 8 x 32 heads of 1000
// keys, trees of 60, 37.9 / 32.3, of 24, 29.1 / 25.1; 10 x 40 heads of 1614 keys, D = 64, one node, 35.6 / 31.2).
struct BlockLanes {
  int first;                // of lane 0
  int block;                // this lane's, moved into the pool
  unsigned long long bad;   // lanes whose entry lies outside the pool (they may lie past the request's end and hold anything)
};
__device__ __forceinline__ BlockLanes block_lanes_of(const Pages& pg, int first, int entry) {
  return {first, min(max(entry, 0), pg.n_blocks - 1), __ballot(entry < 0 || entry >= pg.n_blocks)};
}
__device__ __forceinline__ const int32_t* block_entry(const Pages& pg, int b, int j) {
  return pg.table + (long)b * pg.max_blocks + min(j, pg.max_blocks - 1);
}
__device__ __forceinline__ BlockLanes load_block_lanes(const Pages& pg, int b, int first) {
  return block_lanes_of(pg, first, *block_entry(pg, b, first + (int)(threadIdx.x & 63)));
}
// Place of logical block j (wave-uniform) among the lanes, which move on when it is not among them: once in 64 blocks, so the
// wait for it stands here and not, for every tile, where the compiler would put it.
__device__ __forceinline__ int block_lane(BlockLanes& w, const Pages& pg, int b, int j) {
  if ((unsigned)(j - w.first) >= 64u) {
    int entry;
    asm volatile("global_load_dword %0, %1, off\n\ts_waitcnt vmcnt(0)"
                 : "=v"(entry) : "v"(block_entry(pg, b, j + (int)(threadIdx.x & 63))) : "memory");
    w = block_lanes_of(pg, j, entry);
  }
  return j - w.first;
}
// Whether one of the lanes' blocks up to `last` lies outside the pool.
__device__ __forceinline__ bool blocks_outside(const BlockLanes& w, int last) {
  return last >= w.first && (w.bad & (~0ull >> (63 - min(last - w.first, 63)))) != 0;
}

#endif  // __HIPCC__

}  // namespace spec
