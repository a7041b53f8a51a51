// Token-tree construction on the GPU (Section 3), the step right before verification, so that the
// speculated tree never visits the host:
//   expand_topk_kernel   one step of expansion-based construction: the k most likely next tokens of every
//                        frontier node (most likely first, ties to the lowest token id), written to the
//                        tree's token array at the slots the static expansion configuration assigns.
//   tree_merge_kernel    token tree merge (Definition 3.2): the M trees of a request become one tree that
//                        holds exactly their token sequences, numbered depth-first.
// Both are small integer / comparison kernels: one workgroup per row or per request.
#include <hip/hip_bf16.h>

#include "spec_internal.h"

namespace spec {

constexpr int TOPK_THREADS = 1024;
static_assert(SPEC_MAX_TOPK <= TOPK_THREADS, "a thread per pick");
constexpr int TOPK_U = 8;        // groups a thread requests before it uses any

// ---------------------------------------------------------------------------------------------
// top-k of one row of V logits in one pass over it. An element is a 64-bit key, (value, then lower token id) in one
// unsigned order, 0 for NaN; thread t owns the groups of VEC elements t, t + 1024, ... and keeps its largest key. A pick is
// the largest of the 16 wavefronts' largest keys; only the wavefront that held it goes on to its next: its 64 lanes read
// the winning thread's elements again (a few hundred bytes, from the cache) and reduce what comes after the pick.
//
// What bounds it: one workgroup's latency, a launch, one trip to memory for 16 bytes x 8 per thread and two reductions. Eight
// steps of 16 to 48 rows of 32000 float32 and the merge behind them: 58.6 us with a key and a 64-bit comparison per element,
// 49.6 with one comparison per group, 44.9 to 46.7 over the machines seen with reductions in register moves (exchanges through LDS
// before) and the slots requested with the row (as nodes of a graph 53.0 -> 46.4); 11 to 33 rows of 93776: 93 and 71 with the first two.
// VEC: 16 bytes of elements, from whatever element a row starts at; the last group ends with the row, and what it shares
// with the group before it counts there (2 rows of 22115 float32: 6.1 us by single elements, 5.5). Rows of less: one.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ unsigned long long topk_key(float x, int i) {
  if (x != x) return 0;
  const unsigned u = __float_as_uint(x + 0.f);   // (-0 and +0 are equal: the lower id comes first)
  const unsigned ord = u ^ ((unsigned)((int)u >> 31) | 0x80000000u);
  return ((unsigned long long)ord << 32) | (unsigned)~i;
}
// Largest key of a wavefront (LANES 64) or of its first 16 lanes, in register moves: row shifts, then the last lane of each row of
// 16 into the rows after it (0 where there is no source, which is no key). Every lane must be active; the result is uniform.
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long max_moved(unsigned long long k) {
  const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)k, CTRL, ROWS, 0xf, false);
  const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(k >> 32), CTRL, ROWS, 0xf, false);
  const unsigned long long v = ((unsigned long long)hi << 32) | lo;
  return v > k ? v : k;
}
template <int LANES>
__device__ __forceinline__ unsigned long long wave_max_key(unsigned long long k) {
  k = max_moved<0x111, 0xf>(k);   // row_shr:1, 2, 4, 8
  k = max_moved<0x112, 0xf>(k);
  k = max_moved<0x114, 0xf>(k);
  k = max_moved<0x118, 0xf>(k);
  if (LANES == 64) {
    k = max_moved<0x142, 0xa>(k);   // row_bcast:15 into rows 1 and 3
    k = max_moved<0x143, 0xc>(k);   // row_bcast:31 into rows 2 and 3
  }
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)k, LANES - 1), hi = __builtin_amdgcn_readlane((unsigned)(k >> 32), LANES - 1);
  return ((unsigned long long)hi << 32) | lo;
}

template <bool BF16, int VEC, bool ODD>   // ODD: V is no multiple of VEC, or the rows are not 16-byte aligned
__global__ void __launch_bounds__(TOPK_THREADS) expand_topk_kernel(const void* __restrict__ logits, int F, int V, int k,
                                                                   const int32_t* __restrict__ child_slot, int N,
                                                                   int32_t* __restrict__ tree_token, int32_t* status) {
  __shared__ unsigned long long s_best[2][TOPK_THREADS / 64];   // by parity of the round: one barrier a round
  const int row = blockIdx.x, b = row / F, f = row % F, t = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
  const long base = (long)row * V;
  // the slots first, one per thread: asked for at the pick they were a trip to memory of their own at the end of the launch
  const int my_slot = t < k ? child_slot[(long)f * k + t] : 0;
  const int n_groups = (V + VEC - 1) / VEC;
  auto start = [&](int group) { return ODD ? min(group * VEC, V - VEC) : group * VEC; };
  typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  typedef u32x4 __attribute__((aligned(2))) u32x4_any;
  typedef f32x4 __attribute__((aligned(4))) f32x4_any;
  auto load = [&](int group, float (&x)[VEC]) {
    if constexpr (BF16) {
      const __hip_bfloat16* p = (const __hip_bfloat16*)logits + base + start(group);
      if constexpr (VEC == 1) {
        x[0] = __bfloat162float(*p);
      } else {
        const u32x4 raw = *(const u32x4_any*)p;
        const unsigned w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int e = 0; e < VEC / 2; ++e) {
          x[2 * e] = __uint_as_float(w[e] << 16);
          x[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
        }
      }
    } else {
      const float* p = (const float*)logits + base + start(group);
      if constexpr (VEC == 1) {
        x[0] = *p;
      } else {
        const f32x4 raw = *(const f32x4_any*)p;
        x[0] = raw.x; x[1] = raw.y; x[2] = raw.z; x[3] = raw.w;
      }
    }
  };
  auto key_of = [&](const float (&x)[VEC], int group, int e) {   // 0: the element belongs to the group before
    const int i = start(group) + e;
    return !ODD || i >= group * VEC ? topk_key(x[e], i) : 0ull;
  };
  // The thread's largest: a group costs its maximum, one comparison and the selection of the group; keys are made for the
  // elements of one group at the end (a key and a 64-bit comparison per element were 2 us of arithmetic a row of 32000).
  float best_value = -INFINITY, best_x[VEC];
  int best_group = -1;
  for (int g0 = t; g0 < n_groups; g0 += TOPK_THREADS * TOPK_U) {
    float x[TOPK_U][VEC];
#pragma unroll
    for (int j = 0; j < TOPK_U; ++j)
      if (g0 + j * TOPK_THREADS < n_groups) load(g0 + j * TOPK_THREADS, x[j]);
#pragma unroll
    for (int j = 0; j < TOPK_U; ++j)
      if (g0 + j * TOPK_THREADS < n_groups) {
        const int group = g0 + j * TOPK_THREADS;
        if (ODD && group == n_groups - 1) {
#pragma unroll
          for (int e = 0; e < VEC; ++e)
            if (start(group) + e < group * VEC) x[j][e] = NAN;   // counted with the group before
        }
        float m = x[j][0];
#pragma unroll
        for (int e = 1; e < VEC; ++e) m = fmaxf(m, x[j][e]);   // NaN only if the whole group is
        if (m > best_value) {   // ascending groups: the lowest id first
          best_value = m;
          best_group = group;
#pragma unroll
          for (int e = 0; e < VEC; ++e) best_x[e] = x[j][e];
        }
      }
  }
  unsigned long long mine = 0;
  if (best_group >= 0) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const unsigned long long key = key_of(best_x, best_group, e);
      if (key > mine) mine = key;
    }
  } else {   // nothing above -inf: the lowest -inf, if there is one beside NaN
    for (int g = t; g < n_groups; g += TOPK_THREADS) {
      float x[VEC];
      load(g, x);
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const unsigned long long key = key_of(x, g, e);
        if (key > mine) mine = key;
      }
    }
  }
  unsigned long long wave_best = wave_max_key<64>(mine);
  for (int j = 0; j < k; ++j) {
    if (lane == 0) s_best[j & 1][wave] = wave_best;
    __syncthreads();
    static_assert(TOPK_THREADS / 64 == 16, "one row of lanes holds the wavefronts' keys");
    const unsigned long long best = wave_max_key<16>(s_best[j & 1][lane & 15]);
    const int pick = best == 0 ? -1 : (int)~(unsigned)best;
    if (t == j) {
      const int slot = my_slot;
      if (slot >= 0 && slot < N) tree_token[(long)b * N + slot] = pick;   // nothing left but NaN: -1, a padding node
      else set_status(status, b, SPEC_ST_BAD_TREE);
    }
    if (best == wave_best && best != 0 && j + 1 < k) {   // this wavefront held the pick (keys are distinct)
      const int owner = (pick / VEC) % TOPK_THREADS;
      unsigned long long next = 0;
      for (int g = owner + lane * TOPK_THREADS; g < n_groups; g += 64 * TOPK_THREADS) {
        float x[VEC];
        load(g, x);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const unsigned long long key = key_of(x, g, e);
          if (key < best && key > next) next = key;
        }
      }
      next = wave_max_key<64>(next);
      if (t == owner) mine = next;
      wave_best = wave_max_key<64>(mine);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// token tree merge: one workgroup per request, thread g = i * Nin + u stands for node u of input tree i.
// Two input nodes are the same merged node iff they carry the same token and their parents are the same
// merged node; the representative of a merged node is its input node with the smallest g (first
// appearance), which also orders siblings. Levels are resolved top-down (a node's identity needs its
// parent's), sub-tree sizes bottom-up, depth-first positions top-down.
// The kernel is a chain of LDS steps, three per level: a workgroup has only as many wavefronts as there are nodes, the
// nodes lie in LDS in (depth, g) order, and a level compares one 64-bit key per earlier node of the level, independent
// reads instead of a chain of three. Levels of one node need no comparison and no barrier, repeated tokens end the
// comparison early, and a node's place is counted from the depths below it and the nodes before it. Measured, us, against
// 1024 threads with dependent reads and three barriers a level: 16 requests of three trees of 21 nodes 16 (26), eight trees of
// 128 57 (177..223), eight stars of 128 with three different tokens 23 (25), with 32000 47 (162), a chain of 128 40 (47).
// ---------------------------------------------------------------------------------------------
constexpr int MERGE_THREADS = SPEC_MAX_MERGE_INPUT_NODES;

__global__ void __launch_bounds__(MERGE_THREADS) tree_merge_kernel(
    int M, int Nin, const int32_t* __restrict__ in_parent, const int32_t* __restrict__ in_token,
    const int32_t* __restrict__ in_size, int Nout, int32_t* __restrict__ out_parent, int32_t* __restrict__ out_depth,
    int32_t* __restrict__ out_token, int32_t* __restrict__ out_ssm, int32_t* __restrict__ out_size,
    int32_t* __restrict__ node_map, int32_t* status) {
  __shared__ int s_par[MERGE_THREADS];     // parent as a thread index g (-1 for roots)
  __shared__ __attribute__((aligned(16))) int s_dep[MERGE_THREADS];     // depth, -1 for unused slots
  __shared__ int s_rep[MERGE_THREADS];     // representative (smallest g of the same merged node)
  __shared__ int s_sub[MERGE_THREADS];     // sub-tree size of a representative
  __shared__ int s_pos[MERGE_THREADS];     // depth-first index of a representative
  // in (depth, g) order:
  __shared__ unsigned long long l_key[MERGE_THREADS];   // (merged parent, token)
  __shared__ int l_node[MERGE_THREADS];    // g
  __shared__ int l_sub[MERGE_THREADS];     // sub-tree size of a representative, 0 for the others
  __shared__ __attribute__((aligned(16))) int s_count[MERGE_THREADS];   // nodes of a depth
  __shared__ int s_bad, s_max_depth, s_size;

  const int b = blockIdx.x, g = threadIdx.x, n_threads = blockDim.x;
  const int n_total = M * Nin;
  const int i = g / Nin, u = g % Nin;
  const int32_t* par_b = in_parent + (long)b * n_total;
  const int32_t* tok_b = in_token + (long)b * n_total;
  if (g == 0) { s_bad = 0; s_max_depth = 0; s_size = 0; }
  __syncthreads();

  // ---- load and validate
  bool active = false;
  int my_tok = -1, my_par = -1;
  if (g < n_total) {
    const int sz = in_size[(long)b * M + i], p = par_b[g], tok = tok_b[g], root_tok = tok_b[0];
    if (u == 0 && (sz < 1 || sz > Nin)) atomicOr(&s_bad, 1);
    active = u < sz && sz <= Nin;
    if (active) {
      my_tok = tok;
      if (u == 0) {
        if (p != -1 || my_tok != root_tok) atomicOr(&s_bad, 1);
      } else {
        if (p < 0 || p >= u || my_tok < 0) atomicOr(&s_bad, 1);
        my_par = i * Nin + p;
      }
    }
  }
  s_par[g] = my_par;
  s_dep[g] = -1;
  s_count[g] = 0;
  __syncthreads();
  const bool bad = s_bad != 0;

  // ---- depth (walk up; parents have smaller indices, so the walk ends)
  int my_dep = -1;
  if (active && !bad) {
    my_dep = 0;
    for (int v = my_par; v >= 0; v = s_par[v]) ++my_dep;
    s_dep[g] = my_dep;
    atomicAdd(&s_count[my_dep], 1);
    atomicMax(&s_max_depth, my_dep);
  }
  __syncthreads();
  const int max_depth = s_max_depth;
  // ---- place in (depth, g) order: nodes of smaller depth, then nodes of this depth with a smaller g
  int start = 0, my_rank = 0;
  if (my_dep >= 0) {
    int d = 0, o = 0;
#pragma unroll 4
    for (; d + 4 <= my_dep; d += 4) {
      const int4 c4 = *(const int4*)&s_count[d];
      start += (c4.x + c4.y) + (c4.z + c4.w);
    }
    for (; d < my_dep; ++d) start += s_count[d];
#pragma unroll 4
    for (; o + 4 <= g; o += 4) {
      const int4 d4 = *(const int4*)&s_dep[o];
      my_rank += (d4.x == my_dep) + (d4.y == my_dep) + (d4.z == my_dep) + (d4.w == my_dep);
    }
    for (; o < g; ++o) my_rank += s_dep[o] == my_dep;
  }
  const int place = start + my_rank;
  if (my_dep >= 0) l_node[place] = g;
  s_rep[g] = (my_dep == 0) ? 0 : g;   // every root is the merged root, first seen as thread 0
  s_sub[g] = 1;
  __syncthreads();

  // ---- identity, level by level. A node alone at its depth is its own representative: nothing to compare, nobody to wait
  // for (a chain of 128 nodes otherwise spends two barriers on each of them).
  int my_rep_par = -1;
  for (int d0 = 0; d0 <= max_depth; d0 += 4) {
    const int4 c4 = *(const int4*)&s_count[d0];
    int shared = (d0 > 0 && c4.x > 1) | (c4.y > 1) << 1 | (c4.z > 1) << 2 | (c4.w > 1) << 3;
    for (; shared != 0; shared &= shared - 1) {
      const int d = d0 + __ffs(shared) - 1;
      unsigned long long key = 0;
      if (my_dep == d) {
        my_rep_par = s_rep[my_par];
        key = ((unsigned long long)(unsigned)my_rep_par << 32) | (unsigned)my_tok;
        l_key[place] = key;
      }
      __syncthreads();
      if (my_dep == d) {
        // the first match has the smallest g; eight independent reads between two looks for an early end (trees whose nodes
        // repeat a few tokens find theirs at once)
        int first = my_rank, j = 0;
        for (; j + 8 <= my_rank && first == my_rank; j += 8)
#pragma unroll
          for (int e = 7; e >= 0; --e)
            if (l_key[start + j + e] == key) first = j + e;
        if (first == my_rank)
#pragma unroll 4
          for (; j < my_rank; ++j)
            if (l_key[start + j] == key && j < first) first = j;
        if (first < my_rank) s_rep[g] = l_node[start + first];
      }
      __syncthreads();
    }
  }
  if (my_dep > 0) my_rep_par = s_rep[my_par];
  const bool is_rep = my_dep >= 0 && s_rep[g] == g && (my_dep > 0 || g == 0);
  const unsigned long long reps = __ballot(is_rep);
  if ((g & 63) == 0 && reps != 0) atomicAdd(&s_size, __popcll(reps));
  __syncthreads();
  const int size = s_size;
  const bool overflow = size > Nout;

  if (bad || overflow) {   // defined result: an empty tree (root slot and padding), size 0, everything unmapped
    for (int n = g; n < Nout; n += n_threads) {
      out_parent[(long)b * Nout + n] = n == 0 ? -1 : 0;
      out_depth[(long)b * Nout + n] = n == 0 ? 0 : 1;
      out_token[(long)b * Nout + n] = -1;
      out_ssm[(long)b * Nout + n] = -1;
    }
    if (node_map != nullptr && g < n_total) node_map[(long)b * n_total + g] = -1;
    if (g == 0) {
      out_size[b] = 0;
      set_status(status, b, bad ? SPEC_ST_BAD_TREE : SPEC_ST_CAPACITY);
    }
    return;
  }

  // ---- sub-tree sizes, bottom-up
  for (int d = max_depth; d >= 1; --d) {
    if (my_dep == d) {
      const int sub = is_rep ? s_sub[g] : 0;
      l_sub[place] = sub;
      if (is_rep) atomicAdd(&s_sub[my_rep_par], sub);
    }
    __syncthreads();
  }
  // ---- depth-first positions, top-down: after the parent, behind the sub-trees of the earlier siblings
  int my_pos = 0;
  if (g == 0) s_pos[0] = 0;
  __syncthreads();
  for (int d = 1; d <= max_depth; ++d) {
    if (is_rep && my_dep == d) {
      my_pos = s_pos[my_rep_par] + 1;
#pragma unroll 4
      for (int j = 0; j < my_rank; ++j)
        if ((int)(l_key[start + j] >> 32) == my_rep_par) my_pos += l_sub[start + j];
      s_pos[g] = my_pos;
    }
    __syncthreads();
  }

  // ---- outputs
  if (is_rep) {
    const long n = (long)b * Nout + my_pos;
    out_parent[n] = my_dep == 0 ? -1 : s_pos[my_rep_par];
    out_depth[n] = my_dep;
    out_token[n] = my_tok;
    out_ssm[n] = i;
  }
  for (int n = size + g; n < Nout; n += n_threads) {   // padding nodes: children of the root without a token
    out_parent[(long)b * Nout + n] = 0;
    out_depth[(long)b * Nout + n] = 1;
    out_token[(long)b * Nout + n] = -1;
    out_ssm[(long)b * Nout + n] = -1;
  }
  if (node_map != nullptr && g < n_total) node_map[(long)b * n_total + g] = my_dep >= 0 ? s_pos[s_rep[g]] : -1;
  if (g == 0) out_size[b] = size;
}

// ---------------------------------------------------------------------------------------------
// The same for requests of at most 64 input nodes: one wavefront, a node per lane, sets of nodes as 64-bit masks. A lane
// compares its token with those of its depth once; a level then intersects that mask with the children of its merged parent,
// and the lowest bit is the representative. Depths and positions are sums over the way to the root by pointer doubling.
// What bounds it: a chain of some 40 LDS steps and the launch. Measured, us, against the workgroup form above with its three
// LDS steps and barriers a level: 16 requests of three trees of 21 nodes 6.8 (17.1), two requests of two trees
// 5.8 (12.9); with loops over the merged nodes on the scalar side instead of the masks 14.4 and 10.3.
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(64) tree_merge_wave_kernel(
    int M, int Nin, const int32_t* __restrict__ in_parent, const int32_t* __restrict__ in_token,
    const int32_t* __restrict__ in_size, int Nout, int32_t* __restrict__ out_parent, int32_t* __restrict__ out_depth,
    int32_t* __restrict__ out_token, int32_t* __restrict__ out_ssm, int32_t* __restrict__ out_size,
    int32_t* __restrict__ node_map, int32_t* status) {
  const int b = blockIdx.x, g = threadIdx.x;
  const int n_total = M * Nin;   // <= 64
  const int i = g / Nin, u = g % Nin;
  __shared__ __attribute__((aligned(16))) int s_tok[64], s_dep[64];
  __shared__ unsigned long long s_children[64];   // of a merged node (at its representative): every input node below it
  __shared__ int s_sub[64];                       // merged nodes below a representative, itself included

  // ---- load and validate
  bool active = false, ok = true;
  int my_tok = -1, my_par = -1;
  if (g < n_total) {
    const long at = (long)b * n_total;
    const int sz = in_size[(long)b * M + i], p = in_parent[at + g], tok = in_token[at + g], root_tok = in_token[at];
    if (u == 0 && (sz < 1 || sz > Nin)) ok = false;
    active = u < sz && sz <= Nin;
    if (active) {
      my_tok = tok;
      if (u == 0) {
        ok = ok && p == -1 && tok == root_tok;
      } else {
        ok = p >= 0 && p < u && tok >= 0;
        my_par = i * Nin + p;
      }
    }
  }
  const bool bad = __any(!ok);

  int my_dep = -1, rep = g, size = 0, my_rep_par = -1;
  unsigned long long reps = 0;
  if (!bad) {
    // ---- depth: after each exchange `up` is twice as far away
    my_dep = active ? (my_par >= 0) : -1;
    for (int up = my_par; __any(up >= 0);) {
      const int from = max(up, 0);
      const int d = __shfl(my_dep, from), next = __shfl(up, from);
      if (up >= 0) {
        my_dep += d;
        up = next;
      }
    }
    // ---- nodes of this depth with this token
    s_tok[g] = my_tok;
    s_dep[g] = my_dep;
    s_children[g] = 0;
    s_sub[g] = 1;
    __syncthreads();
    unsigned alike[2] = {0, 0};
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int j = 0; j < 32; j += 4) {
        const int4 t4 = *(const int4*)&s_tok[half * 32 + j], d4 = *(const int4*)&s_dep[half * 32 + j];
        alike[half] |= (unsigned)(t4.x == my_tok && d4.x == my_dep) << j | (unsigned)(t4.y == my_tok && d4.y == my_dep) << (j + 1) |
                       (unsigned)(t4.z == my_tok && d4.z == my_dep) << (j + 2) | (unsigned)(t4.w == my_tok && d4.w == my_dep) << (j + 3);
      }
    const unsigned long long same = (unsigned long long)alike[1] << 32 | alike[0];
    // ---- identity, level by level: of the nodes alike below one merged parent the first represents all
    if (my_dep == 0) rep = 0;
    for (int d = 1; __any(my_dep >= d); ++d) {
      const int rep_par = __shfl(rep, max(my_par, 0));
      if (my_dep == d) {
        my_rep_par = rep_par;
        atomicOr(&s_children[rep_par], 1ull << g);
      }
      __syncthreads();
      if (my_dep == d) rep = __ffsll((long long)(same & s_children[rep_par])) - 1;
    }
    reps = __ballot(my_dep >= 0 && rep == g);
    size = __popcll(reps);
  }

  if (bad || size > Nout) {   // defined result: an empty tree (root slot and padding), size 0, everything unmapped
    for (int n = g; n < Nout; n += 64) {
      out_parent[(long)b * Nout + n] = n == 0 ? -1 : 0;
      out_depth[(long)b * Nout + n] = n == 0 ? 0 : 1;
      out_token[(long)b * Nout + n] = -1;
      out_ssm[(long)b * Nout + n] = -1;
    }
    if (node_map != nullptr && g < n_total) node_map[(long)b * n_total + g] = -1;
    if (g == 0) {
      out_size[b] = 0;
      set_status(status, b, bad ? SPEC_ST_BAD_TREE : SPEC_ST_CAPACITY);
    }
    return;
  }

  // ---- sub-tree sizes: every merged node counts at each one above it
  const bool is_rep = (reps >> g) & 1;
  for (int a = is_rep ? my_rep_par : -1; __any(a >= 0);) {
    const int next = __shfl(my_rep_par, max(a, 0));
    if (a >= 0) {
      atomicAdd(&s_sub[a], 1);
      a = next;
    }
  }
  __syncthreads();
  // ---- depth-first positions: a node comes one behind its parent and behind its earlier siblings' sub-trees
  int pos = 0, up = is_rep ? my_rep_par : -1;
  if (up >= 0) {
    pos = 1;
    for (unsigned long long before = s_children[up] & reps & ((1ull << g) - 1); before != 0; before &= before - 1)
      pos += s_sub[__ffsll((long long)before) - 1];
  }
  while (__any(up >= 0)) {
    const int from = max(up, 0);
    const int more = __shfl(pos, from), next = __shfl(up, from);
    if (up >= 0) {
      pos += more;
      up = next;
    }
  }

  // ---- outputs
  const int par_pos = __shfl(pos, max(my_rep_par, 0)), rep_pos = __shfl(pos, rep);
  if (is_rep) {
    const long n = (long)b * Nout + pos;
    out_parent[n] = my_dep == 0 ? -1 : par_pos;
    out_depth[n] = my_dep;
    out_token[n] = my_tok;
    out_ssm[n] = i;
  }
  for (int n = size + g; n < Nout; n += 64) {   // padding nodes: children of the root without a token
    out_parent[(long)b * Nout + n] = 0;
    out_depth[(long)b * Nout + n] = 1;
    out_token[(long)b * Nout + n] = -1;
    out_ssm[(long)b * Nout + n] = -1;
  }
  if (node_map != nullptr && g < n_total) node_map[(long)b * n_total + g] = my_dep >= 0 ? rep_pos : -1;
  if (g == 0) out_size[b] = size;
}

hipError_t launch_expand_topk(int B, int F, int V, int logits_dtype, const void* logits, int k, const int32_t* child_slot,
                              int N, int32_t* tree_token, int32_t* status, hipStream_t s) {
  const bool bf16 = logits_dtype == SPEC_BF16;
  const int vec = bf16 ? 8 : 4;   // elements of a 16-byte load
  const bool odd = V % vec != 0 || (reinterpret_cast<uintptr_t>(logits) & 15u) != 0;
#define SPEC_TOPK(BF, VE, OD)                                                                                             \
  hipLaunchKernelGGL((expand_topk_kernel<BF, VE, OD>), dim3(B * F), dim3(TOPK_THREADS), 0, s, logits, F, V, k, child_slot, N, \
                     tree_token, status)
  if (V < vec) { if (bf16) SPEC_TOPK(true, 1, false); else SPEC_TOPK(false, 1, false); }
  else if (bf16) { if (odd) SPEC_TOPK(true, 8, true); else SPEC_TOPK(true, 8, false); }
  else { if (odd) SPEC_TOPK(false, 4, true); else SPEC_TOPK(false, 4, false); }
#undef SPEC_TOPK
  return hipGetLastError();
}

hipError_t launch_tree_merge(int B, int M, int Nin, const int32_t* in_parent, const int32_t* in_token,
                             const int32_t* in_size, int Nout, int32_t* out_parent, int32_t* out_depth,
                             int32_t* out_token, int32_t* out_ssm, int32_t* out_size, int32_t* node_map, int32_t* status,
                             hipStream_t s) {
  const int threads = (M * Nin + 63) / 64 * 64;   // one per input node
  hipLaunchKernelGGL(threads == 64 ? tree_merge_wave_kernel : tree_merge_kernel, dim3(B), dim3(threads), 0, s, M, Nin,
                     in_parent, in_token, in_size, Nout, out_parent, out_depth, out_token, out_ssm, out_size, node_map, status);
  return hipGetLastError();
}

}  // namespace spec
