// Token-tree verification on the GPU (Algorithm 2: VerifyGreedy and VerifyStochastic, Section 4.3).
//
// The paper runs verification on the host after copying the LLM's per-node outputs back; here it
// stays on the device so an iteration needs no host round trip. The kernels:
//   node_stats_kernel      one workgroup per (request, node) row of logits: argmax (lowest token id on
//                          ties), max, and sum of exp((x - max)/T). All nodes in parallel, so the
//                          sequential tree walk that follows needs P(x) at a node in O(1).
//   greedy_walk_kernel     one workgroup per request: follow children whose token equals the node's
//                          argmax; emit the bonus token.
//   stochastic_walk_kernel one workgroup per request: multi-step speculative sampling. A node's softmax statistics
//                          are the precomputed ones or (many nodes) taken when the walk reaches it; only a rejection
//                          needs the residual distribution norm(max(0, P - Q)) (one pass over the vocabulary per
//                          rejection, kept un-normalised with its mass Z). The last token is drawn by inverse CDF with
//                          a float64 block scan in token-id order. Two forms: the current distribution in the
//                          workgroup's registers (vocabularies up to 32768), or in a buffer in memory.
//   node_sample_kernel     naive sampling (the alternative of Section 4.3): one inverse-CDF draw per
//                          (request, node) row; the greedy walk then runs on the sampled tokens.
#include <hip/hip_bf16.h>

#include "spec_internal.h"

namespace spec {

template <bool BF16>
__device__ inline float load_logit(const void* base, long idx) {
  if (BF16) return __bfloat162float(((const __hip_bfloat16*)base)[idx]);
  return ((const float*)base)[idx];
}

// ---------------------------------------------------------------------------------------------
// Vocabulary sweeps. A row of V values is visited in groups of VEC consecutive elements: 4 (16 bytes of float, 8 of bf16; the
// arg-max alone takes 8 of bf16) for every V of at least as many, the last group ending with the row, and 1 for shorter rows.
// A block of NT threads takes U groups per thread at a time, all loads issued before any is used: with V = 32000, NT = 1024,
// U = 8 a whole row is one round trip to memory.
// ---------------------------------------------------------------------------------------------
constexpr int SWEEP_U = 8;

// Barrier for LDS contents only: __syncthreads() also waits for the loads in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Rows of any length by whole groups of VEC elements: the last group ends with the row and so repeats elements of the one
// before it where VEC does not divide V. Rows of odd vocabularies start at any element; the memory unit takes such loads
// (single elements before. Stochastic verification, 4 trees of 32, 31999 bfloat16: 48.6 us, 30.9 now; greedy, 1024 rows of
// 50257 bfloat16: 94, 22 now, 8 rows of 56877: 13.3, 7.8).
__device__ __forceinline__ int group_start(int group, int vec, int V) { return min(group * vec, V - vec); }
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef u32x4 __attribute__((aligned(2))) u32x4_any;
typedef u32x2 __attribute__((aligned(2))) u32x2_any;
typedef f32x4 __attribute__((aligned(4))) f32x4_any;

template <int VEC>
__device__ __forceinline__ void load_f32_group(const float* p, float (&v)[VEC]) {
  if (VEC == 4) {
    const f32x4 raw = *(const f32x4_any*)p;
    v[0] = raw.x; v[1] = raw.y; v[2] = raw.z; v[3] = raw.w;
  } else {
    v[0] = *p;
  }
}
template <int VEC>
__device__ __forceinline__ void store_f32_group(float* p, const float (&v)[VEC]) {
  if (VEC == 4) *(f32x4_any*)p = (f32x4){v[0], v[1], v[2], v[3]};
  else *p = v[0];
}

// ---------------------------------------------------------------------------------------------
// block-wide reductions (blockDim.x multiple of 64, <= 1024); `scratch` holds >= 16 entries
// ---------------------------------------------------------------------------------------------
template <typename T>
__device__ inline T block_sum(T v, T* scratch) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) scratch[w] = v;
  __syncthreads();
  T tot = 0;
  for (int i = 0; i < nw; ++i) tot += scratch[i];
  return tot;
}

// VEC elements of a row of logits as they lie in memory: a row's loads are all requested before the first one is converted (a
// conversion beside its load waits for it, 32 bf16 elements per thread one after the other).
template <bool BF16, int VEC>
struct LogitGroup {
  unsigned raw[BF16 ? (VEC + 1) / 2 : VEC];
  __device__ __forceinline__ void load(const void* base, unsigned elem) {
    if constexpr (VEC == 4 && BF16) {
      const u32x2 v = *(const u32x2_any*)((const unsigned short*)base + elem);
      raw[0] = v.x; raw[1] = v.y;
    } else if constexpr (VEC == 4) {
      const u32x4 v = *(const u32x4_any*)((const float*)base + elem);
      raw[0] = v.x; raw[1] = v.y; raw[2] = v.z; raw[3] = v.w;
    } else if constexpr (BF16) {
      raw[0] = ((const unsigned short*)base)[elem];
    } else {
      raw[0] = __float_as_uint(((const float*)base)[elem]);
    }
  }
  __device__ __forceinline__ void set_minus_infinity() {
#pragma unroll
    for (unsigned& r : raw) r = BF16 ? 0xff80ff80u : 0xff800000u;
  }
  __device__ __forceinline__ void expand(float (&v)[VEC]) {
    if constexpr (BF16 && VEC == 1) asm("" : "+v"(raw[0]));   // (the compiler moves this one back to its load otherwise)
#pragma unroll
    for (int e = 0; e < VEC; ++e) v[e] = __uint_as_float(!BF16 ? raw[e] : e % 2 == 0 ? raw[e / 2] << 16 : raw[e / 2] & 0xffff0000u);
  }
};

// The elements of the row's last group that the group before it holds too.
template <int VEC>
__device__ __forceinline__ void drop_repeated(float (&v)[VEC], int group, int n_groups, int V, float with) {
  if (group == n_groups - 1) {
    const int repeated = group * VEC - group_start(group, VEC, V);
#pragma unroll
    for (int e = 0; e < VEC; ++e)
      if (e < repeated) v[e] = with;
  }
}

// ---------------------------------------------------------------------------------------------
// per-node statistics: one block of 256 or 1024 threads per (request, node) row, one pass over the row.
// Each thread keeps (max, lowest index of the max, sum of exp((x - max) / T)) of its elements; the
// block combines the triples.
// ---------------------------------------------------------------------------------------------
// Workgroup size: 1024 threads when there are few rows (a row is then one round trip to memory), 256 when there
// are thousands: eight small workgroups per compute unit overlap one another's loads and arithmetic, where two
// large ones alternate between a load phase and a compute phase (2048 rows of 32000 floats: 61 us before). A sweep has as many
// groups per thread as the row needs of 2, 4 and 8 (U): empty ones cost their exponentials like full ones (the pass over 315 rows
// of 4224 float32 12.1 us with eight, 6.7 with two; of 4098, by eight single elements a thread before, 6.5, 6.5 now).

// exp(x) for x <= 0 as one v_exp_f32 (1 ulp; results below 2^-126 become 0). The sum over a vocabulary row is
// bound by this instruction count: the library expf costs about ten instructions per element, and the
// statistics kernel ran at half the speed of its max-only form with it.
__device__ __forceinline__ float fast_exp(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }

// Whether a tree has at most `levels` nodes on every path from its root: nodes `lane` and `lane + 64` have the parents par0
// and par1 (-1: none), all 64 lanes ask together. After i exchanges a lane knows the distance to its ancestor 2^i up, so a
// deep tree is found out after log2(levels) of them. Parents that form no tree get some answer, the same one every time.
__device__ inline bool tree_within(int par0, int par1, int levels) {
  static_assert(SPEC_MAX_TREE_NODES == 128, "two nodes per lane");
  int up[2] = {par0, par1}, d[2] = {1, 1};   // the nodes from this one up to, without, node up
  for (int i = 0; i < 7 && __any(up[0] >= 0 || up[1] >= 0); ++i) {
    int nu[2], nd[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int f = min(max(up[e], 0), SPEC_MAX_TREE_NODES - 1), l = f & 63;
      const int u0 = __shfl(up[0], l), u1 = __shfl(up[1], l), d0 = __shfl(d[0], l), d1 = __shfl(d[1], l);
      nu[e] = up[e] < 0 ? -1 : f < 64 ? u0 : u1;
      nd[e] = up[e] < 0 ? d[e] : d[e] + (f < 64 ? d0 : d1);
    }
    up[0] = nu[0]; up[1] = nu[1]; d[0] = nd[0]; d[1] = nd[1];
    if (__any(max(d[0], d[1]) > levels)) return false;
  }
  return !__any(max(d[0], d[1]) > levels);
}

// parent != nullptr: the rows of requests whose tree is within `own_levels` levels are left out (the stochastic walk takes
// their nodes' statistics itself).
template <bool BF16, int VEC, int NS_THREADS, int U>
__global__ void __launch_bounds__(NS_THREADS) node_stats_kernel(const void* __restrict__ logits, int V, float inv_temp,
                                                                int32_t* __restrict__ node_argmax,
                                                                float* __restrict__ node_max,
                                                                float* __restrict__ node_sumexp,
                                                                const int32_t* __restrict__ parent, int N, int own_levels) {
  __shared__ float s_val[NS_THREADS / 64];
  __shared__ int s_idx[NS_THREADS / 64];
  __shared__ float s_sum[NS_THREADS / 64];
  const long row = blockIdx.x;
  const int t = threadIdx.x;
  const long base = row * V;
  const int n_groups = (V + VEC - 1) / VEC;
  const bool want_sum = node_sumexp != nullptr;
  if (parent != nullptr) {
    const int lane = t & 63;
    const int32_t* par = parent + row / N * N;
    if (tree_within(lane < N ? par[lane] : -1, lane + 64 < N ? par[lane + 64] : -1, own_levels)) return;
  }
  float best = -INFINITY, sum = 0.f;
  int best_i = 0x7fffffff;
  for (int g0 = 0; g0 < n_groups; g0 += NS_THREADS * U) {
    float x[U][VEC];
    LogitGroup<BF16, VEC> raw[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int gi = g0 + j * NS_THREADS + t;
      if (gi < n_groups) raw[j].load((const char*)logits + base * (BF16 ? 2 : 4), (unsigned)group_start(gi, VEC, V));
      else raw[j].set_minus_infinity();
    }
#pragma unroll
    for (int j = 0; j < U; ++j) raw[j].expand(x[j]);
    if (V % VEC != 0) {
#pragma unroll
      for (int j = 0; j < U; ++j) drop_repeated<VEC>(x[j], g0 + j * NS_THREADS + t, n_groups, V, -INFINITY);
    }
    float m = best;
#pragma unroll
    for (int j = 0; j < U; ++j)
#pragma unroll
      for (int e = 0; e < VEC; ++e)
        if (x[j][e] > m) { m = x[j][e]; best_i = group_start(g0 + j * NS_THREADS + t, VEC, V) + e; }   // ascending index: lowest wins ties
    if (want_sum && m > -INFINITY) {
      sum *= fast_exp((best - m) * inv_temp);     // best = -inf gives 0
#pragma unroll
      for (int j = 0; j < U; ++j)
#pragma unroll
        for (int e = 0; e < VEC; ++e) sum += fast_exp((x[j][e] - m) * inv_temp);   // padding: exp(-inf) = 0
    }
    best = m;
  }
  // combine (value desc, index asc); sums are rescaled to the common maximum
  const float my_best = best;
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(best, o);
    const int oi = __shfl_xor(best_i, o);
    if (ov > best || (ov == best && oi < best_i)) { best = ov; best_i = oi; }
  }
  if ((t & 63) == 0) { s_val[t >> 6] = best; s_idx[t >> 6] = best_i; }
  __syncthreads();
  best = s_val[0]; best_i = s_idx[0];
  for (int w = 1; w < NS_THREADS / 64; ++w)
    if (s_val[w] > best || (s_val[w] == best && s_idx[w] < best_i)) { best = s_val[w]; best_i = s_idx[w]; }
  if (best_i == 0x7fffffff) best_i = 0;   // all -inf / NaN row
  if (want_sum) {
    if (my_best > -INFINITY) sum *= fast_exp((my_best - best) * inv_temp); else sum = 0.f;
    sum = block_sum(sum, s_sum);
  }
  if (t == 0) {
    if (node_argmax != nullptr) node_argmax[row] = best_i;
    if (node_max != nullptr) node_max[row] = best;
    if (want_sum) node_sumexp[row] = sum;
  }
}

constexpr int SW_THREADS = 1024;

// ---------------------------------------------------------------------------------------------
// arg-max (and maximum) of a row without the sum, for rows of at least one 16-byte group (4 floats or 8 bf16). The pass over all
// nodes of greedy verification is bound by memory only if an element costs few instructions: a group costs its maximum, one
// comparison and the selection of the group's raw bits, and which element it was is found once per thread at the end
// (1024 rows of 32000 bf16: 17.0 us with a comparison and two selections per element and 8-byte loads, 12.4 now;
// 2048 rows of 32000 float32: 47 before, 45 now).
//
// HALVES: half a sweep is on its way while the other half is looked at, and an odd number of halves costs no empty one; which
// form is the faster is in argmax_by_halves.
// ---------------------------------------------------------------------------------------------
template <bool BF16, int NT, bool ODD, bool HALVES>   // ODD: V is no multiple of VEC (by halves only)
__global__ void __launch_bounds__(NT) node_argmax_kernel(const void* __restrict__ logits, int V, int32_t* __restrict__ node_argmax,
                                                         float* __restrict__ node_max) {
  constexpr int VEC = BF16 ? 8 : 4, WAVES = NT / 64;
  typedef std::conditional_t<HALVES, u32x4, uint4> Raw;   // (as u32x4 the whole sweeps take 72 registers, and one workgroup per unit)
  __shared__ float s_val[WAVES];
  __shared__ int s_idx[WAVES];
  const long row = blockIdx.x;
  const int t = threadIdx.x;
  // ODD: groups lie on 16-byte boundaries but for the first, which starts with the row, and the last, which ends with it; they
  // repeat elements of their neighbours, which changes nothing here.
  const int n_groups = ODD ? (V + VEC - 1) / VEC + 2 : V / VEC;
  const int lead = ODD ? (int)(row * V % VEC == 0 ? 0 : VEC - row * V % VEC) - VEC : 0;
  const char* base = (const char*)logits + row * V * (BF16 ? 2 : 4);
  auto start_of = [&](int group) { return ODD ? max(0, min(group * VEC + lead, V - VEC)) : group * VEC; };
  auto expand = [](const Raw raw, float (&x)[VEC]) {
    const unsigned w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (BF16) {
        x[2 * i] = __uint_as_float(w[i] << 16);
        x[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
      } else {
        x[i] = __uint_as_float(w[i]);
      }
    }
  };
  float best = -INFINITY;
  int best_g = -1;
  Raw best_raw = {0u, 0u, 0u, 0u};
  constexpr int U = HALVES ? SWEEP_U / 2 : SWEEP_U;
  auto load = [&](Raw (&raw)[U], int g0) {
#pragma unroll
    for (int j = 0; j < U; ++j) {   // (past the end: the last group again, which changes nothing)
      const int g = min(g0 + j * NT, n_groups - 1);
      if constexpr (ODD) raw[j] = *(const u32x4_any*)(base + start_of(g) * (BF16 ? 2 : 4));
      else raw[j] = ((const Raw*)base)[g];
    }
  };
  auto look_at = [&](const Raw (&raw)[U], int g0) {
#pragma unroll
    for (int j = 0; j < U; ++j) {
      float x[VEC];
      expand(raw[j], x);
      float m = x[0];
#pragma unroll
      for (int e = 1; e < VEC; ++e) m = fmaxf(m, x[e]);   // NaN only if the whole group is
      if (m > best) {   // ascending groups: the lowest wins ties
        best = m;
        best_g = min(g0 + j * NT, n_groups - 1);
        best_raw = raw[j];
      }
    }
  };
  if constexpr (!HALVES) {
    for (int g0 = t; g0 < n_groups; g0 += NT * U) {
      Raw raw[U];
      load(raw, g0);
      look_at(raw, g0);
    }
  } else if (ODD || t < n_groups) {
    Raw even[U], odd[U];
    load(even, t);
    for (int g0 = t;; g0 += 2 * U * NT) {   // (the last half apart: nothing is requested behind it)
      if (g0 - t + U * NT >= n_groups) {
        look_at(even, g0);
        break;
      }
      load(odd, g0 + U * NT);
      look_at(even, g0);
      if (g0 - t + 2 * U * NT >= n_groups) {
        look_at(odd, g0 + U * NT);
        break;
      }
      load(even, g0 + 2 * U * NT);
      look_at(odd, g0 + U * NT);
    }
  }
  int best_i = 0x7fffffff;
  if (best_g >= 0) {
    float x[VEC];
    expand(best_raw, x);
#pragma unroll
    for (int e = VEC - 1; e >= 0; --e)
      if (x[e] == best) best_i = start_of(best_g) + e;
  }
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(best, o);
    const int oi = __shfl_xor(best_i, o);
    if (ov > best || (ov == best && oi < best_i)) { best = ov; best_i = oi; }
  }
  if ((t & 63) == 0) { s_val[t >> 6] = best; s_idx[t >> 6] = best_i; }
  __syncthreads();
  if (t == 0) {
    for (int w = 1; w < WAVES; ++w)
      if (s_val[w] > best || (s_val[w] == best && s_idx[w] < best_i)) { best = s_val[w]; best_i = s_idx[w]; }
    if (node_argmax != nullptr) node_argmax[row] = best_i == 0x7fffffff ? 0 : best_i;   // all -inf / NaN row
    if (node_max != nullptr) node_max[row] = best;
  }
}

// ---------------------------------------------------------------------------------------------
// greedy walk: one wavefront per request, lane v <-> nodes v and v + 64. Everything is read once at the start; a step is
// one LDS read and two ballots, without a barrier (a launch of nothing else: bound by its latency, 3.8 us with a workgroup,
// three barriers and a read from memory per step, 2.2 to 3.4 now).
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(64) greedy_walk_kernel(int N, const int32_t* __restrict__ node_argmax,
                                                         const int32_t* __restrict__ token,
                                                         const int32_t* __restrict__ parent, int Lmax,
                                                         int32_t* __restrict__ path, int32_t* __restrict__ len,
                                                         int32_t* __restrict__ out_tokens, int32_t* status) {
  static_assert(SPEC_MAX_TREE_NODES == 128, "two nodes per lane");
  __shared__ int s_arg[SPEC_MAX_TREE_NODES], s_tok[SPEC_MAX_TREE_NODES], s_path[SPEC_MAX_TREE_NODES];
  const int b = blockIdx.x, lane = threadIdx.x;
  int par[2], tok[2];
  bool ok = true;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int v = lane + 64 * i;
    const long at = (long)b * N + min(v, N - 1);
    par[i] = parent[at];
    tok[i] = token[at];
    const int a = node_argmax[at];
    if (v >= N) par[i] = -2;
    else ok = ok && (v == 0 ? par[i] == -1 : (par[i] >= 0 && par[i] < v));
    s_tok[v] = tok[i];
    s_arg[v] = a;
  }
  const bool valid = __all(ok);
  __builtin_amdgcn_wave_barrier();
  int u = 0, k = 0;
  if (lane == 0) s_path[0] = 0;
  while (valid && k + 1 < Lmax) {
    const int want = s_arg[u];
    const unsigned long long m0 = __ballot(par[0] == u && tok[0] == want), m1 = __ballot(par[1] == u && tok[1] == want);
    if ((m0 | m1) == 0) break;
    u = m0 != 0 ? __ffsll((long long)m0) - 1 : 63 + __ffsll((long long)m1);   // the lowest index
    ++k;
    if (lane == 0) s_path[k] = u;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  for (int j = lane; j < Lmax; j += 64) {   // node path[j] emits the token of the next node, the last its arg-max
    path[(long)b * Lmax + j] = valid && j <= k ? s_path[j] : -1;
    out_tokens[(long)b * Lmax + j] = !valid || j > k ? -1 : j < k ? s_tok[s_path[j + 1]] : s_arg[u];
  }
  if (lane == 0) {
    len[b] = valid ? k + 1 : 0;
    if (!valid) set_status(status, b, SPEC_ST_BAD_TREE);
  }
}

// ---------------------------------------------------------------------------------------------
// stochastic walk with the current distribution in registers: blockDim = 1024, thread t holds the groups t, t + 1024, ...
// of VEC elements (NG of them, so V <= 1024 NG VEC). A row is read once per visited node, a draft's distribution once per
// rejection, nothing is written but the result; the buffer form below reads and writes the residual per rejection and
// reads the row again for every rejection and for the final draw.
//
// own_levels > 0: the softmax statistics of the nodes of a tree within that many levels are taken here, from rows that are
// then in registers if a child is rejected or the last token is drawn. That saves the pass over all nodes, most of whose rows
// the walk does not reach, and makes an accepted node dearer: see stochastic_own_levels for the line between them.
// node_max == nullptr: every tree is such a tree.
//
// What bounds it: one compute unit per request: a row of 32000 float32 takes it about 2.5 us, and a step of the walk is one
// or two of them in a chain, with one barrier each. What the tests need of the tree is fetched and ordered for all nodes while
// the root's row is on its way, and every wavefront follows the walk by itself (a node's children listed, sorted and fetched
// as the walk reached them: six barriers and a trip to memory more per node). Measured, us, before and now: 16 requests, trees
// of 128, 32000 float32, three drafts, 49.1 / 44.6; chains of 128, all accepted, 231 / 130; 32 trees of 128, 4000 float32,
// 25.2 / 22.9.
// ---------------------------------------------------------------------------------------------

// exp(x) for x <= 0, subnormal results included (a draw at 0 takes the first token that has any weight): 2^n 2^f with n the integer
// nearest x log2(e), whose rest f is taken before anything is rounded away. n comes out of a sum with 1.5 * 2^23, as a float and
// in that sum's last bits (an integer conversion is as slow as v_exp_f32); below 2^-200 it stops, so that -inf has a rest.
// Largest relative error over [-87, 0] 8.5e-8, of subnormals one step. The walk of 16 trees of 128, 32000 float32, three drafts
// takes 42.7 us; with expf, whose own error is 2.7e-6 when it is compiled with contraction, 45.8; with one v_exp_f32 of the whole
// exponent and its rounding put back afterwards (1.4e-7, and 0 below 2^-126), 41.7.
__device__ __forceinline__ float exp_of_nonpositive(float x) {
  const float shifted = fmaxf(fmaf(x, 1.44269502f, 12582912.f), 12582912.f - 200.f), n = shifted - 12582912.f;
  const float f = fmaf(x, 1.925963033500e-08f, fmaf(x, 1.44269502f, -n));   // log2(e) = 1.44269502162933 + 1.926e-8
  return ldexpf(__builtin_amdgcn_exp2f(f), (int)(__float_as_uint(shifted) - 0x4b400000u));
}
// Sums and maxima over a wavefront in register moves (row shifts, then the last lane of a row into the rows after it).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_f32(float identity, float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(identity), __float_as_int(v), CTRL, ROW_MASK, 0xf, false));
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_f64(double v) {   // 0 where there is no source
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROW_MASK, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROW_MASK, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
struct MaxOp {
  static constexpr float identity = -INFINITY;
  static __device__ __forceinline__ float f(float a, float b) { return fmaxf(a, b); }
};
struct SumOp {
  static constexpr float identity = 0.f;
  static __device__ __forceinline__ float f(float a, float b) { return a + b; }
};
template <class Op>
__device__ __forceinline__ float row_reduce(float v) {   // lane 15: over its row of 16
  v = Op::f(v, dpp_f32<0x111, 0xf>(Op::identity, v));
  v = Op::f(v, dpp_f32<0x112, 0xf>(Op::identity, v));
  v = Op::f(v, dpp_f32<0x114, 0xf>(Op::identity, v));
  return Op::f(v, dpp_f32<0x118, 0xf>(Op::identity, v));
}
template <class Op>
__device__ __forceinline__ float wave_reduce(float v) {   // lane 63: over the wavefront
  v = row_reduce<Op>(v);
  v = Op::f(v, dpp_f32<0x142, 0xa>(Op::identity, v));
  return Op::f(v, dpp_f32<0x143, 0xc>(Op::identity, v));
}
__device__ __forceinline__ float readlane_f32(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
// Sum over the block; every thread gets the result. `slot` points at 16 floats that no thread still reads from the call
// before the last (two areas used in turn): one barrier.
__device__ __forceinline__ float block_total(float v, float* slot) {
  v = wave_reduce<SumOp>(v);
  if ((threadIdx.x & 63) == 63) slot[threadIdx.x >> 6] = v;
  __syncthreads();
  return readlane_f32(row_reduce<SumOp>(slot[threadIdx.x & 15]), 15);
}
// (max, sum of exp((x - max) / T)) over the block from those of its threads; every thread gets the result. `slot`: 16 pairs
// that no thread still reads; one barrier.
__device__ __forceinline__ void block_softmax_stats(float m, float sum, float inv_temp, float2* slot, float* max_out, float* sum_out) {
  auto rescaled = [&](float s, float from, float to) { return from > -INFINITY ? s * fast_exp((from - to) * inv_temp) : 0.f; };
  const float wave_max = readlane_f32(wave_reduce<MaxOp>(m), 63);
  const float wave_sum = wave_reduce<SumOp>(rescaled(sum, m, wave_max));
  if ((threadIdx.x & 63) == 63) slot[threadIdx.x >> 6] = make_float2(wave_max, wave_sum);
  __syncthreads();
  const float2 p = slot[threadIdx.x & 15];
  *max_out = readlane_f32(row_reduce<MaxOp>(p.x), 15);
  *sum_out = readlane_f32(row_reduce<SumOp>(rescaled(p.y, p.x, *max_out)), 15);
}
__device__ __forceinline__ double wave_inclusive_sum_f64(double v) {
  v += dpp_f64<0x111, 0xf>(v);
  v += dpp_f64<0x112, 0xf>(v);
  v += dpp_f64<0x114, 0xf>(v);
  v += dpp_f64<0x118, 0xf>(v);
  v += dpp_f64<0x142, 0xa>(v);
  v += dpp_f64<0x143, 0xc>(v);
  return v;
}
__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const long long b = __double_as_longlong(v);
  return __longlong_as_double(((long long)__builtin_amdgcn_readlane((int)(b >> 32), lane) << 32) |
                              (unsigned)__builtin_amdgcn_readlane((int)b, lane));
}

template <bool BF16, int VEC, int NG, bool ODD>   // ODD: V is no multiple of VEC
__global__ void __launch_bounds__(SW_THREADS) stochastic_walk_reg_kernel(
    int N, int V, const void* __restrict__ logits, const float* __restrict__ probs_ssm, int R,
    const int32_t* __restrict__ ssm_row, const int32_t* __restrict__ token, const int32_t* __restrict__ parent,
    const float* __restrict__ u_accept, const float* __restrict__ u_order, const float* __restrict__ u_final,
    float inv_temp, const float* __restrict__ node_max, const float* __restrict__ node_sumexp, int own_levels, int Lmax,
    int32_t* __restrict__ path, int32_t* __restrict__ len, int32_t* __restrict__ out_tokens, int32_t* status) {
  constexpr int WAVES = SW_THREADS / 64, NTOT = NG * WAVES < 64 ? 64 : NG * WAVES;   // final scan: (group round, wavefront)
  static_assert(NTOT % 64 == 0, "whole rounds of lanes");
  __shared__ int s_flag, s_ans;
  // per node: its parent if it is a candidate (else -2) and what a ratio test needs; siblings' order of testing
  __shared__ __attribute__((aligned(16))) int s_par[SPEC_MAX_TREE_NODES];
  __shared__ __attribute__((aligned(16))) float s_ord[SPEC_MAX_TREE_NODES];
  __shared__ int s_rank[SPEC_MAX_TREE_NODES], s_tok[SPEC_MAX_TREE_NODES], s_row[SPEC_MAX_TREE_NODES];
  __shared__ float s_acc[SPEC_MAX_TREE_NODES], s_cq[SPEC_MAX_TREE_NODES], s_cl[SPEC_MAX_TREE_NODES];
  __shared__ float s_red[2][WAVES];
  __shared__ float2 s_stats[2][WAVES];
  __shared__ double s_tot[NTOT];

  const int b = blockIdx.x, t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int n_groups = (V + VEC - 1) / VEC;

  float w[NG][VEC];   // the row of node u: its logits, then the current distribution, un-normalised: P(i) = w_i / Z
  // Rows are addressed as a wave-uniform base per round plus one offset per lane, or (ODD) a base and a 32-bit offset per load:
  // 64-bit addresses would not leave room for the row in registers; u and rows of probs_ssm are made uniform for that.
  auto load_row = [&](int u) {   // the logits of node u; elements past the end are -inf
    const char* row = (const char*)logits + ((long)b * N + u) * V * (BF16 ? 2 : 4);
    LogitGroup<BF16, VEC> raw[NG];
#pragma unroll
    for (int j = 0; j < NG; ++j) {
      if (j * SW_THREADS + t >= n_groups) raw[j].set_minus_infinity();
      else if (ODD) raw[j].load(row, (unsigned)group_start(j * SW_THREADS + t, VEC, V));
      else raw[j].load(row + j * SW_THREADS * VEC * (BF16 ? 2 : 4), (unsigned)(t * VEC));
    }
#pragma unroll
    for (int j = 0; j < NG; ++j) raw[j].expand(w[j]);
    if (ODD) {
#pragma unroll
      for (int j = 0; j < NG; ++j) drop_repeated<VEC>(w[j], j * SW_THREADS + t, n_groups, V, -INFINITY);
    }
  };

  static_assert(SPEC_MAX_TREE_NODES == 128, "two nodes per lane, parents in the bits from 7 up");
  // Everything that the ratio tests need of the tree, for all nodes at once while the root's row is on its way: a node has one
  // parent, so its Q(x), its logit and its place among its siblings are known without the walk. From then on every wavefront
  // follows the walk by itself, nodes lane and lane + 64 in its registers, and waits for the others only in the sums.
  if (own_levels > 0) load_row(0);
  if (t == 0) s_flag = 0;
  int my_par = -2, my_tok = -1, my_row = 0;
  float my_ord = 0.f, my_acc = 0.f;
  bool ok = true;
  if (t < N) {
    my_par = parent[(long)b * N + t];
    my_tok = token[(long)b * N + t];
    my_row = ssm_row[(long)b * N + t];
    my_ord = u_order[(long)b * N + t];
    my_acc = u_accept[(long)b * N + t];
    ok = t == 0 ? my_par == -1 : (my_par >= 0 && my_par < t);
    if (t >= 1 && my_tok >= 0 && (my_tok >= V || my_row < 0 || my_row >= R)) ok = false;
  }
  const bool candidate = t < N && t >= 1 && my_tok >= 0 && ok;   // a negative token: a padding node, never a candidate
  float my_q0 = 0.f, my_logit = 0.f;   // on their way while the siblings are ordered
  if (candidate) {
    my_q0 = probs_ssm[(long)my_row * V + my_tok];
    my_logit = load_logit<BF16>(logits, ((long)b * N + my_par) * V + my_tok);
  }
  if (t < SPEC_MAX_TREE_NODES) {
    s_par[t] = candidate ? my_par : -2;
    s_ord[t] = my_ord;
    s_tok[t] = my_tok;
    s_row[t] = my_row;
    s_acc[t] = my_acc;
    s_rank[t] = 0;
  }
  lds_barrier();
  if (!ok) atomicOr(&s_flag, 1);
  {   // place among the siblings in ascending (u_order, index): eight threads per node, each against a part of the others
    constexpr int PART = SPEC_MAX_TREE_NODES * SPEC_MAX_TREE_NODES / SW_THREADS;
    const int v = t % SPEC_MAX_TREE_NODES, from = t / SPEC_MAX_TREE_NODES * PART;
    const int par = s_par[v];
    const float ord = s_ord[v];
    int rank = 0;
    if (par >= 0 && from < N) {
#pragma unroll
      for (int j = from; j < from + PART; j += 4) {
        const int4 p4 = *(const int4*)&s_par[j];
        const float4 o4 = *(const float4*)&s_ord[j];
        rank += p4.x == par && (o4.x < ord || (o4.x == ord && j < v));
        rank += p4.y == par && (o4.y < ord || (o4.y == ord && j + 1 < v));
        rank += p4.z == par && (o4.z < ord || (o4.z == ord && j + 2 < v));
        rank += p4.w == par && (o4.w < ord || (o4.w == ord && j + 3 < v));
      }
    }
    if (rank > 0) atomicAdd(&s_rank[v], rank);
  }
  if (t < SPEC_MAX_TREE_NODES) {
    s_cq[t] = my_q0;
    s_cl[t] = my_logit;
  }
  if (wave == 0) {   // (the wavefront that writes over these: its own order is all that orders them)
    for (int k = lane; k < Lmax; k += 64) {
      path[(long)b * Lmax + k] = -1;
      out_tokens[(long)b * Lmax + k] = -1;
    }
  }
  lds_barrier();
  if (s_flag != 0) {
    if (t == 0) { len[b] = 0; set_status(status, b, SPEC_ST_BAD_TREE); }
    return;
  }
  if (t == 0) path[(long)b * Lmax] = 0;
  bool own = node_max == nullptr;
  if (!own && own_levels > 0) {   // (padding nodes count as levels too: the tree as the pass over all nodes sees it)
    const int32_t* par = parent + (long)b * N;
    own = tree_within(lane < N ? par[lane] : -1, lane + 64 < N ? par[lane + 64] : -1, own_levels);
  }
  // this lane's two nodes: (parent, place among the siblings) as one number, and P(x), un-normalised, while the walk is at the
  // parent
  const int c_key[2] = {s_par[lane] * SPEC_MAX_TREE_NODES + s_rank[lane], s_par[lane + 64] * SPEC_MAX_TREE_NODES + s_rank[lane + 64]};
  float c_p[2];

  int u = 0, k = 0, red = 0;
  bool have_row = own_levels > 0, have_weights = false;   // w holds node u's logits, its distribution
  float Z, mx;
  auto need_weights = [&]() {
    if (have_weights) return;
    if (!have_row) load_row(u);
#pragma unroll
    for (int j = 0; j < NG; ++j)
#pragma unroll
      for (int e = 0; e < VEC; ++e) w[j][e] = exp_of_nonpositive((w[j][e] - mx) * inv_temp);
    have_weights = true;
  };
  while (true) {
    if (own) {   // as the pass over all nodes takes them; w keeps the logits: most nodes need nothing else
      float m = -INFINITY, sum = 0.f;
#pragma unroll
      for (int j = 0; j < NG; ++j)
#pragma unroll
        for (int e = 0; e < VEC; ++e) m = fmaxf(m, w[j][e]);
      if (m > -INFINITY) {
#pragma unroll
        for (int j = 0; j < NG; ++j)
#pragma unroll
          for (int e = 0; e < VEC; ++e) sum += fast_exp((w[j][e] - m) * inv_temp);
      }
      block_softmax_stats(m, sum, inv_temp, s_stats[red ^= 1], &mx, &Z);
    } else {
      mx = node_max[(long)b * N + u];
      Z = node_sumexp[(long)b * N + u];
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) c_p[i] = exp_of_nonpositive((s_cl[lane + 64 * i] - mx) * inv_temp);
    bool accepted = false;
    for (int j = 0; k + 1 < Lmax; ++j) {
      const int key = u * SPEC_MAX_TREE_NODES + j;
      const unsigned long long m0 = __ballot(c_key[0] == key), m1 = __ballot(c_key[1] == key);
      if ((m0 | m1) == 0) break;   // no child left
      const bool high = m0 == 0;
      const int l = __ffsll((long long)(high ? m1 : m0)) - 1, c = l + (high ? 64 : 0);
      if (s_acc[c] * s_cq[c] <= readlane_f32(high ? c_p[1] : c_p[0], l) / Z) {
        accepted = true;
        if (t == 0) {
          out_tokens[(long)b * Lmax + k] = s_tok[c];
          path[(long)b * Lmax + k + 1] = c;
        }
        u = c;
        break;
      }
      // rejected: P := norm(max(0, P - Q)), kept as un-normalised values plus their sum Z
      const float* Q = probs_ssm + (long)uniform(s_row[c]) * V;
      float my_q[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) my_q[i] = (c_key[i] >> 7) == u ? Q[s_tok[lane + 64 * i]] : 0.f;
      need_weights();
      const float invZ = 1.f / Z;
      float part = 0.f;
      float q[NG][VEC];
#pragma unroll
      for (int jj = 0; jj < NG; ++jj) {
        const int gi = jj * SW_THREADS + t;
        if (gi < n_groups) {
          if (ODD) load_f32_group<VEC>(Q + (unsigned)group_start(gi, VEC, V), q[jj]);   // (what the last group repeats meets weights of 0)
          else load_f32_group<VEC>(Q + jj * SW_THREADS * VEC + (unsigned)(t * VEC), q[jj]);
        } else {
#pragma unroll
          for (int e = 0; e < VEC; ++e) q[jj][e] = 0.f;
        }
      }
#pragma unroll
      for (int jj = 0; jj < NG; ++jj)
#pragma unroll
        for (int e = 0; e < VEC; ++e) part += fmaxf(0.f, fmaf(w[jj][e], invZ, -q[jj][e]));
      const float Znew = block_total(part, s_red[red ^= 1]);
      if (Znew > 0.f) {
#pragma unroll
        for (int jj = 0; jj < NG; ++jj)
#pragma unroll
          for (int e = 0; e < VEC; ++e) w[jj][e] = fmaxf(0.f, fmaf(w[jj][e], invZ, -q[jj][e]));
        Z = Znew;
#pragma unroll
        for (int i = 0; i < 2; ++i) c_p[i] = fmaxf(0.f, fmaf(c_p[i], invZ, -my_q[i]));
      } else if (t == 0) {   // an empty residual keeps the previous P
        set_status(status, b, SPEC_ST_ZERO_RESIDUAL);
      }
    }
    if (!accepted) break;
    ++k;
    have_weights = false;
    have_row = own;
    if (own) load_row(u);
  }

  // ---- final token: inverse CDF in ascending token id over the current P. Order of the elements: group round, thread,
  // element. Float64: inclusive sums over the lanes per round, then over the (round, wavefront) totals.
  need_weights();
  auto group_sum = [&](int j) {
    double sum = 0.0;
#pragma unroll
    for (int e = 0; e < VEC; ++e) sum += (double)w[j][e];
    return sum;
  };
#pragma unroll
  for (int j = 0; j < NG; ++j) {
    const double incl = wave_inclusive_sum_f64(group_sum(j));
    if (lane == 63) s_tot[j * WAVES + wave] = incl;
  }
  if (t >= NG * WAVES && t < NTOT) s_tot[t] = 0.0;
  if (t == 0) s_ans = V - 1;
  __syncthreads();
  constexpr int EPL = NTOT / 64;   // totals per lane
  double mine = 0.0;
#pragma unroll
  for (int i = 0; i < EPL; ++i) mine += s_tot[lane * EPL + i];
  const double upto = wave_inclusive_sum_f64(mine);
  const double target = (double)u_final[b] * readlane_f64(upto, 63);
  const unsigned long long past = __ballot(upto > target);
  if (past != 0) {   // the first lane whose totals reach past the target, then the first of its totals
    const int f = __ffsll((long long)past) - 1;
    double before = f == 0 ? 0.0 : readlane_f64(upto, f - 1);
    int entry = f * EPL;
#pragma unroll
    for (int i = 0; i < EPL - 1; ++i) {
      const double next = before + s_tot[f * EPL + i];
      if (entry == f * EPL + i && next <= target) { before = next; ++entry; }
    }
    if (entry % WAVES == wave) {
      const int jr = entry / WAVES;
#pragma unroll
      for (int j = 0; j < NG; ++j) {
        if (j == jr) {
          const double sum = group_sum(j), incl = wave_inclusive_sum_f64(sum);
          const unsigned long long hit = __ballot(before + incl > target);
          const int fl = hit != 0 ? __ffsll((long long)hit) - 1 : 63;
          if (lane == fl) {
            const double run = before + incl - sum;
            const int first = ODD ? group_start(j * SW_THREADS + t, VEC, V) : (j * SW_THREADS + t) * VEC;
            int ans = first + VEC - 1;
#pragma unroll
            for (int e = VEC - 1; e >= 0; --e) {   // the first element whose running sum exceeds the target
              double upto_e = run;
#pragma unroll
              for (int i = 0; i <= e; ++i) upto_e += (double)w[j][i];
              if (upto_e > target) ans = first + e;
            }
            s_ans = min(ans, V - 1);
          }
        }
      }
    }
  }
  __syncthreads();
  if (t == 0) {
    out_tokens[(long)b * Lmax + k] = s_ans;
    len[b] = k + 1;
  }
}

// ---------------------------------------------------------------------------------------------
// stochastic walk with the residual in a buffer (vocabularies that do not fit the registers): blockDim = 1024
// ---------------------------------------------------------------------------------------------

// Weights of eight rounds of 64 groups from group `first` on, of which `hi` is the end: exp((logits[i] - mx) / T) or resid[i];
// 0 past the end.
template <bool BF16, int VEC>
__device__ __forceinline__ void weights_of(const void* __restrict__ logits, long lrow, const float* resid, bool implicit, float mx,
                                           float inv_temp, int V, int first, int stride, int hi, float (&w)[SWEEP_U][VEC]) {
  const int n_groups = (V + VEC - 1) / VEC;
  if (implicit) {
    LogitGroup<BF16, VEC> raw[SWEEP_U];
#pragma unroll
    for (int j = 0; j < SWEEP_U; ++j) {
      if (first + j * stride < hi) raw[j].load((const char*)logits + lrow * (BF16 ? 2 : 4), (unsigned)group_start(first + j * stride, VEC, V));
      else raw[j].set_minus_infinity();
    }
#pragma unroll
    for (int j = 0; j < SWEEP_U; ++j) {
      raw[j].expand(w[j]);
#pragma unroll
      for (int e = 0; e < VEC; ++e) w[j][e] = exp_of_nonpositive((w[j][e] - mx) * inv_temp);
    }
  } else {
#pragma unroll
    for (int j = 0; j < SWEEP_U; ++j) {
      if (first + j * stride < hi) {
        load_f32_group<VEC>(resid + group_start(first + j * stride, VEC, V), w[j]);
      } else {
#pragma unroll
        for (int e = 0; e < VEC; ++e) w[j][e] = 0.f;
      }
    }
  }
  if (V % VEC != 0) {
#pragma unroll
    for (int j = 0; j < SWEEP_U; ++j) drop_repeated<VEC>(w[j], first + j * stride, n_groups, V, 0.f);
  }
}

// Inverse-CDF draw by a block of SW_THREADS threads over V weights in ascending token id: every wavefront owns a run of groups
// and sums it, in float64, 64 groups side by side; the wavefront whose run holds the target r * total goes through its run again,
// 64 groups at a time. Returns, to every thread, the first index whose inclusive sum exceeds the target. (A run per thread, whose
// owner then read it element by element, took most of the walk: 8 trees of 32, 128256 float32, 177 us, 142 now; 4 trees of 16,
// 50257 float32 by single elements, 81, 50 now.)
template <bool BF16, int VEC>
__device__ inline int inverse_cdf_draw(const void* __restrict__ logits, long lrow, const float* resid, bool implicit,
                                       float mx, float inv_temp, int V, float r, double* s_scan, int* s_ans) {
  constexpr int WAVES = SW_THREADS / 64;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int n_groups = (V + VEC - 1) / VEC;
  const int run_groups = (n_groups + 64 * WAVES - 1) / (64 * WAVES) * 64;   // per wavefront, whole rounds
  const int lo = min(wave * run_groups, n_groups), hi = min(lo + run_groups, n_groups);
  float w[SWEEP_U][VEC];
  double mine = 0.0;
  for (int g0 = lo; g0 < hi; g0 += 64 * SWEEP_U) {
    weights_of<BF16, VEC>(logits, lrow, resid, implicit, mx, inv_temp, V, g0 + lane, 64, hi, w);
#pragma unroll
    for (int j = 0; j < SWEEP_U; ++j)
#pragma unroll
      for (int e = 0; e < VEC; ++e) mine += (double)w[j][e];
  }
  const double incl = wave_inclusive_sum_f64(mine);
  __syncthreads();   // earlier readers of the shared slots are done
  if (lane == 63) s_scan[wave] = incl;
  if (t == 0) *s_ans = V - 1;
  __syncthreads();
  double total = 0.0;
  for (int i = 0; i < WAVES; ++i) total += s_scan[i];
  const double target = (double)r * total;
  double before = 0.0;
  int owner = -1;
  for (int i = 0; i < WAVES; ++i) {
    if (owner < 0 && before + s_scan[i] > target) owner = i;
    if (owner < 0) before += s_scan[i];
  }
  if (wave == owner) {
    if (lane == 0) *s_ans = min(hi * VEC, V) - 1;   // (if rounding leaves none)
    bool found = false;
    for (int g0 = lo; g0 < hi && !found; g0 += 64 * SWEEP_U) {
      weights_of<BF16, VEC>(logits, lrow, resid, implicit, mx, inv_temp, V, g0 + lane, 64, hi, w);
#pragma unroll
      for (int j = 0; j < SWEEP_U; ++j) {
        if (!found) {
          double sum = 0.0;
#pragma unroll
          for (int e = 0; e < VEC; ++e) sum += (double)w[j][e];
          const double upto = wave_inclusive_sum_f64(sum);
          const unsigned long long hit = __ballot(before + upto > target);
          if (hit != 0) {
            found = true;
            if (lane == __ffsll((long long)hit) - 1) {
              double run = before + upto - sum;
              const int first = group_start(g0 + j * 64 + lane, VEC, V);
              int ans = first + VEC - 1;
              bool past = false;
#pragma unroll
              for (int e = 0; e < VEC; ++e) {
                run += (double)w[j][e];
                if (!past && run > target) { ans = first + e; past = true; }
              }
              *s_ans = ans;
            }
          } else {
            before += readlane_f64(upto, 63);
          }
        }
      }
    }
  }
  __syncthreads();
  return *s_ans;
}

template <bool BF16, int VEC>
__global__ void __launch_bounds__(SW_THREADS) stochastic_walk_kernel(
    int N, int V, const void* __restrict__ logits, const float* __restrict__ probs_ssm, int R,
    const int32_t* __restrict__ ssm_row, const int32_t* __restrict__ token, const int32_t* __restrict__ parent,
    const float* __restrict__ u_accept, const float* __restrict__ u_order, const float* __restrict__ u_final,
    float inv_temp, const float* __restrict__ node_max, const float* __restrict__ node_sumexp, float* resid_all, int Lmax,
    int32_t* __restrict__ path, int32_t* __restrict__ len, int32_t* __restrict__ out_tokens, int32_t* status) {
  __shared__ int s_flag;
  __shared__ int s_child[SPEC_MAX_TREE_NODES];
  __shared__ int s_sorted[SPEC_MAX_TREE_NODES];
  __shared__ int s_cx[SPEC_MAX_TREE_NODES];       // per child in test order: its token,
  __shared__ float s_cq[SPEC_MAX_TREE_NODES];     // the draft's probability of that token,
  __shared__ float s_cl[SPEC_MAX_TREE_NODES];     // the LLM's logit of that token at u,
  __shared__ float s_cr[SPEC_MAX_TREE_NODES];     // and the child's uniform
  __shared__ int s_nchild;
  __shared__ float s_fsum[SW_THREADS / 64];
  __shared__ double s_scan[SW_THREADS / 64];
  __shared__ int s_ans;

  const int b = blockIdx.x, t = threadIdx.x;
  float* resid0 = resid_all + (long)b * V;
  float* resid1 = resid_all + ((long)gridDim.x + b) * V;
  float* resid = resid0;
  int cur = 0;   // resid == (cur ? resid1 : resid0)
  const int32_t* par = parent + (long)b * N;
  const int32_t* tok = token + (long)b * N;
  const int n_groups = (V + VEC - 1) / VEC;

  bool valid = tree_is_valid(par, N, &s_flag);
  __syncthreads();
  if (t == 0) s_flag = 0;
  __syncthreads();
  if (valid && t >= 1 && t < N) {   // a negative token marks a padding node: never a candidate, nothing to check
    const int x = tok[t], r = ssm_row[(long)b * N + t];
    if (x >= 0 && (x >= V || r < 0 || r >= R)) atomicOr(&s_flag, 1);
  }
  __syncthreads();
  valid = valid && (s_flag == 0);
  for (int k = t; k < Lmax; k += SW_THREADS) {
    path[(long)b * Lmax + k] = -1;
    out_tokens[(long)b * Lmax + k] = -1;
  }
  if (!valid) {
    if (t == 0) { len[b] = 0; set_status(status, b, SPEC_ST_BAD_TREE); }
    return;
  }
  __syncthreads();
  if (t == 0) path[(long)b * Lmax] = 0;

  int u = 0, k = 0;
  bool implicit = true;   // current P is softmax(logits[u]) given by (node_max, node_sumexp); else resid / Z
  float Z = 1.f;
  float mx = node_max[(long)b * N], se = node_sumexp[(long)b * N];
  while (true) {
    // children of u in ascending (u_order, index)
    if (t == 0) s_nchild = 0;
    __syncthreads();
    if (t < N && par[t] == u && tok[t] >= 0) s_child[atomicAdd(&s_nchild, 1)] = t;
    __syncthreads();
    const int nchild = (k + 1 < Lmax) ? s_nchild : 0;
    if (nchild == 0) break;
    if (t < nchild) {
      const int me = s_child[t];
      const float mk = u_order[(long)b * N + me];
      int rank = 0;
      for (int j = 0; j < nchild; ++j) {
        const int o = s_child[j];
        const float ok = u_order[(long)b * N + o];
        rank += (ok < mk) || (ok == mk && o < me);
      }
      s_sorted[rank] = me;
    }
    __syncthreads();
    bool accepted = false;
    int next_u = -1;
    const long lrow = ((long)b * N + u) * V;
    // everything a ratio test needs from memory, for all children at once (one round trip instead of one
    // chain of dependent loads per test)
    if (t < nchild) {
      const int s = s_sorted[t];
      const int x = tok[s];
      s_cx[t] = x;
      s_cq[t] = probs_ssm[(long)ssm_row[(long)b * N + s] * V + x];
      s_cl[t] = load_logit<BF16>(logits, lrow + x);
      s_cr[t] = u_accept[(long)b * N + s];
    }
    __syncthreads();
    for (int j = 0; j < nchild; ++j) {
      const int s = s_sorted[j];
      const int x = s_cx[j];
      const float* Q = probs_ssm + (long)ssm_row[(long)b * N + s] * V;
      const float r = s_cr[j];
      float px;
      if (implicit) px = exp_of_nonpositive((s_cl[j] - mx) * inv_temp) / se;
      else px = resid[x] / Z;
      if (r * s_cq[j] <= px) {
        accepted = true;
        next_u = s;
        if (t == 0) {
          out_tokens[(long)b * Lmax + k] = x;
          path[(long)b * Lmax + k + 1] = s;
        }
        break;
      }
      // rejected: P := norm(max(0, P - Q)), kept as un-normalised values plus their sum Z. The new
      // residual goes to the other buffer, so an empty residual simply keeps the previous P.
      float* dst = cur ? resid0 : resid1;
      float part = 0.f;
      const float invZ = 1.f / Z, inv_se = 1.f / se;
      for (int g0 = 0; g0 < n_groups; g0 += SW_THREADS * SWEEP_U) {
        float pv[SWEEP_U][VEC], qv[SWEEP_U][VEC];
#pragma unroll
        for (int jj = 0; jj < SWEEP_U; ++jj) {
          const int gi = g0 + jj * SW_THREADS + t;
          if (gi < n_groups) load_f32_group<VEC>(Q + group_start(gi, VEC, V), qv[jj]);
        }
        weights_of<BF16, VEC>(logits, lrow, resid, implicit, mx, inv_temp, V, g0 + t, SW_THREADS, n_groups, pv);
        const float scale = implicit ? inv_se : invZ;
#pragma unroll
        for (int jj = 0; jj < SWEEP_U; ++jj) {
          const int gi = g0 + jj * SW_THREADS + t;
          if (gi < n_groups) {
            const int at = group_start(gi, VEC, V), repeated = gi * VEC - at;   // (elements of the group before: no weight here)
            float d[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
              d[e] = fmaxf(0.f, pv[jj][e] * scale - qv[jj][e]);
              part += d[e];
            }
            if (repeated == 0) {
              store_f32_group<VEC>(dst + at, d);
            } else {
#pragma unroll
              for (int e = 0; e < VEC; ++e)
                if (e >= repeated) dst[at + e] = d[e];
            }
          }
        }
      }
      const float Znew = block_sum(part, s_fsum);
      if (Znew > 0.f) {
        Z = Znew;
        implicit = false;
        resid = dst;
        cur ^= 1;
      } else if (t == 0) {
        set_status(status, b, SPEC_ST_ZERO_RESIDUAL);
      }
      __syncthreads();   // the new residual is visible to every thread before the next test reads it
    }
    if (!accepted) break;
    u = next_u;
    ++k;
    implicit = true;
    resid = resid0;
    cur = 0;
    mx = node_max[(long)b * N + u];
    se = node_sumexp[(long)b * N + u];
    __syncthreads();
  }

  // final token: inverse CDF in ascending token id over the current P
  const int ans = inverse_cdf_draw<BF16, VEC>(logits, ((long)b * N + u) * V, resid, implicit, mx, inv_temp, V, u_final[b],
                                              s_scan, &s_ans);
  if (t == 0) {
    out_tokens[(long)b * Lmax + k] = ans;
    len[b] = k + 1;
  }
}

// ---------------------------------------------------------------------------------------------
// naive sampling (Section 4.3): x_u ~ softmax(logits[u] / T) for every node at once, one block per
// (request, node) row, by inverse CDF with the caller's uniform. The walk that follows is the greedy
// walk on these tokens: move to the child whose token equals x_u, else emit x_u and stop.
// ---------------------------------------------------------------------------------------------
template <bool BF16, int VEC>
__global__ void __launch_bounds__(SW_THREADS) node_sample_kernel(const void* __restrict__ logits, int V, float inv_temp,
                                                                 const float* __restrict__ node_max,
                                                                 const float* __restrict__ u_sample,
                                                                 int32_t* __restrict__ node_sample) {
  __shared__ double s_scan[SW_THREADS / 64];
  __shared__ int s_ans;
  const long row = blockIdx.x;
  const int ans = inverse_cdf_draw<BF16, VEC>(logits, row * V, nullptr, true, node_max[row], inv_temp, V, u_sample[row],
                                              s_scan, &s_ans);
  if (threadIdx.x == 0) node_sample[row] = ans;
}

// ---------------------------------------------------------------------------------------------
// Whether the arg-max takes its rows by half sweeps. An odd number of halves: yes, the last half sweep would be loaded for nothing
// (us, whole / halves, workgroups of 1024: 320 rows of 45232 float32 16.2 / 15.5, 4 rows 7.5 / 7.1; 480 of 80000 bfloat16 19.9 / 17.3; one
// row of 32000 bfloat16 6.7 / 6.1; of 256: 2000 rows of 40000 bfloat16 32.0 / 31.4). An even one: no, the fewer instructions tell (300 rows
// of 17000 float32 10.0 / 10.6, of 100000 bfloat16 16.8 / 17.6, 4 rows of it 8.4 / 8.8; 16 of 128256 bfloat16 8.6 / 8.9), but for
// float32 rows of two sweeps and more, one for every second compute unit and above, which are bound by memory (65536: 128 rows 11.4 /
// 11.1, 300 rows 19.7 / 18.6, 16 rows 7.7 / 7.85).
static bool argmax_by_halves(int rows, int V, bool bf16, int threads) {
  const int half = threads * SWEEP_U / 2 * (bf16 ? 8 : 4), halves = (V + half - 1) / half;
  return halves % 2 == 1 || (!bf16 && threads == 1024 && halves >= 4 && rows >= compute_units() / 2);
}

hipError_t launch_node_stats(int B, int N, int V, int logits_dtype, const void* logits, float inv_temp,
                             int32_t* node_argmax, float* node_max, float* node_sumexp, hipStream_t s,
                             const int32_t* parent, int own_levels) {
  const bool bf16 = logits_dtype == SPEC_BF16;
  // 256 threads where there are a thousand rows or more (see above), and for rows that they take in one go: four wavefronts'
  // results are merged sooner than sixteen's (440 rows of 1051 bfloat16 with the walk: 8.35 us, 6.55 now)
  const bool many = (long)B * N >= 1024;
  if (node_sumexp == nullptr && V >= (bf16 ? 8 : 4)) {   // (the entry points require 16-byte aligned logits)
    const bool small = many || V <= 256 * SWEEP_U * (bf16 ? 8 : 4) / 2;
    const int form = V % (bf16 ? 8 : 4) != 0 ? 2 : argmax_by_halves(B * N, V, bf16, small ? 256 : 1024) ? 1 : 0;
#define SPEC_NA_F(BF, NT, OD, HA) \
  hipLaunchKernelGGL((node_argmax_kernel<BF, NT, OD, HA>), dim3(B * N), dim3(NT), 0, s, logits, V, node_argmax, node_max)
#define SPEC_NA(BF, NT)                              \
  do {                                               \
    if (form == 2) SPEC_NA_F(BF, NT, true, true);    \
    else if (form == 1) SPEC_NA_F(BF, NT, false, true); \
    else SPEC_NA_F(BF, NT, false, false);            \
  } while (0)
    if (bf16) { if (small) SPEC_NA(true, 256); else SPEC_NA(true, 1024); }
    else { if (small) SPEC_NA(false, 256); else SPEC_NA(false, 1024); }
#undef SPEC_NA
#undef SPEC_NA_F
    return hipGetLastError();
  }
#define SPEC_NS_U(BF, VE, NT, U)                                                                                         \
  hipLaunchKernelGGL((node_stats_kernel<BF, VE, NT, U>), dim3(B * N), dim3(NT), 0, s, logits, V, inv_temp, node_argmax,   \
                     node_max, node_sumexp, parent, N, own_levels)
#define SPEC_NS(BF, NT)                              \
  do {                                               \
    if (V <= 2 * 4 * NT) SPEC_NS_U(BF, 4, NT, 2);    \
    else if (V <= 4 * 4 * NT) SPEC_NS_U(BF, 4, NT, 4); \
    else SPEC_NS_U(BF, 4, NT, SWEEP_U);              \
  } while (0)
  const bool small = many || V <= 256 * SWEEP_U * 4 / 2;
  if (V < 4) { if (bf16) SPEC_NS_U(true, 1, 256, 2); else SPEC_NS_U(false, 1, 256, 2); }
  else if (bf16) { if (small) SPEC_NS(true, 256); else SPEC_NS(true, 1024); }
  else { if (small) SPEC_NS(false, 256); else SPEC_NS(false, 1024); }
#undef SPEC_NS_U
#undef SPEC_NS
  return hipGetLastError();
}

hipError_t launch_node_sample(int B, int N, int V, int logits_dtype, const void* logits, float inv_temp,
                              const float* node_max, const float* u_sample, int32_t* node_sample, hipStream_t s) {
  const bool bf16 = logits_dtype == SPEC_BF16;
#define SPEC_NSM(BF, VE)                                                                                          \
  hipLaunchKernelGGL((node_sample_kernel<BF, VE>), dim3(B * N), dim3(SW_THREADS), 0, s, logits, V, inv_temp, node_max, \
                     u_sample, node_sample)
  if (V < 4) { if (bf16) SPEC_NSM(true, 1); else SPEC_NSM(false, 1); }
  else if (bf16) SPEC_NSM(true, 4);
  else SPEC_NSM(false, 4);
#undef SPEC_NSM
  return hipGetLastError();
}

hipError_t launch_greedy_walk(int B, int N, const int32_t* node_argmax, const int32_t* token, const int32_t* parent,
                              int Lmax, int32_t* path, int32_t* len, int32_t* out_tokens, int32_t* status,
                              hipStream_t s) {
  hipLaunchKernelGGL(greedy_walk_kernel, dim3(B), dim3(64), 0, s, N, node_argmax, token, parent, Lmax, path, len,
                     out_tokens, status);
  return hipGetLastError();
}

hipError_t launch_stochastic_walk(int B, int N, int V, int logits_dtype, const void* logits, const float* probs_ssm,
                                  int R, const int32_t* ssm_row, const int32_t* token, const int32_t* parent,
                                  const float* u_accept, const float* u_order, const float* u_final, float inv_temp,
                                  const float* node_max, const float* node_sumexp, float* resid, int Lmax,
                                  int32_t* path, int32_t* len, int32_t* out_tokens, int32_t* status, hipStream_t s,
                                  int own_levels) {
  const bool bf16 = logits_dtype == SPEC_BF16;
  if (stochastic_walk_in_registers(V)) {
#define SPEC_SWR_O(BF, VE, NGR, OD)                                                                                         \
  hipLaunchKernelGGL((stochastic_walk_reg_kernel<BF, VE, NGR, OD>), dim3(B), dim3(SW_THREADS), 0, s, N, V, logits, probs_ssm, \
                     R, ssm_row, token, parent, u_accept, u_order, u_final, inv_temp, node_max, node_sumexp, own_levels,  \
                     Lmax, path, len, out_tokens, status)
#define SPEC_SWR(BF, VE, NGR)                                                                      \
  do {                                                                                              \
    if (V % VE != 0) SPEC_SWR_O(BF, VE, NGR, true); else SPEC_SWR_O(BF, VE, NGR, false);            \
  } while (0)
  // (registers for twice the vocabulary at most: rounds past its end cost as much as the others)
#define SPEC_SWR_T(BF)                                          \
  if (V < 4) SPEC_SWR_O(BF, 1, 1, false);                       \
  else if (V <= SW_THREADS * 4) SPEC_SWR(BF, 4, 1);             \
  else if (V <= SW_THREADS * 8) SPEC_SWR(BF, 4, 2);             \
  else if (V <= SW_THREADS * 16) SPEC_SWR(BF, 4, 4);            \
  else SPEC_SWR(BF, 4, 8)
    if (bf16) { SPEC_SWR_T(true); } else { SPEC_SWR_T(false); }
#undef SPEC_SWR_T
#undef SPEC_SWR
#undef SPEC_SWR_O
    return hipGetLastError();
  }
#define SPEC_SW(BF, VE)                                                                                              \
  hipLaunchKernelGGL((stochastic_walk_kernel<BF, VE>), dim3(B), dim3(SW_THREADS), 0, s, N, V, logits, probs_ssm, R,    \
                     ssm_row, token, parent, u_accept, u_order, u_final, inv_temp, node_max, node_sumexp, resid, Lmax, \
                     path, len, out_tokens, status)
  if (bf16) SPEC_SW(true, 4); else SPEC_SW(false, 4);   // (a vocabulary this large)
#undef SPEC_SW
  return hipGetLastError();
}

}  // namespace spec
