// LM head in front of the greedy verifier (Algorithm 2, VerifyGreedy: O(u) is the arg-max of the LLM's
// distribution at node u, so for greedy decoding the logits [B*N, V] never have to exist in memory):
//     node_argmax[m] = argmax_v  sum_k hidden[m, k] * weight[v, k]        (lowest v on ties)
// bf16 inputs, float32 accumulation on the matrix cores. With the few hundred rows a verification pass has
// (M = B*N), the product is bound by streaming the weight matrix once from HBM (V x K x 2 bytes, 262 MB for
// a 32000 x 4096 head), not by arithmetic.
//
// lm_head_argmax_kernel: a workgroup of four wavefronts owns 128 (64 for small vocabularies) vocabulary rows and up to
// 256 rows of `hidden` (MT = 32 to 256). Both operands go from global memory straight into LDS (global_load_lds_dwordx4) in
// stages of 64 k, 16 (8) KB of W and MT rows of `hidden` (L2-resident), into a ring of as many stages as fit: two (256 rows)
// to five (32 rows) stages of 16 KB of W, or two workgroups' four stages of 8 KB, are in flight per compute unit while one
// is multiplied, to cover the two microseconds of loaded latency. A lane's 16 bytes land at a fixed place, so the swizzle
// that keeps the operand reads off each other's banks is applied to the source: slot s of row r holds the 16-byte piece
// s ^ ((r >> 1) & 7) of the row. The product is taken transposed, C[v, m] on 32 x 32 x 16 tiles, so a lane ends up with 16
// vocabulary entries of ONE row m per tile and the arg-max over v is in the lane, one cross-lane step and one pass through
// LDS over the wavefronts. Each workgroup writes its (max, arg-max) per row; lm_head_reduce_kernel merges a row's partials
// (one per workgroup).
//
// What bounds it: the stream of W. Nothing but these loads takes 45.3 us for 32000 x 4096 (5.8 TB/s), 52.7 without the
// non-temporal hint, when every workgroup reads the same k of rows that lie 8 KB apart. Starting each workgroup at another k
// takes 39.5, but equal rows of W in different workgroups must not be summed in different orders: they could differ in the last bit,
// which the arg-max rule (lowest token among equal logits) does not allow. A logit is therefore cut into two sums, and half of the
// workgroups take them in the other order (see APART and the rule at its launch). Measured at 32000 x 4096 with six weight
// matrices in turn (1.6 GB: W comes from HBM every time), with logits and statistics and the merge, us, in step / apart: 16 rows
// 54.8 / 48.2, 128 rows 61.5 / 57.3, 250 rows 87.8 / 87.3. Of 4.1 million logits 1109 (in step) and 1084 (apart) are not the nearest
// bfloat16 to the sum in float64. Up to 32 rows of K = 256 to 512 over 4000 to 8000 vocabulary rows take up to 4 % (0.3 us) longer
// than they did.
// The order of a logit's sum is a matter of V and K alone, so that a row of `hidden` has the same logits in a batch of any
// size: the 64 x 32 tile (up to 32 rows, vocabularies up to 16384 on 256 compute units) has two wavefronts for each place of
// the product, which sum every other pair of k-steps, and where it is in use the other tiles keep the same two sums
// (TWO; 8000 x 4096, 64 / 128 / 256 rows, arg-max only: 27.0 / 33.3 / 34.2 us with one sum, 27.0 / 34.3 / 35.6 with two; the
// 64 x 32 tile without the second pair of wavefronts takes 28.0 instead of 19.0 for one row).
// More than 256 rows of `hidden` take several slices; the slices of one vocabulary tile are numbered eight apart, which
// puts them on one XCD at the same time, so W is fetched once for all of them.
#include <hip/hip_bf16.h>

#include <algorithm>

#include "spec_internal.h"

namespace spec {
namespace lmh {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

constexpr int KC = 64;                        // k per ring stage
constexpr int ROWB = KC * 2;                  // LDS bytes per row of a stage
constexpr int NTHREADS = 256;
constexpr int HEAD = 16;                      // stages (2 KB of a row) that workgroups are apart where the sums are cut there

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
template <int N>
__device__ __forceinline__ void wait_loads_but() {   // at most N vector memory operations of this lane still in flight
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// 16 bytes per lane from global memory to LDS address lds_dst + 16 * lane (lds_dst wave-uniform). W is read once per launch
// (NT: non-temporal), `hidden` by every workgroup.
template <bool NT>
__device__ __forceinline__ void load_to_lds(const unsigned char* src, unsigned lds_dst) {
  if (NT) asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(src), "s"(lds_dst) : "memory");
  else asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_dst) : "memory");
}

// (value desc, index asc): does (v2, i2) beat (v1, i1)?
__device__ __forceinline__ bool beats(float v2, int i2, float v1, int i1) { return v2 > v1 || (v2 == v1 && i2 < i1); }

// STATS: the logits are also written out, rounded to bf16, and every partial carries the sum of
// exp((x - max) / T) over the workgroup's vocabulary rows - of the ROUNDED values, which are what a verifier
// reading those logits will see (maximum and arg-max are then those of the rounded values too).
// RING_KB: the ring's share of the LDS. 128: one workgroup per compute unit with as many stages in flight as fit; 64 (up to 32
// rows): two workgroups, whose starts and ends overlap.
// APART: a logit is the sum over the first HEAD stages of k plus that over the others, and every other sixteen workgroups (two of an
// XCD's) start with the others: a sum of two does not depend on its order, so equal rows of W have equal logits wherever they lie.
template <int VT, int MT, int RING_KB, bool TWO, bool APART, bool STATS>
__global__ void __launch_bounds__(NTHREADS, RING_KB == 64 ? 2 : 1) lm_head_argmax_kernel(const __hip_bfloat16* __restrict__ hidden,
                                                                    const __hip_bfloat16* __restrict__ weight,
                                                                    float* __restrict__ part_val, int32_t* __restrict__ part_idx,
                                                                    float* __restrict__ part_sum,
                                                                    __hip_bfloat16* __restrict__ logits_out, float inv_temp_log2,
                                                                    int M, int K, int V, int n_vtiles, int slices_per_row) {
  constexpr int WV = VT / 32 < (MT >= 128 ? 2 : 4) ? VT / 32 : (MT >= 128 ? 2 : 4);   // wavefronts along v,
  constexpr int WM = MT / 32 < 4 / WV ? MT / 32 : 4 / WV, KW = 4 / (WV * WM);         // along m, and along the k of a stage
  constexpr int SUMS = TWO && KW == 1 ? 2 : 1;
  constexpr int TV = VT / WV / 32, TM = MT / WM / 32;               // 32 x 32 tiles of a wavefront
  constexpr int W_BYTES = VT * ROWB, STAGE = W_BYTES + MT * ROWB;
  constexpr int NST = MT == 256 ? 3 : (RING_KB << 10) / STAGE < 8 ? (RING_KB << 10) / STAGE : 8, AHEAD = NST - 1;
  constexpr int WL = VT / 32, HL = MT / 32, LPS = WL + HL;          // loads per lane and stage: 32 rows of eight pieces each
  constexpr int CROW = VT * 2 + 16;                                 // LDS bytes per row of the logits on their way out
  static_assert(MT * CROW <= NST * STAGE, "the logits reuse the ring");
  __shared__ __attribute__((aligned(16))) unsigned char ring[NST * STAGE];
  __shared__ float s_val[WV][MT];
  __shared__ int s_idx[WV][MT];
  __shared__ float s_sum[STATS ? WV : 1][MT];
  __shared__ float s_part[KW == 2 ? WV * WM * TV * TM * 16 * 64 : 1];

  const int blk = uniform(blockIdx.x / (8 * slices_per_row)), in_blk = blockIdx.x - blk * 8 * slices_per_row;
  const int vt = blk * 8 + in_blk % 8, slice = blockIdx.y * slices_per_row + in_blk / 8;
  if (vt >= n_vtiles || (long)slice * MT >= M) return;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wv = wave / WM % WV, wm = wave % WM, kw = wave / (WV * WM);
  static_assert(KW == 1 || (KW == 2 && TWO), "at most two sums per logit");
  const int r = lane & 31, h = lane >> 5;
  const int v0 = vt * VT, m0 = slice * MT;
  const int NC = K / KC;

  // loader: row j * 32 + t / 8 of the stage's W (and hidden) part, 16-byte slot t % 8; rows past the end repeat the last
  // (their results are masked or not written)
  const int piece = (t & 7) ^ ((t >> 4) & 7);
  const unsigned char *wsrc[WL], *hsrc[HL];
#pragma unroll
  for (int j = 0; j < WL; ++j) wsrc[j] = (const unsigned char*)(weight + (long)min(v0 + j * 32 + (t >> 3), V - 1) * K) + piece * 16;
#pragma unroll
  for (int j = 0; j < HL; ++j) hsrc[j] = (const unsigned char*)(hidden + (long)min(m0 + j * 32 + (t >> 3), M - 1) * K) + piece * 16;
  const unsigned wave_lds = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)ring + wave * 1024;
  // stages are requested in the order of their use: from `start` to the end, then from 0
  const bool turned = APART && ((vt >> 4) & 1) != 0;
  const int start = turned ? HEAD : 0;
  int next = start;
  // 64 x 64 tiles in step take the stage's number c from the loop: a counter of their own holds them up (us, counter / loop / before there was a
  // counter: 40 rows, 8192 x 3000 40.8 / 38.9 / 39.3, 4096 x 8000 26.6 / 26.1 / 26.5); other tiles gain from it
  // (300 rows, 8192 x 16500 165.5 / 170.3 / 170.9; 20 rows 74.9 / 78.7 / 76.4).
  constexpr bool COUNTED = APART || VT != 64 || MT != 64;
  auto issue = [&](int c, int slot) {
    const unsigned dst = wave_lds + slot * STAGE;
    const long k = (long)(COUNTED ? next : c) * ROWB;
    if (COUNTED) ++next;
    if (APART && next == NC) next = 0;
#pragma unroll
    for (int j = 0; j < HL; ++j) load_to_lds<false>(hsrc[j] + k, dst + W_BYTES + j * 4096);
#pragma unroll
    for (int j = 0; j < WL; ++j) load_to_lds<true>(wsrc[j] + k, dst + j * 4096);
  };
#pragma unroll
  for (int c = 0; c < AHEAD; ++c)
    if (c < NC) issue(c, c);

  // TWO: a logit is the sum of two, over the first and over the second two k-steps of every stage. The tile of 64 x 32 gives
  // them to two wavefronts. Where that tile serves the smallest M (V and K decide), the others take the same two sums, so that
  // a row of `hidden` has the same logits whatever M is.
  f32x16 sums[SUMS][TV][TM];
#pragma unroll
  for (int p = 0; p < SUMS; ++p)
#pragma unroll
    for (int tv = 0; tv < TV; ++tv)
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int i = 0; i < 16; ++i) sums[p][tv][tm][i] = 0.f;
  // operand of this wavefront's k-step ks: row r of a 32-row tile, piece 2 k-step + h (the swizzle depends on r alone)
  unsigned off[4 / KW];
#pragma unroll
  for (int ks = 0; ks < 4 / KW; ++ks) off[ks] = r * ROWB + (((2 * (kw * (4 / KW) + ks) + h) ^ ((r >> 1) & 7)) << 4);

  static_assert(!APART || SUMS == 1, "one sum per logit at a time");
  int slot = 0, c = 0;
  f32x16 sum_before[APART ? TV : 1][APART ? TM : 1];
#pragma unroll
  for (int part = 0; part < (APART ? 2 : 1); ++part) {
    for (const int end = !APART || part == 1 ? NC : turned ? NC - HEAD : HEAD; c < end; ++c) {
      if (c + AHEAD <= NC) wait_loads_but<(AHEAD - 1) * LPS>();
      else wait_loads_but<0>();
      lds_barrier();   // stage c has landed for every lane, and every wavefront is done with stage c - 1, whose slot is free
      if (c + AHEAD < NC) issue(c + AHEAD, slot == 0 ? NST - 1 : slot - 1);
      const unsigned char* ws = ring + slot * STAGE + wv * TV * 32 * ROWB;
      const unsigned char* hs = ring + slot * STAGE + W_BYTES + wm * TM * 32 * ROWB;
#pragma unroll
      for (int ks = 0; ks < 4 / KW; ++ks) {
        bf16x8 a[TV], b[TM];
#pragma unroll
        for (int tv = 0; tv < TV; ++tv) a[tv] = *(const bf16x8*)(ws + tv * 32 * ROWB + off[ks]);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) b[tm] = *(const bf16x8*)(hs + tm * 32 * ROWB + off[ks]);
#pragma unroll
        for (int tv = 0; tv < TV; ++tv)
#pragma unroll
          for (int tm = 0; tm < TM; ++tm)
            sums[ks / 2 % SUMS][tv][tm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[tv], b[tm], sums[ks / 2 % SUMS][tv][tm], 0, 0, 0);
      }
      slot = slot == NST - 1 ? 0 : slot + 1;
    }
    if constexpr (APART) {
#pragma unroll
      for (int tv = 0; tv < TV; ++tv)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
          f32x16& sum = sums[0][tv][tm];
          if (part == 0) {
            sum_before[tv][tm] = sum;
#pragma unroll
            for (int i = 0; i < 16; ++i) sum[i] = 0.f;
          } else {
            sum += sum_before[tv][tm];
          }
        }
    }
  }

  f32x16 (&acc)[TV][TM] = sums[0];
  if constexpr (SUMS == 2) {
#pragma unroll
    for (int tv = 0; tv < TV; ++tv)
#pragma unroll
      for (int tm = 0; tm < TM; ++tm) acc[tv][tm] += sums[1][tv][tm];
  }
  if constexpr (KW == 2) {   // the second wavefront hands its sums over
    float* part = s_part + ((wv * WM + wm) * TV * TM * 16) * 64 + lane;   // [wave tiles][i][lane]
#pragma unroll
    for (int tv = 0; tv < TV; ++tv)
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (kw > 0) part[((tv * TM + tm) * 16 + i) * 64] = acc[tv][tm][i];
    lds_barrier();
    if (kw == 0) {
#pragma unroll
      for (int tv = 0; tv < TV; ++tv)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[tv][tm][i] += part[((tv * TM + tm) * 16 + i) * 64];
    }
  }

  // ---- tile (tv, tm): the lane holds row m0 + (wm TM + tm) 32 + r, vocabulary rows v0 + (wv TV + tv) 32 + 8 (i / 4) + 4 h + i % 4
  if (STATS) {   // round to the stored type first: statistics and arg-max are those of the stored logits
    if (KW == 1) lds_barrier();   // every wavefront is done with the ring: the logits go through it, to leave as whole rows
    if (kw == 0)
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int tv = 0; tv < TV; ++tv)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          union { uint2 u; __hip_bfloat16 h4[4]; } pk;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            pk.h4[i] = __float2bfloat16(acc[tv][tm][i4 * 4 + i]);
            acc[tv][tm][i4 * 4 + i] = __bfloat162float(pk.h4[i]);
          }
          *(uint2*)(ring + ((wm * TM + tm) * 32 + r) * CROW + ((wv * TV + tv) * 32 + i4 * 8 + 4 * h) * 2) = pk.u;
        }
    lds_barrier();
    const int rows = min(MT, M - m0), cols = min(VT, V - v0);
    // Rows of an odd vocabulary start on any even byte: the 16-byte stores may be unaligned, which the hardware takes
    // (one element per store cost 17 us of 78 at 50257 x 2304, 128 rows).
    struct __attribute__((packed, aligned(2))) Piece { u32x4 v; };
    for (int i = t; i < rows * (VT / 8); i += NTHREADS) {
      const int m = i / (VT / 8), c = (i % (VT / 8)) * 8;
      __hip_bfloat16* dst = logits_out + (long)(m0 + m) * V + v0 + c;
      const unsigned char* src = ring + m * CROW + c * 2;
      if (c + 8 <= cols) ((Piece*)dst)->v = *(const u32x4*)src;
      else
        for (int e = c; e < cols; ++e) dst[e - c] = *(const __hip_bfloat16*)(src + (e - c) * 2);
    }
  }
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
    float best = -INFINITY;
    int best_i = 0x7fffffff;
#pragma unroll
    for (int tv = 0; tv < TV; ++tv)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int v = v0 + (wv * TV + tv) * 32 + 8 * (i / 4) + 4 * h + i % 4;
        if (v < V && acc[tv][tm][i] > best) { best = acc[tv][tm][i]; best_i = v; }   // ascending v: the lowest wins ties
      }
    {
      const float ov = __shfl_xor(best, 32);
      const int oi = __shfl_xor(best_i, 32);
      if (beats(ov, oi, best, best_i)) { best = ov; best_i = oi; }
    }
    float sum = 0.f;
    if (STATS) {   // sum of exp((x - best) / T) over the wavefront's vocabulary rows (best: the wavefront's maximum)
      if (best > -INFINITY) {
#pragma unroll
        for (int tv = 0; tv < TV; ++tv)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (v0 + (wv * TV + tv) * 32 + 8 * (i / 4) + 4 * h + i % 4 < V)
              sum += __builtin_amdgcn_exp2f((acc[tv][tm][i] - best) * inv_temp_log2);
      }
      sum += __shfl_xor(sum, 32);
    }
    if (h == 0 && kw == 0) {
      const int m = (wm * TM + tm) * 32 + r;
      s_val[wv][m] = best;
      s_idx[wv][m] = best_i;
      if (STATS) s_sum[wv][m] = sum;
    }
  }
  __syncthreads();
  if (t < MT && m0 + t < M) {
    float best = s_val[0][t];
    int best_i = s_idx[0][t];
#pragma unroll
    for (int w = 1; w < WV; ++w)
      if (beats(s_val[w][t], s_idx[w][t], best, best_i)) { best = s_val[w][t]; best_i = s_idx[w][t]; }
    part_val[(long)(m0 + t) * n_vtiles + vt] = best;
    part_idx[(long)(m0 + t) * n_vtiles + vt] = best_i;
    if (STATS) {
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < WV; ++w)
        if (s_val[w][t] > -INFINITY) sum += s_sum[w][t] * __builtin_amdgcn_exp2f((s_val[w][t] - best) * inv_temp_log2);
      part_sum[(long)(m0 + t) * n_vtiles + vt] = sum;
    }
  }
}

template <int CTRL, int ROWS>
__device__ __forceinline__ void best_moved(float& best, int& best_i) {
  const float ov = __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(-INFINITY), __float_as_int(best), CTRL, ROWS, 0xf, false));
  const int oi = __builtin_amdgcn_update_dpp(0x7fffffff, best_i, CTRL, ROWS, 0xf, false);
  if (beats(ov, oi, best, best_i)) { best = ov; best_i = oi; }
}

// One workgroup per row: merges the row's n_vtiles partials (part_sum != nullptr: also the sums, rescaled to
// the row's maximum). Bound by its launch and one trip to memory (two, and exchanges through LDS, before: 64.7 -> 63.9 us with the
// product in front of it, 128 rows of 32000 x 4096).
__global__ void __launch_bounds__(256) lm_head_reduce_kernel(const float* __restrict__ part_val,
                                                             const int32_t* __restrict__ part_idx,
                                                             const float* __restrict__ part_sum, float inv_temp_log2,
                                                             int n_vtiles, int32_t* __restrict__ node_argmax,
                                                             float* __restrict__ node_max, float* __restrict__ node_sumexp) {
  __shared__ float s_val[4];
  __shared__ int s_idx[4];
  __shared__ float s_sum[4];
  const int m = blockIdx.x, t = threadIdx.x;
  // The first partials of a thread (all of them up to 512 workgroups), sums too, are requested at once: sums asked for when the
  // maximum is known are a second trip to memory.
  constexpr int PRE = 2;
  float pre_v[PRE], pre_s[PRE];
  int pre_i[PRE];
#pragma unroll
  for (int p = 0; p < PRE; ++p) {
    const int j = t + 256 * p;
    const long at = (long)m * n_vtiles + min(j, n_vtiles - 1);
    pre_v[p] = part_val[at];
    pre_i[p] = part_idx[at];
    pre_s[p] = part_sum != nullptr ? part_sum[at] : 0.f;
    if (j >= n_vtiles) pre_v[p] = -INFINITY;
  }
  float best = -INFINITY;
  int best_i = 0x7fffffff;
#pragma unroll
  for (int p = 0; p < PRE; ++p)
    if (t + 256 * p < n_vtiles && beats(pre_v[p], pre_i[p], best, best_i)) { best = pre_v[p]; best_i = pre_i[p]; }
  for (int j = t + 256 * PRE; j < n_vtiles; j += 256) {
    const float v = part_val[(long)m * n_vtiles + j];
    const int i = part_idx[(long)m * n_vtiles + j];
    if (beats(v, i, best, best_i)) { best = v; best_i = i; }
  }
  // the wavefront's best into its last lane, in register moves (row shifts, then the last lane of a row of 16 into later rows)
  best_moved<0x111, 0xf>(best, best_i);
  best_moved<0x112, 0xf>(best, best_i);
  best_moved<0x114, 0xf>(best, best_i);
  best_moved<0x118, 0xf>(best, best_i);
  best_moved<0x142, 0xa>(best, best_i);
  best_moved<0x143, 0xc>(best, best_i);
  if ((t & 63) == 63) { s_val[t >> 6] = best; s_idx[t >> 6] = best_i; }
  __syncthreads();
  best = s_val[0]; best_i = s_idx[0];
  for (int w = 1; w < 4; ++w)
    if (beats(s_val[w], s_idx[w], best, best_i)) { best = s_val[w]; best_i = s_idx[w]; }
  if (part_sum != nullptr) {
    float sum = 0.f;
#pragma unroll
    for (int p = 0; p < PRE; ++p)
      if (pre_v[p] > -INFINITY) sum += pre_s[p] * __builtin_amdgcn_exp2f((pre_v[p] - best) * inv_temp_log2);
    for (int j = t + 256 * PRE; j < n_vtiles; j += 256) {
      const float v = part_val[(long)m * n_vtiles + j];
      if (v > -INFINITY) sum += part_sum[(long)m * n_vtiles + j] * __builtin_amdgcn_exp2f((v - best) * inv_temp_log2);
    }
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    if ((t & 63) == 0) s_sum[t >> 6] = sum;
    __syncthreads();
    if (t == 0 && node_sumexp != nullptr) node_sumexp[m] = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
  }
  if (t == 0) {
    if (node_argmax != nullptr) node_argmax[m] = best_i == 0x7fffffff ? 0 : best_i;   // a row of NaN / -inf logits
    if (node_max != nullptr) node_max[m] = best;
  }
}

}  // namespace lmh

// logits_out != nullptr: the kernel also writes the bf16 logits [M, V] and the softmax statistics of the rounded
// values (node_sumexp; inv_temp = 1 / temperature); the workspace then holds a third partial array.
hipError_t launch_lm_head(int M, int K, int V, const void* hidden, const void* weight, void* logits_out, float inv_temp,
                          int32_t* node_argmax, float* node_max, float* node_sumexp, void* ws, hipStream_t s) {
  const bool stats = logits_out != nullptr;
  const size_t arr = lm_head_partials_bytes(M, V) / 2;
  float* part_val = (float*)ws;
  int32_t* part_idx = (int32_t*)((char*)ws + arr);
  float* part_sum = stats ? (float*)((char*)ws + 2 * arr) : nullptr;
  const float itl2 = inv_temp * 1.4426950408889634f;
  // Tile of the vocabulary and of `hidden`: the least of rounds of workgroups (one per compute unit at a time) times
  // (start and end of a workgroup + stages times the microseconds a stage takes it), with the stage times as measured on
  // 32000 and 8000 x 4096 with one workgroup per compute unit. 8000 x 4096, 16 / 128 rows: 21.1 / 33.3 us with 64 vocabulary
  // rows, 28.8 / 45.2 with 128; 20000 x 768, 8 rows (313 workgroups of 64): 15.0 with 64, 12.2 with 128; 11198 x 2560, 227
  // rows: 57.3 with 256 rows of `hidden`, 38.3 with 128.
  const int cus = compute_units();
  int mt = 0, vt = 0;
  float least = 0.f;
  auto consider = [&](int rows, int v, int m, float stage_us) {
    const long wgs = (long)((V + v - 1) / v) * ((rows + m - 1) / m);
    const float us = (float)((wgs + cus - 1) / cus) * (3.f + (float)(K / lmh::KC) * stage_us);
    if (mt == 0 || us < least) { least = us; mt = m; vt = v; }
  };
  consider(1, 128, 32, 0.63f);
  consider(1, 64, 32, 0.3f);
  const bool two = vt == 64;   // whether up to 32 rows take the 64 x 32 tile: decides the order of sums for every M
  if (M > 32) {
    const int first_mt = M <= 64 ? 64 : 128;
    mt = 0;
    consider(M, 128, first_mt, first_mt == 128 ? 0.73f : 0.63f);
    consider(M, 64, first_mt, first_mt == 128 ? 0.42f : 0.3f);
    if (M > 128) consider(M, 128, 256, 1.15f);
  }
  // 128 x 32 tiles: two workgroups per compute unit for short sums, whose starts and ends would otherwise stand by themselves,
  // one with a long ring for long ones (16 rows, arg-max only, us, one / two: 32000 x 4096 51.5 / 55.4, x 2048 30.1 / 29.9, x 512
  // 11.3 / 10.5, x 256 9.1 / 8.3; 50257 x 512 17.3 / 13.8; 128256 x 4096 202 / 207, x 2048 110 / 104, x 512 33 / 25, x 256
  // 24.5 / 16.9, where W straight into registers took 201, 107, 30 and 18.9). 64 x 32 tiles gain from two at every K (16000 x
  // 4096 30.0 / 28.3, 8000 x 512 8.4 / 8.1).
  const bool pairs = K <= 2048;
  // Rows of W a multiple of 4 KB apart: workgroups that read the same k at the same time meet in the same few memory channels. Half
  // of them 2 KB further on, us with logits and statistics, in step / apart, 16 and 128 rows over 32000: K = 2048 32.5 / 27.3, 39.3 /
  // 35.8; 4096 54.8 / 48.2, 61.5 / 57.3; 6144 84.5 / 64.4, 100.1 / 83.7; 8192 103.9 / 94.0, 116.3 / 103.1 (4096 by 1 KB 50.9, 4 KB
  // 53.2, each workgroup at another k 46.3, four quarters 47.4; every other eight instead of sixteen 59.1). No gain at K = 1024,
  // 1536, 3072, 3328 and 5120, nor for 250 rows (arithmetic).
  const bool apart = K % 2048 == 0;
  const int m_slices = (M + mt - 1) / mt;
  const int n_vtiles = (V + vt - 1) / vt;
  const int per_row = std::min(m_slices, 16);   // slices numbered eight apart within a grid row
  const dim3 grid((unsigned)((n_vtiles + 7) / 8 * 8) * per_row, (m_slices + per_row - 1) / per_row);
#define SPEC_LMH(VTT, MT, RK, TW, AP, ST)                                                                                     \
  hipLaunchKernelGGL((lmh::lm_head_argmax_kernel<VTT, MT, RK, TW, AP, ST>), grid, dim3(lmh::NTHREADS), 0, s,                      \
                     (const __hip_bfloat16*)hidden, (const __hip_bfloat16*)weight, part_val, part_idx, part_sum,              \
                     (__hip_bfloat16*)logits_out, itl2, M, K, V, n_vtiles, per_row)
#define SPEC_LMH_T(TW, AP, ST)                              \
  if (mt == 256) SPEC_LMH(128, 256, 128, TW, AP, ST);            \
  else if (vt == 128 && mt == 128) SPEC_LMH(128, 128, 128, TW, AP, ST); \
  else if (vt == 128 && mt == 64) SPEC_LMH(128, 64, 128, TW, AP, ST);        \
  else if (mt == 128) SPEC_LMH(64, 128, 128, TW, AP, ST);        \
  else SPEC_LMH(64, 64, 128, TW, AP, ST)
#define SPEC_LMH_1(AP, ST)                              \
  if (mt == 32 && pairs) SPEC_LMH(128, 32, 64, false, AP, ST); \
  else if (mt == 32) SPEC_LMH(128, 32, 128, false, AP, ST); \
  else { SPEC_LMH_T(false, AP, ST); }
#define SPEC_LMH_ST(ST)                                 \
  if (mt == 32 && two) SPEC_LMH(64, 32, 64, true, false, ST);  \
  else if (two) { SPEC_LMH_T(true, false, ST); }               \
  else if (apart) { SPEC_LMH_1(true, ST); }                  \
  else { SPEC_LMH_1(false, ST); }
  if (stats) { SPEC_LMH_ST(true); } else { SPEC_LMH_ST(false); }
#undef SPEC_LMH_ST
#undef SPEC_LMH_1
#undef SPEC_LMH_T
#undef SPEC_LMH
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(lmh::lm_head_reduce_kernel, dim3(M), dim3(256), 0, s, part_val, part_idx, part_sum, itl2, n_vtiles,
                     node_argmax, node_max, node_sumexp);
  return hipGetLastError();
}

hipError_t launch_lm_head_argmax(int M, int K, int V, const void* hidden, const void* weight, int32_t* node_argmax,
                                 float* node_max, void* ws, hipStream_t s) {
  return launch_lm_head(M, K, V, hidden, weight, nullptr, 1.f, node_argmax, node_max, nullptr, ws, s);
}

}  // namespace spec
