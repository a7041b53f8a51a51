// Tree attention for bf16 K/V on the gfx950 matrix cores (Definition 4.1; topology-aware causal mask
// of Section 4.2), written for the decode-shaped case: few tree queries (N <= 16, one MFMA query
// tile; larger trees go to the kernel in tree_attention_bf16_wide.hip) against a long cached prefix,
// so the kernel is bound by streaming K and V from HBM exactly once.
//
// Decomposition
//   grid = (n_splits, H, B), or (PLAN 1, 2) workgroups that share the 32-key tiles of all (request, head)
//   pairs evenly (see balanced_deal() and contiguous_deal()). A workgroup owns one segment of the key
//   range of one (request, head) at a time and all its tree queries. It has five wavefronts:
//     - four streaming wavefronts take the chunk's mask-free 32-key tiles (entirely inside the cached
//       prefix) round-robin; they never need the tree, a mask, or a barrier inside their loop;
//     - one tail wavefront owns the ragged end: the tiles that reach past prefix_len (the tree rows,
//       the end of the sequence). It alone validates the tree, builds the ancestor masks, applies
//       them, and (fused append) writes the new rows to the cache. Its few tiles run concurrently
//       with the stream instead of forming a serial tail, and the stream stays evenly divided.
//   Each wavefront keeps its own online-softmax state; the five are merged once, through LDS.
//
// Per 32-key tile and wavefront
//   S^T = K Q^T   v_mfma_f32_16x16x32_bf16, A = K rows read straight from global memory into the
//                 MFMA operand layout (lane r of a 16-lane group holds 8 consecutive d of key r),
//                 B = Q^T resident in registers. The transposed product leaves lane l with scores of
//                 query l%16 for keys 4*(l/16)+v of each 16-key half: exactly the B-operand layout
//                 P^T needs for the second product, so probabilities never leave registers.
//   mask          tail wavefront only: bit (key - prefix_len) of the query's ancestor-or-self mask of 16 bits,
//                 built between the lanes by pointer doubling (a lane holds a node).
//   softmax       online, in the exp2 domain, with a lazy running maximum (refreshed, with two cross-lane
//                 exchanges and a rescale of the lane-local O^T fragment, only when a score outgrows it).
//   O^T += V^T P^T  A = V^T needs 8 keys x 1 d per lane, the transpose of how V lies in memory: V is
//                 loaded fully coalesced (four 256-byte rows per instruction), staged in a
//                 wavefront-private LDS tile and read back with ds_read_b64_tr_b16.
//
// Latency structure. A workgroup's fixed costs are what separate this kernel from a pure stream: the
// streaming wavefronts' first tiles are issued before prefix_len is known (rows clamped to the cache capacity),
// in straight-line code so that all kernel arguments arrive in one batch; every tile's loads are issued
// one tile ahead; nothing in the loop waits on more than its own tile. A compute unit returns its wavefronts'
// loads in the order of their requests, so what a later step waits for must not stand behind the tiles: the tree
// words come through the scalar cache, the tail wavefront requests nothing else before it has them, and it alone
// fetches the rotary angles and rotates the queries, for all five through LDS (each wavefront on its own, behind
// its first tile, before: two layers of 8 requests, 1024 keys, trees of 16 with the embedding 55.2 -> 54.2 us; 8 x
// 12 heads of 708 keys, trees of 5, without it, 27.7 -> 25.2; 4 x 40 heads of 98 keys 8.2 -> 7.5).
//
// With APPEND the kernel also performs the KV append of the tree tokens (Section 4.2): rows at and
// beyond prefix_len are taken from k_new / v_new and written to the cache by query group 0.
//
// Results are written as the final bf16 output when one workgroup covers the whole key range of a
// pair, else as float32 partials (m, l, O) merged by attn_combine_kernel.
#include <hip/hip_bf16.h>

#include <cstdlib>
#include <type_traits>

#include "spec_internal.h"

namespace spec {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef f32x4 __attribute__((aligned(4))) f32x4_any;   // the rotary tables may start at any float
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;   // 16-byte load/store unit (plain vector: stays in registers)


constexpr float kLog2eB = 1.4426950408889634f;
constexpr int TILE = SPEC_SMALL_TILE_KEYS;          // keys per wavefront tile
constexpr int SWAVES = 4;         // streaming wavefronts
constexpr int WAVES = SWAVES + 1; // plus the tail wavefront
constexpr int TAIL = SWAVES;      // its index

__device__ inline float wave_max_over_lane_groups(float v) {
  // lanes l, l^16, l^32, l^48 hold the same query: reduce over the four 16-lane groups
  v = fmaxf(v, __shfl_xor(v, 16));
  v = fmaxf(v, __shfl_xor(v, 32));
  return v;
}
__device__ inline float wave_sum_over_lane_groups(float v) {
  v += __shfl_xor(v, 16);
  v += __shfl_xor(v, 32);
  return v;
}
// 16-byte load of a K/V row piece. Marked non-temporal: the K/V stream is read once per launch, and a plain
// read of the same bytes is measurably faster with the hint (the lines do not displace one another in the L2).
__device__ __forceinline__ u32x4 load_kv(const unsigned char* p) {
  return __builtin_nontemporal_load((const u32x4*)p);
}
// 16-byte store of an appended cache row. Marked non-temporal: the rows are not read again by this
// kernel, and dirty lines left in the L2 lengthen the write-back at the end of the kernel.
__device__ __forceinline__ void store_cache_row(void* p, u32x4 v) {
  // (the builtin, not inline assembly: the compiler then keeps the store's data registers untouched for the wait
  // states a 16-byte store needs after issue)
  __builtin_nontemporal_store(v, (u32x4*)p);
}

// Barrier for LDS contents only: __syncthreads() also waits for the tiles in flight and for the appended rows' stores.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int D, int NT>
struct AttnTraits {
  static constexpr int KS = D / 32;            // k-steps of the QK^T product
  static constexpr int DB = D / 16;            // 16-wide d blocks of the output
  static constexpr int LPR = D * 2 / 16;       // lanes (16-byte pieces) per K/V row
  static constexpr int RPI = 64 / LPR;         // rows covered by one wave-wide 16-byte load
  static constexpr int NVL = TILE / RPI;       // V loads per lane per tile
  static constexpr int VROW = D * 2 + 16;      // LDS bytes per staged V row (+16 B pad)
  static constexpr int VTILE_BYTES = TILE * VROW;
  static constexpr int NQ = NT * 16;           // queries per workgroup
  static constexpr int MROW = D + 4;           // floats per merge row: O[D], m, l, 2 pad (16-byte aligned rows)
  static constexpr int STAGE_BYTES = WAVES * VTILE_BYTES;
  // the merge area lies behind the staging tiles: a wavefront publishes its partial result as soon as it is done
  static constexpr int LDS_BYTES = STAGE_BYTES + WAVES * NQ * MROW * 4;
};

// Pointers and strides one lane needs to fetch its pieces of a tile.
struct TileSrc {
  const unsigned char* kc;   // cache K of this (request, head), byte pointer at the lane's column
  const unsigned char* vc;
  const unsigned char* kn;   // new K of this (request, head) at node 0, lane's column (APPEND only)
  const unsigned char* vn;
  unsigned cache_row_bytes;
  unsigned new_row_bytes;
};

// Loads of one tile, V rows and K rows separately (V is consumed first). CLEAN: every row lies inside
// the cached prefix (no clamp, no source select). Otherwise rows are clamped to `last_row`; with
// APPEND rows >= P come from the new K/V.
template <int D, int NT, bool APPEND, bool CLEAN>
__device__ __forceinline__ void issue_v_loads(const TileSrc& s, int k0, int P, int last_row, int lane,
                                              u32x4 (&Vn)[AttnTraits<D, NT>::NVL], long shift = 0) {
  using T = AttnTraits<D, NT>;
#pragma unroll
  for (int j = 0; j < T::NVL; ++j) {
    int row = k0 + j * T::RPI + lane / T::LPR;
    const unsigned char* p;
    if (CLEAN) {
      p = s.vc + (unsigned)row * s.cache_row_bytes + shift;
    } else {
      row = min(row, last_row);
      p = (APPEND && row >= P) ? s.vn + (unsigned)(row - P) * s.new_row_bytes
                               : s.vc + (unsigned)row * s.cache_row_bytes + shift;
    }
    Vn[j] = load_kv(p);
  }
}
template <int D, int NT, bool APPEND, bool CLEAN>
__device__ __forceinline__ void issue_k_loads(const TileSrc& s, int k0, int P, int last_row, int r16,
                                              u32x4 (&Kn)[2][AttnTraits<D, NT>::KS], long shift = 0) {
  using T = AttnTraits<D, NT>;
#pragma unroll
  for (int hf = 0; hf < 2; ++hf) {
    int row = k0 + hf * 16 + r16;
    const unsigned char* p;
    if (CLEAN) {
      p = s.kc + (unsigned)row * s.cache_row_bytes + shift;
    } else {
      row = min(row, last_row);
      p = (APPEND && row >= P) ? s.kn + (unsigned)(row - P) * s.new_row_bytes
                               : s.kc + (unsigned)row * s.cache_row_bytes + shift;
    }
#pragma unroll
    for (int ks = 0; ks < T::KS; ++ks) Kn[hf][ks] = load_kv(p + ks * 64);
  }
}
template <int D, int NT, bool APPEND, bool CLEAN>
__device__ __forceinline__ void issue_tile_loads(const TileSrc& s, int k0, int P, int last_row, int r16, int lane,
                                                 u32x4 (&Kn)[2][AttnTraits<D, NT>::KS],
                                                 u32x4 (&Vn)[AttnTraits<D, NT>::NVL], long shift = 0) {
  issue_v_loads<D, NT, APPEND, CLEAN>(s, k0, P, last_row, lane, Vn, shift);
  issue_k_loads<D, NT, APPEND, CLEAN>(s, k0, P, last_row, r16, Kn, shift);
}

// PAGED: the caches are pools of blocks addressed through pg.table (see cache_row_offset). A wavefront's
// 32-key tile starts at a multiple of 32 rows and a block holds a multiple of 64, so a tile lies inside one
// block: its rows are addressed as in a contiguous cache plus one per-tile offset (page_shift below).
// PLAN: 0 fixed chunks, 1 the balanced deal, 2 its contiguous form. work: keys per chunk (0), chunks the deal aims at (1).
// NT and n_qgroups are 1 (larger trees and grouped heads go to the wide kernels). Both stay written out: without n_qgroups the
// first loads come in another order, which costs 8 requests of 1024 keys 1.2 % (trees of 16, rotary) to 2.3 % (trees of 7), and
// without NT one request loses 0.9 %.
// EARLY: with the rotary embedding, the first tile moved to LDS while the queries are rotated (see s_k): D = 128, PLAN 0 and 1. The
// other instances have the embedding behind a run-time branch on rope.cos. D = 64 and PLAN 2 take it; for D = 128 under PLAN 0 and 1
// rope.cos is always null there, and the branch with its 12.5 KB of LDS stays for what it does to the order of the first loads:
// compiled out, launches without the embedding take up to 4 % longer (us, with the branch / without: 8 x 32 heads of 400 keys, trees
// of 13, 12.8 / 13.2; 4 x 32 of 900, 16, 17.7 / 18.0; 24 x 40 of 1000, 16, 102.0 / 102.8; others the same).
template <int D, int NT, bool APPEND, bool EARLY, int PLAN, bool PAGED>
__global__ void __launch_bounds__(WAVES * 64, 2) tree_attention_bf16_kernel(
    const __hip_bfloat16* __restrict__ q, __hip_bfloat16* k_cache, __hip_bfloat16* v_cache,
    const __hip_bfloat16* __restrict__ k_new, const __hip_bfloat16* __restrict__ v_new,
    const int32_t* __restrict__ parent, const int32_t* __restrict__ depth, const int32_t* __restrict__ prefix_len,
    __hip_bfloat16* __restrict__ out, float* __restrict__ ws_o, float* __restrict__ ws_ml, int32_t* status, int B, int N,
    int H, int S_cap, int n_qgroups, int work, int n_splits, long q_sb, long q_sn, long q_sh, long kv_sb,
    long kv_sh, long kv_ss, float scale_log2, Pages pg, Rope rope) {
  using T = AttnTraits<D, NT>;
  constexpr int KS = T::KS, DB = T::DB, LPR = T::LPR, RPI = T::RPI, NVL = T::NVL, VROW = T::VROW, NQ = T::NQ,
                MROW = T::MROW;
  constexpr int NTHREADS = WAVES * 64;

  // With the rotary embedding the tail wavefront hands over the rotated queries, as the streaming wavefronts' lanes take them,
  // and keeps its nodes' angles (rows of D/2 cosines and D/2 sines, 16 bytes more so that rows start on other banks).
  constexpr int ANGLE_ROW = D + 4;
  __shared__ __attribute__((aligned(16))) unsigned char lds[T::LDS_BYTES];
  __shared__ __attribute__((aligned(16))) u32x4 s_q[APPEND ? KS * 64 : 1];
  __shared__ __attribute__((aligned(16))) float s_angle[APPEND ? 16 * ANGLE_ROW : 4];
  // With the embedding the streaming wavefronts wait for the rotated queries with one tile on its way each. Their first tile moves to
  // LDS meanwhile (V where it is staged anyway, a lane's pieces of K into slots of its own), and the second is requested into its
  // registers. us, before / now, trees of 16: 1 x 32 heads of 1024 keys 12.7 / 12.0, of 4000 20.1 / 18.5; 4 x 32 of 300 11.8 / 10.7, of 900
  // 18.4 / 16.8; 8 x 32 of 400 14.2 / 12.6, of 1024 29.4 / 27.9, of 2000 47.9 / 46.4; 24 x 40 of 1000 105.5 / 101.2, 20 x 40 of 150 (one or two
  // tiles per wavefront) 42.5 / 42.0; paged 8 x 32 of 500, trees of 9, 16.9 / 15.8. Seven streaming wavefronts do as much for the
  // wait, but then sum in another order than the call without the embedding, whose bits this one has. At D = 64 the LDS would cost a
  // workgroup per compute unit, and the contiguous plan has no register left.
  __shared__ __attribute__((aligned(16))) u32x4 s_k[EARLY ? SWAVES * 2 * KS * 64 : 1];
  __shared__ int s_bad_tree;
  static_assert(NT == 1, "a tree of at most 16 nodes: lane r16 holds node r16, which is also its query");

  // One argument from each 64-byte line of the argument block, all asked for at once: with branches in between, the compiler asks
  // for a line where it is first used, one trip to memory after the other (with the tree words of a tree of sixteen in one wait: 8 x 32
  // heads of 1024 keys, rotary, two layers 54.0 -> 53.2 us; 32 layers of 1 x 32 heads and what follows 473 -> 458 and 462 in two runs).
  // Not under the contiguous plan, where a hundred scalars are spilled already and arguments held from the start are more of them (us,
  // with / without: 6 x 32 heads x 64 of 2251-4500 keys, trees of 11, rotary, 43.1 / 42.2, paged without it 49.1 / 48.3; 5 x 40 x 64 of
  // 1559-3116, 2, rotary, 34.5 / 33.9; 7 x 32 x 64 of 3000-6000, one node, 54.6 / 53.9; 5 x 32 x 128 of 3000-6000, 12, 76.5 / 75.0).
  if constexpr (PLAN != 2) asm("" : "+s"(N) : "s"(prefix_len), "s"(kv_ss), "s"(rope.len));
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r16 = lane & 15, g = lane >> 4;

  // Paged cache: byte offset that, added to `row * row_bytes`, gives the place of logical row `row` of request
  // b for every row of the 32-row tile at k0 (clamped rows stay inside the tile, hence inside its block).
  // `ok`: the table entry lies inside the pool; one that does not is replaced by a block of the pool.
  // The contiguous plan, whose loop over segments has no register left for the lanes, reads the table for every tile.
  constexpr bool LANES = PAGED && PLAN != 2;
  BlockLanes blocks = {0, 0, 0ull};
  auto page_shift = [&](int b, int k0, bool* ok) -> long {
    const int j = __builtin_amdgcn_readfirstlane(min(k0, S_cap - 1) >> pg.log2_tokens);
    int blk;
    if constexpr (LANES) {
      const int l = block_lane(blocks, pg, b, j);
      *ok = !((blocks.bad >> l) & 1ull);
      blk = __builtin_amdgcn_readlane(blocks.block, l);
    } else {
      const int e = pg.table[(long)b * pg.max_blocks + j];
      *ok = e >= 0 && e < pg.n_blocks;
      blk = min(max(e, 0), pg.n_blocks - 1);
    }
    return (long)blk * kv_sb * 2 - (long)((unsigned)(j << pg.log2_tokens) * ((unsigned)kv_ss * 2u));
  };

  // One segment: keys [c0, min(c1_cap, prefix_len + N)) of request b, head h, query group qg. The result is
  // the final output (part_row < 0) or the float32 partial whose first row in the workspace is part_row.
  auto segment = [&](const int b, const int h, const int qg, const int c0, const int c1_cap, const long part_row) {
  const bool final_out = part_row < 0;
  const int q0 = qg * NQ;

  // ---- straight-line prologue (no branch before the first loads, so every kernel argument is
  // fetched in one batch): the streaming wavefronts' first tile does not depend on prefix_len (rows
  // clamped to the cache capacity keep the addresses valid; the tail wavefront's copy is discarded),
  // Q, and a tree node per lane.
  const int P = prefix_len[b];
  TileSrc src;
  src.cache_row_bytes = (unsigned)kv_ss * 2u;
  src.new_row_bytes = (unsigned)q_sn * 2u;
  src.kc = (const unsigned char*)(k_cache + (PAGED ? 0 : b * kv_sb) + h * kv_sh) + g * 16;
  src.vc = (const unsigned char*)(v_cache + (PAGED ? 0 : b * kv_sb) + h * kv_sh) + (lane % LPR) * 16;
  src.kn = APPEND ? (const unsigned char*)(k_new + b * q_sb + h * q_sh) + g * 16 : nullptr;
  src.vn = APPEND ? (const unsigned char*)(v_new + b * q_sb + h * q_sh) + (lane % LPR) * 16 : nullptr;

  const int first_block = LANES ? min(c0, S_cap - 1) >> pg.log2_tokens : 0;
  if (LANES) blocks = load_block_lanes(pg, b, first_block);

  // The tail wavefront: a tree node per lane, from scalar loads. More than eight nodes: four groups of four in one wait, the last two
  // moved up to end with the tree (1 x 32 heads of 1024 keys, trees of 16: 11.4 us, 11.9 rotated, the same as by one load of 64 bytes;
  // 11.9 and 13.0 by groups one after the other; trees of 9 to 15 gain less than 1 %). Fewer: four at a time as far as
  // there are any (all at once, clamped, cost the smallest calls what they wait for: 2 x 64 heads of 58 keys, one node, D = 64, 5.2 us,
  // 4.7 by fours). Rows past N repeat the last query (their results are never written): the loads are unconditional.
  const bool is_tail = wave == TAIL;
  const bool rotates = EARLY || (APPEND && rope.cos != nullptr);
  int par = 0, dep = 0;
  if (is_tail && N > 8) {
#pragma unroll
    for (int i0 = 0; i0 < 16; i0 += 4) {
      const int first = i0 < 8 ? i0 : min(i0, N - 4);
      const int32_t *pw = parent + (long)b * N + first, *dw = depth + (long)b * N + first;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int p = pw[i], d = dw[i];
        par = r16 == first + i ? p : par;
        dep = r16 == first + i ? d : dep;
      }
    }
  } else if (is_tail) {
#pragma unroll
    for (int i0 = 0; i0 < 16; i0 += 4) {
      if (i0 >= N) break;
#pragma unroll
      for (int i = i0; i < i0 + 4; ++i) {
        const long at = (long)b * N + min(i, N - 1);
        const int p = parent[at], d = depth[at];
        par = r16 == i ? p : par;
        dep = r16 == i ? d : dep;
      }
    }
  }
  bf16x8 qB[NT][KS];   // Q^T as the B operand: lane (r16, g) holds Q[n = r16][d = ks*32 + g*8 .. +8]
  if (is_tail || !rotates) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const u32x4 raw = *(const u32x4*)(q + b * q_sb + min(r16, N - 1) * q_sn + h * q_sh + ks * 32 + g * 8);
      qB[0][ks] = __builtin_bit_cast(bf16x8, raw);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  u32x4 KA[2][KS], VA[NVL];   // tile buffer: loads land here one step ahead of use
  bool in_pool;   // entries past the request's end may hold anything: the speculative tile does not judge them
  if (!is_tail)
    issue_tile_loads<D, NT, false, false>(src, c0 + wave * TILE, 0, S_cap - 1, r16, lane, KA, VA,
                                          PAGED ? page_shift(b, c0 + wave * TILE, &in_pool) : 0);
  __builtin_amdgcn_sched_barrier(0);

  const bool cap_ok = (P >= 0) && (P <= S_cap - N);
  const int len = P + N;
  if (!cap_ok) {
    if (final_out) {
      for (int i = t; i < NQ * D; i += NTHREADS) {
        const int n = q0 + i / D;
        if (n < N) out[b * q_sb + n * q_sn + h * q_sh + (i % D)] = __float2bfloat16(0.f);
      }
      if (h == 0 && qg == 0 && t == 0) set_status(status, b, SPEC_ST_CAPACITY);
    }
    return;
  }
  if (c0 >= len) return;
  const int c1 = min(c1_cap, len);
  const bool touches_tree = c1 > P;
  const int n_tiles = (c1 - c0 + TILE - 1) / TILE;
  const int n_clean = max(0, min(P, c1) - c0) / TILE;     // tiles entirely inside the prefix and the chunk
  const int last_row = len - 1;

  // Rotary embedding: a lane's pieces of a query or key row pair up within the lane (k-step ks holds dimensions
  // 32 ks + 8 g .., its partner ks + KS/2 the same dimensions + D/2), so a row is rotated in registers. `angle`: the row's
  // cosines, the sines D/2 behind them.
  auto rotate_row = [&](auto& lo, auto& hi, const float* angle, int ks) {
    uint4 olo, ohi;
    rope_pair<true>(__builtin_bit_cast(uint4, lo), __builtin_bit_cast(uint4, hi), angle + ks * 32 + g * 8,
                    angle + D / 2 + ks * 32 + g * 8, &olo, &ohi);
    lo = __builtin_bit_cast(std::remove_reference_t<decltype(lo)>, olo);
    hi = __builtin_bit_cast(std::remove_reference_t<decltype(hi)>, ohi);
  };
  const int last_block = LANES ? (c1 - 1) >> pg.log2_tokens : 0;
  if (LANES && is_tail && lane == 0 && blocks_outside(blocks, last_block)) set_status(status, b, SPEC_ST_BAD_BLOCK);
  // tiles of this wavefront: first and end (the streaming wavefronts take every SWAVES-th)
  const int ti_first = is_tail ? n_clean : wave;
  const int ti_end = is_tail ? n_tiles : n_clean;
  if (is_tail) {
    if constexpr (APPEND) {
      if (rotates) {   // lane (r16, g) fetches its pieces of node r16's angles
        const long at = (long)min(max(P + dep, 0), rope.len - 1) * (D / 2) + g * 8;
        float* row = s_angle + r16 * ANGLE_ROW;
        f32x4 cs[KS / 2][2], sn[KS / 2][2];
#pragma unroll
        for (int ks = 0; ks < KS / 2; ++ks)
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            cs[ks][i] = *(const f32x4_any*)(rope.cos + at + ks * 32 + i * 4);
            sn[ks][i] = *(const f32x4_any*)(rope.sin + at + ks * 32 + i * 4);
          }
#pragma unroll
        for (int ks = 0; ks < KS / 2; ++ks)
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            *(f32x4*)(row + ks * 32 + g * 8 + i * 4) = cs[ks][i];
            *(f32x4*)(row + D / 2 + ks * 32 + g * 8 + i * 4) = sn[ks][i];
          }
#pragma unroll
        for (int ks = 0; ks < KS / 2; ++ks) rotate_row(qB[0][ks], qB[0][ks + KS / 2], row, ks);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) s_q[ks * 64 + lane] = __builtin_bit_cast(u32x4, qB[0][ks]);
      }
    }
  }
  unsigned char* vst = lds + wave * T::VTILE_BYTES;
  if constexpr (EARLY) {
    if (!is_tail && ti_first < ti_end) {
      const int second = ti_first + SWAVES < ti_end ? ti_first + SWAVES : -1;
      const int k1 = c0 + second * TILE;
      const long shift = (PAGED && second >= 0) ? page_shift(b, k1, &in_pool) : 0;
#pragma unroll
      for (int j = 0; j < NVL; ++j) *(u32x4*)(vst + (j * RPI + lane / LPR) * VROW + (lane % LPR) * 16) = VA[j];
      __builtin_amdgcn_sched_barrier(0);
      if (second >= 0) issue_v_loads<D, NT, APPEND, true>(src, k1, P, last_row, lane, VA, shift);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) s_k[((wave * 2 + hf) * KS + ks) * 64 + lane] = KA[hf][ks];
      __builtin_amdgcn_sched_barrier(0);
      if (second >= 0) issue_k_loads<D, NT, APPEND, true>(src, k1, P, last_row, r16, KA, shift);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if constexpr (APPEND) {
    if (rotates) {
      lds_barrier();
      if (!is_tail) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qB[0][ks] = __builtin_bit_cast(bf16x8, s_q[ks * 64 + lane]);
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);   // (otherwise the requests move down to the masks)
  if (is_tail && ti_first < ti_end)   // the tail wavefront's first tile (needs prefix_len: rows >= P have other sources)
    issue_tile_loads<D, NT, APPEND, false>(src, c0 + ti_first * TILE, P, last_row, r16, lane, KA, VA,
                                           PAGED ? page_shift(b, c0 + ti_first * TILE, &in_pool) : 0);
  __builtin_amdgcn_sched_barrier(0);

  f32x4 O[NT][DB];
  float m_run[NT], l_run[NT];
  unsigned anc = 0;   // ancestor-or-self mask of this lane's query
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    m_run[nt] = -INFINITY;
    l_run[nt] = 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db) O[nt][db] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }

  // ---- tail wavefront: validate the tree and build the ancestor-or-self masks, between the lanes: after i exchanges a
  // lane's mask reaches 2^i - 1 ancestors up, and `up` is the node after those.
  bool bad_tree = false;
  if (is_tail) {
    if (lane == 0) s_bad_tree = 0;
    if (touches_tree) {
      const int par_dep = __shfl(dep, min(max(par, 0), 15));
      const bool ok = r16 >= N || (r16 == 0 ? par == -1 && dep == 0 : par >= 0 && par < r16 && dep == par_dep + 1);
      bad_tree = __any(!ok);
      anc = 1u << r16;
      int up = par;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int from = min(max(up, 0), 15);
        const unsigned m = __shfl(anc, from);
        const int next = __shfl(up, from);
        if (up >= 0) {
          anc |= m;
          up = next;
        }
      }
      if (bad_tree && lane == 0) s_bad_tree = 1;
    }
  }
  // One tile: consume the buffer filled by earlier loads, refill it for the next step, S^T, softmax, O^T.
  // MOVED: the tile lies in LDS and the buffer's loads are under way.
  auto tile_step = [&](const int ti, const int ti_refill, auto masked_tag, auto moved_tag) {
    constexpr bool MASKED = decltype(masked_tag)::value, MOVED = decltype(moved_tag)::value;
    const int k0 = c0 + ti * TILE;
    if (MASKED) {
      // rows at and beyond the end of the chunk hold stale data: their V must not reach the product
#pragma unroll
      for (int j = 0; j < NVL; ++j)
        if (k0 + j * RPI + lane / LPR >= c1) VA[j] = (u32x4){0u, 0u, 0u, 0u};
      if (rotates) {   // new K rows are rotated before they are used and stored
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          const int row = k0 + hf * 16 + r16;
          if (row >= P && row < c1) {
#pragma unroll
            for (int ks = 0; ks < KS / 2; ++ks)
              rotate_row(KA[hf][ks], KA[hf][ks + KS / 2], s_angle + (row - P) * ANGLE_ROW, ks);
          }
        }
      }
      if (APPEND && qg == 0) {   // this tile carries tree rows taken from k_new / v_new: put them in the cache
        bool dst_ok = true;      // paged cache: rows of a block outside the pool are not written
        const long dst_shift = PAGED ? page_shift(b, k0, &dst_ok) : 0;
#pragma unroll
        for (int j = 0; j < NVL; ++j) {
          const int row = k0 + j * RPI + lane / LPR;
          if (row >= P && row < c1 && dst_ok)
            store_cache_row((unsigned char*)src.vc + (unsigned)row * src.cache_row_bytes + dst_shift, VA[j]);
        }
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          const int row = k0 + hf * 16 + r16;
          if (row >= P && row < c1 && dst_ok) {
            unsigned char* dst = (unsigned char*)src.kc + (unsigned)row * src.cache_row_bytes + dst_shift;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) store_cache_row(dst + ks * 64, KA[hf][ks]);
          }
        }
      }
    }
    if (!MOVED) {
#pragma unroll
      for (int j = 0; j < NVL; ++j) *(u32x4*)(vst + (j * RPI + lane / LPR) * VROW + (lane % LPR) * 16) = VA[j];
    }
    // Refill in place: V's registers are free once staged, K's once the S^T products have read them. The
    // scheduling fences keep the compiler from moving the requests above those uses: it would then need a second
    // set of registers for the rows in flight and copy it into the first on every tile, after the rows have arrived
    // and before the next request, which is time with nothing in flight.
    const int kn0 = c0 + ti_refill * TILE;
    bool refill_ok;
    const long refill_shift = (PAGED && ti_refill >= 0) ? page_shift(b, kn0, &refill_ok) : 0;
    __builtin_amdgcn_sched_barrier(0);
    if (ti_refill >= 0) issue_v_loads<D, NT, APPEND, !MASKED>(src, kn0, P, last_row, lane, VA, refill_shift);
    __builtin_amdgcn_sched_barrier(0);

    // ---- S^T = K Q^T : sc[nt][hf][v] = score of query nt*16+r16 and key k0 + hf*16 + 4g + v
    f32x4 sc[NT][2];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(bf16x8, MOVED ? s_k[((wave * 2 + hf) * KS + ks) * 64 + lane] : KA[hf][ks]), qB[nt][ks], acc, 0, 0, 0);
        sc[nt][hf] = acc;
      }
    __builtin_amdgcn_sched_barrier(0);
    if (ti_refill >= 0) issue_k_loads<D, NT, APPEND, !MASKED>(src, kn0, P, last_row, r16, KA, refill_shift);
    __builtin_amdgcn_sched_barrier(0);

    bf16x8 pB[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      float s[8];
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int v = 0; v < 4; ++v) s[hf * 4 + v] = sc[nt][hf][v] * scale_log2;
      if (MASKED) {
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int key = k0 + hf * 16 + 4 * g + v;
            const int rel = key - P;
            bool vis = key < c1;
            if (vis && rel >= 0) {
              vis = (anc >> rel) & 1u;
            }
            if (!vis) s[hf * 4 + v] = -INFINITY;
          }
      }
      // Lazy running maximum. m_run (exp2 domain, identical in the four lanes of a query) only has to be close to
      // the true maximum: probabilities are exp2(score - m_run) and everything is normalised by the same sum at the
      // end. It is refreshed, with the exact cross-lane maximum and the usual rescaling of l and O, only when some
      // score of the wavefront exceeds it by more than 2^16 (or it is still -inf); otherwise a tile costs no
      // cross-lane exchange and no pass over the accumulators, which a lone wavefront on its SIMD cannot hide.
      const float mx = fmaxf(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])), fmaxf(fmaxf(s[4], s[5]), fmaxf(s[6], s[7])));
      if (__any(mx > m_run[nt] + 16.f)) {
        const float m_new = fmaxf(m_run[nt], wave_max_over_lane_groups(mx));
        const float m_ref = (m_new == -INFINITY) ? 0.f : m_new;
        const float alpha = __builtin_amdgcn_exp2f(m_run[nt] - m_ref);
        m_run[nt] = m_new;
        l_run[nt] *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db) O[nt][db] *= alpha;
      }
      const float neg_m = (m_run[nt] == -INFINITY) ? 0.f : -m_run[nt];
      float psum = 0.f;
      bf16x8 pb;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float p = __builtin_amdgcn_exp2f(s[i] + neg_m);
        psum += p;
        pb[i] = (__bf16)p;
      }
      pB[nt] = pb;
      l_run[nt] += psum;
    }

    // ---- O^T += V^T P^T : A operand = V^T through the transposing LDS read
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      const unsigned char* base = vst + (4 * g + (r16 >> 2)) * VROW + db * 32 + (r16 & 3) * 8;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(base));
      const s16x4 hi =
          __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(base + 16 * VROW));
      union { struct { s16x4 a, b; } p; bf16x8 v; } vt;
      vt.p.a = lo;
      vt.p.b = hi;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        O[nt][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt.v, pB[nt], O[nt][db], 0, 0, 0);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };

  if (is_tail) {
    if (!bad_tree)
      for (int ti = ti_first; ti < ti_end; ++ti) tile_step(ti, ti + 1 < ti_end ? ti + 1 : -1, std::true_type{}, std::false_type{});
    if (PAGED) {   // every block this segment reads must lie inside the pool (those not in the lanes looked at last: nothing waits)
      for (int j = LANES ? first_block + 64 + lane : (c0 >> pg.log2_tokens) + lane; j <= (c1 - 1) >> pg.log2_tokens; j += 64) {
        const int e = pg.table[(long)b * pg.max_blocks + j];
        if (e < 0 || e >= pg.n_blocks) set_status(status, b, SPEC_ST_BAD_BLOCK);
      }
    }
  } else {
    int ti = ti_first;
    if constexpr (EARLY) {
      if (ti < ti_end) {
        tile_step(ti, -1, std::false_type{}, std::true_type{});
        ti += SWAVES;
      }
    }
    for (; ti < ti_end; ti += SWAVES)
      tile_step(ti, ti + SWAVES < ti_end ? ti + SWAVES : -1, std::false_type{}, std::false_type{});
  }

  // ---- merge the five wavefronts through LDS: layout [wave][n][MROW] floats (O row, m, l)
  float* mg = (float*)(lds + T::STAGE_BYTES);
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const float l_tot = wave_sum_over_lane_groups(l_run[nt]);
    float* row = mg + ((wave * NQ) + nt * 16 + r16) * MROW;
#pragma unroll
    for (int db = 0; db < DB; ++db) *(f32x4*)(row + db * 16 + 4 * g) = O[nt][db];
    if (g == 0) {
      row[D] = m_run[nt];
      row[D + 1] = l_tot;
    }
  }
  lds_barrier();
  if (s_bad_tree != 0) {   // malformed tree: defined result = zeros (written here when this workgroup owns the output)
    if (final_out) {
      for (int i = t; i < NQ * D; i += NTHREADS) {
        const int n = q0 + i / D;
        if (n < N) out[b * q_sb + n * q_sn + h * q_sh + (i % D)] = __float2bfloat16(0.f);
      }
      if (h == 0 && qg == 0 && t == 0) set_status(status, b, SPEC_ST_BAD_TREE);
    } else if (t < N) {
      mark_partial(ws_ml, part_row + t, PARTIAL_BAD_TREE);
    }
    return;
  }
  constexpr int CG = D / 4;
  for (int idx = t; idx < NQ * CG; idx += NTHREADS) {
    const int nl = idx / CG, cg = idx % CG;
    const int n = q0 + nl;
    if (n >= N) continue;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) M = fmaxf(M, mg[(w * NQ + nl) * MROW + D]);
    const float M_use = (M == -INFINITY) ? 0.f : M;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    float l = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const float* row = mg + (w * NQ + nl) * MROW;
      const float wgt = __builtin_amdgcn_exp2f(row[D] - M_use);
      l += row[D + 1] * wgt;
      o += *(const f32x4*)(row + cg * 4) * wgt;
    }
    if (final_out) {
      const float inv = 1.f / l;
      union { uint2 u; __hip_bfloat16 h4[4]; } pk;
#pragma unroll
      for (int i = 0; i < 4; ++i) pk.h4[i] = __float2bfloat16(o[i] * inv);
      *(uint2*)(out + b * q_sb + n * q_sn + h * q_sh + cg * 4) = pk.u;
    } else {
      const long base = part_row + n;
      *(f32x4*)(ws_o + base * D + cg * 4) = o;
      if (cg == 0) {
        ws_ml[base * 2 + 0] = M;
        ws_ml[base * 2 + 1] = partial_sum(l, c1 == len);
      }
    }
  }
  };   // segment

  if constexpr (PLAN == 0) {
    // grid = (n_splits, H * n_qgroups, B): one fixed-size chunk of one (request, head, query group)
    const int split = blockIdx.x;
    const int h = uniform_div(blockIdx.y, n_qgroups), qg = blockIdx.y - h * n_qgroups;
    const int b = blockIdx.z;
    segment(b, h, qg, split * work, split * work + work,
            n_splits == 1 ? -1l : partial_row<false>(b, h, split, B, H, N, n_splits));
  } else if constexpr (PLAN == 2) {
    // Equal contiguous shares of all pairs' tiles; the workgroups overlapping a pair fill slots 0, 1, ... in order.
    const ContiguousDeal deal = contiguous_deal(prefix_len, B, N, H, S_cap, TILE, (int)gridDim.x);
    long pos = (long)blockIdx.x * deal.share;
    const long end = min(deal.total, pos + deal.share);
    if (pos >= end) return;
    const DealRequest first = contiguous_find(prefix_len, B, N, H, S_cap, TILE, pos);
    int b = first.b, tb = first.tiles;
    long req_start = first.start;
    while (pos < end) {
      while (pos >= req_start + (long)H * tb) {   // pos < total: a request with tiles left lies ahead
        req_start += (long)H * tb;
        ++b;
        tb = request_tiles(prefix_len[b], N, S_cap, TILE);
      }
      const long in_req = pos - req_start;
      const int h = uniform((int)deal_div(in_req, tb)), tile0 = uniform((int)(in_req - (long)h * tb));
      const int n_take = (int)min((long)(tb - tile0), end - pos);
      const int slot = (int)blockIdx.x - uniform((int)deal_div(req_start + (long)h * tb, deal.share));
      segment(b, h, 0, tile0 * TILE, (tile0 + n_take) * TILE, partial_row<true>(b, h, slot, B, H, N, n_splits));
      pos += n_take;
      __syncthreads();   // LDS (staging tiles, merge area, flags) is reused by the next segment
    }
  } else {
    // Balanced stream: the 32-key tiles of every pair in equal chunks, as many as the request's length asks for.
    const BalancedDeal deal = balanced_deal(prefix_len, B, N, H, S_cap, TILE, work);
    if ((long)blockIdx.x >= deal.count) return;
    const DealChunk c = deal_find(prefix_len, B, N, H, 1, S_cap, TILE, deal, blockIdx.x);
    if (c.n_tiles > 0) {
      segment(c.b, c.h, 0, c.tile0 * TILE, (c.tile0 + c.n_tiles) * TILE,
              c.chunks == 1 ? -1l : partial_row<true>(c.b, c.h, c.chunk, B, H, N, n_splits));
      if (c.chunks == 1 && t < N) mark_partial(ws_ml, partial_row<true>(c.b, c.h, 0, B, H, N, n_splits) + t, PARTIAL_FINAL);
    }
  }
}

hipError_t launch_tree_attention_bf16(const spec_attn_desc_t& d, const AttnPlan& plan, const Pages& pg, const void* q, void* k_cache,
                                      void* v_cache, const void* k_new, const void* v_new, const int32_t* parent,
                                      const int32_t* depth, const int32_t* prefix_len, void* out, void* ws,
                                      int32_t* status, hipStream_t s, const Rope& rope) {
  // This kernel: one 16-query tile per K/V head, k_new / v_new laid out like q. Larger trees, grouped-query
  // heads and separately laid out k_new go to the wide kernel (the plan decides).
  if (plan.wide)
    return launch_tree_attention_bf16_wide(d, plan, pg, q, k_cache, v_cache, k_new, v_new, parent, depth, prefix_len, out, ws,
                                           status, s, rope);
  const float scale = (d.softmax_scale != 0.f ? d.softmax_scale : 1.0f / sqrtf((float)d.D)) * kLog2eB;
  float* ws_o = ws ? (float*)((char*)ws + plan.ws_o_off) : nullptr;
  float* ws_ml = ws ? (float*)((char*)ws + plan.ws_ml_off) : nullptr;
  const int n_qgroups = 1;   // one 16-query tile covers the trees this kernel serves
  const bool append = k_new != nullptr;
  const bool bal = plan.balanced_wgs > 0;
  const dim3 grid = plan.contiguous ? dim3(plan.balanced_wgs, 1, 1) : bal ? dim3(balanced_grid(plan, d.B, d.H), 1, 1) : dim3(plan.n_splits, d.H * n_qgroups, d.B);
#define SPEC_LAUNCH(DD, NTT, APP, EA, PLAN, PGD)                                                                     \
  hipLaunchKernelGGL((tree_attention_bf16_kernel<DD, NTT, APP, EA, PLAN, PGD>), grid, dim3(WAVES * 64), 0, s,         \
                     (const __hip_bfloat16*)q, (__hip_bfloat16*)k_cache, (__hip_bfloat16*)v_cache,               \
                     (const __hip_bfloat16*)k_new, (const __hip_bfloat16*)v_new, parent, depth, prefix_len,      \
                     (__hip_bfloat16*)out, ws_o, ws_ml, status, d.B, d.N, d.H, d.S_cap, n_qgroups,               \
                     bal ? plan.balanced_wgs : plan.chunk_keys, plan.n_splits, (long)d.q_stride_b, (long)d.q_stride_n, (long)d.q_stride_h, \
                     (long)d.kv_stride_b, (long)d.kv_stride_h, (long)d.kv_stride_s, scale, pg, rope)
#define SPEC_DIMS(APP, EA, PLAN, PGD)                      \
  if (d.D == 128) SPEC_LAUNCH(128, 1, APP, EA, PLAN, PGD); \
  else SPEC_LAUNCH(64, 1, APP, EA, PLAN, PGD)
#define SPEC_PAGED(APP, EA, PLAN)                               \
  if (pg.table != nullptr) { SPEC_DIMS(APP, EA, PLAN, true); }  \
  else { SPEC_DIMS(APP, EA, PLAN, false); }
#define SPEC_DISPATCH(APP)                                  \
  if (plan.contiguous) { SPEC_PAGED(APP, false, 2); }              \
  else if (bal) { SPEC_PAGED(APP, false, 1); }                     \
  else { SPEC_PAGED(APP, false, 0); }
#define SPEC_EARLY(PLAN)                                                \
  if (pg.table != nullptr) SPEC_LAUNCH(128, 1, true, true, PLAN, true); \
  else SPEC_LAUNCH(128, 1, true, true, PLAN, false)
  if (append && rope.cos != nullptr && d.D == 128 && !plan.contiguous) {
    if (bal) { SPEC_EARLY(1); } else { SPEC_EARLY(0); }
  } else if (append) { SPEC_DISPATCH(true); } else { SPEC_DISPATCH(false); }
#undef SPEC_EARLY
#undef SPEC_DISPATCH
#undef SPEC_PAGED
#undef SPEC_DIMS
#undef SPEC_LAUNCH
  return hipGetLastError();
}

}  // namespace spec
