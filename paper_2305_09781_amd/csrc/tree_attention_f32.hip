// Tree attention for float32 inputs (Definition 4.1 with the topology-aware causal mask of Section
// 4.2), plus the split-combine step shared with the bf16 kernels.
//
// float32 K/V cannot use the bf16 matrix cores without losing the accuracy this dtype is held to, so both products
// run on v_mfma_f32_16x16x4_f32 (exact float32 products, float32 accumulation: as many operations per cycle as the
// vector unit's float32 fma, without its operand traffic).
//
// Work split: a workgroup owns one chunk of the key range of one (request, K/V head) and NT 16-query tiles of the
// group * N queries that share that head (query index = head in group * N + node). Its four wavefronts take the
// chunk's 16-key tiles round-robin, each with its own online softmax and no barrier in the loop, and are merged
// through LDS at the end; the workgroup writes the final output (one chunk) or a partial (m, l, O) that
// attn_combine_kernel merges.
//
// Layouts. S^T = K Q^T is taken with the head dimension permuted the same way for K and Q, so that a lane's operands
// are whole 16-byte pieces: lane (r, g) of a tile holds pieces 4j + g of key r (K, straight from global memory) and of
// query r (Q). The product leaves it with query r's scores for keys 4g + i, which is the operand O^T += V^T P^T wants
// for k-step i with row 4g + i of V in 16-byte pieces again: neither K, V nor the probabilities pass through LDS.
//
// Precision. A score is four sums of D / 4 products, added in pairs: with two sums of D / 2 the outputs over short key ranges,
// whose error is that of the scores, were further from float64 than those of a plain float32 loop with four sums (relative
// error over 59 keys, D = 128: 2.15e-7 with two, 2.0e-7 for the loop, 1.7e-7 with four; over 2000 keys 3.0e-7, 3.8e-7,
// 2.5e-7). The four cost 0 to 1 % (3 % for 16 requests x 32 / 8 heads, trees of 33, 2000 keys: 262 -> 271 us). exp2 is
// v_exp_f32: probabilities below 2^-126 of the largest are 0 instead of subnormal.
//
// What bounds it: float32 MFMA rate and the stream of K/V are close to each other (16 keys x 16 queries x 128
// dimensions are 2048 cycles of one SIMD for 16 KB); small calls, one trip to memory after the other. So the tree words are requested
// before the tiles and the masks built by one wavefront (a parent chain walked after two barriers and a dependent load before), new rows go
// to the cache from the registers of the tile that uses them (read a second time before), and the scores wait for K and the queries but not
// for V. Measured, us a layer as nodes of a graph over 600 MB of caches, before / now: 4 requests x 32 heads x 128, 300 to 1000 keys, trees
// of 24 (95 MB), append and merge launch included 41.0 / 38.5 (2.5 TB/s, 27 TFLOP/s); 1 x 4 heads x 64, 128 keys, trees of 8, 7.8 / 7.5; 32 x
// 32 heads x 128, 100 keys, trees of 8, 37.2 / 35.2; 8 x 32 heads x 64, 1000 keys, trees of 32, 47.5 / 39.5.
// One tile is on its way per wavefront. A second register set was measured for every instance and is not used: it costs a wavefront per
// SIMD (and spills at D = 128), and each wavefront requests a second tile whether it has one or not. us, one set / two: 32 x 32 heads of
// 100 keys, trees of 8, D = 128 35.1 / 39.4, D = 64 19.4 / 22.6; 1 x 12 of 40 keys, 3, D = 128 6.3 / 7.4; 8 x 32 of 500-1000, 16, D = 128
// 51.9 / 53.5; 16 x 32 of 300, 20, D = 64 26.2 / 28.7. The one gain is two query tiles at D = 64 over long uncut ranges with a workgroup
// per compute unit (8 x 32 heads of 2000 keys: trees of 24 65.6 / 63.2, of 32 75.1 / 75.7), too narrow a range for an instance of its own.
// Keeping the queries in LDS to pay for a second set at D = 128 with two query tiles spills too (50 us).
#include <hip/hip_bf16.h>

#include <algorithm>
#include <type_traits>

#include "spec_internal.h"

namespace spec {

constexpr int F32_WAVES = 4;     // wavefronts per workgroup
constexpr int F32_TK = 16;       // keys per wavefront tile
constexpr float kLog2e = 1.4426950408889634f;

typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ void f32_lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// APPEND: rows >= prefix_len are taken from k_new / v_new, and the workgroups of the first query group write them to
// the cache (also for a malformed tree: the append does not depend on it).
template <int D, int NT, bool APPEND>
__global__ void __launch_bounds__(F32_WAVES * 64, 2) tree_attention_f32_kernel(
    const float* __restrict__ q, float* k_cache, float* v_cache, const float* __restrict__ k_new,
    const float* __restrict__ v_new, const int32_t* __restrict__ parent, const int32_t* __restrict__ depth,
    const int32_t* __restrict__ prefix_len, float* __restrict__ out, float* __restrict__ ws_o, float* __restrict__ ws_ml,
    int32_t* status, int B, int N, int H, int H_kv, int S_cap, int n_qg, int chunk_keys, int n_splits, long q_sb, long q_sn,
    long q_sh, long n_sb, long n_sn, long n_sh, long kv_sb, long kv_sh, long kv_ss, float scale_log2, Pages pg) {
  constexpr int NTHREADS = F32_WAVES * 64;
  constexpr int KJ = D / 16;       // 16-byte pieces of a K row per lane
  constexpr int VH = D / 64;       // 16-byte pieces of a V row per lane
  constexpr int QT = NT * 16;      // queries of the workgroup
  constexpr int OROW = D + 4;      // floats per merged output row in LDS (+4: rows start on different banks)
  __shared__ float s_o[F32_WAVES][QT][OROW];
  __shared__ float s_m[F32_WAVES][QT], s_l[F32_WAVES][QT];
  __shared__ TreeLds s_tree;

  // The query groups of one chunk read the same K/V: they are numbered eight apart, which puts them on one XCD (
  // workgroups go to the eight XCDs round-robin), close in time, so that the repeats can be hits of its L2.
  const int blk = uniform(blockIdx.x / (8 * n_qg)), in_blk = blockIdx.x - blk * 8 * n_qg;
  const int qg = in_blk / 8;
  const int pc = blk * 8 + in_blk % 8;
  if (pc >= B * H_kv * n_splits) return;
  const int pair = uniform_div(pc, n_splits), split = pc - pair * n_splits;
  const int b = uniform_div(pair, H_kv), hk = pair - b * H_kv;
  const int group = uniform_div(H, H_kv), M = group * N;   // queries that share this K/V head
  const int t = threadIdx.x, lane = t & 63, r16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);

  // the tree words first: what waits for them then leaves the tiles in flight
  const int my_parent = parent[(long)b * N + min(t, N - 1)], my_depth = depth[(long)b * N + min(t, N - 1)];
  const int P = prefix_len[b];
  const bool cap_ok = (P >= 0) && (P <= S_cap - N);
  const int len = P + N;
  const int c0 = split * chunk_keys;
  const int c1 = min(c0 + chunk_keys, len);
  // query row qi of this workgroup: head in the group and node
  auto query_off = [&](int qi) { return b * q_sb + (long)(qi % N) * q_sn + (long)(hk * group + qi / N) * q_sh; };
  auto fail = [&](int bit) {   // a request without a result: zeros, from the workgroups that own final outputs
    if (n_splits != 1) {
      const int qi = qg * QT + t;
      if (bit == SPEC_ST_BAD_TREE && t < QT && qi < M)
        mark_partial(ws_ml, partial_row<false>(b, hk * group + qi / N, split, B, H, N, n_splits) + qi % N, PARTIAL_BAD_TREE);
      return;
    }
    for (int i = t; i < QT * (D / 4); i += NTHREADS) {
      const int qi = qg * QT + i / (D / 4);
      if (qi < M) *(float4*)(out + query_off(qi) + (i % (D / 4)) * 4) = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (hk == 0 && qg == 0 && t == 0) set_status(status, b, bit);
  };
  if (!cap_ok) {
    if (APPEND && hk == 0 && qg == 0 && split == 0 && t == 0) set_status(status, b, SPEC_ST_CAPACITY);
    fail(SPEC_ST_CAPACITY);
    return;
  }
  if (c0 >= len) return;   // the combine step never reads this split

  // ---- first tile of this wavefront, queries, tree
  const float* kn = APPEND ? k_new + b * n_sb + hk * n_sh : nullptr;
  const float* vn = APPEND ? v_new + b * n_sb + hk * n_sh : nullptr;
  const int n_tiles = (c1 - c0 + F32_TK - 1) / F32_TK;
  float4 kf[KJ], vf[4][VH];   // one tile (see "What bounds it" for a second one)
  // A tile starts at a multiple of 16 rows, so it lies inside one block of a paged cache; rows past the chunk repeat its
  // last one (their scores are masked).
  auto tile_base = [&](int k0) {
    bool blk_ok;
    const long off = cache_row_offset(pg, b, k0, kv_sb, kv_ss, &blk_ok) - k0 * kv_ss + hk * kv_sh;
    if (!blk_ok && lane == 0) set_status(status, b, SPEC_ST_BAD_BLOCK);
    return off;
  };
  auto load_k = [&](int k0, long base) {
    const int row = min(k0 + r16, c1 - 1);
    const float* p = (APPEND && row >= P) ? kn + (long)(row - P) * n_sn : k_cache + base + (long)row * kv_ss;
#pragma unroll
    for (int j = 0; j < KJ; ++j) kf[j] = *(const float4*)(p + (4 * j + g) * 4);
  };
  auto load_v = [&](int k0, long base) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = min(k0 + 4 * g + i, c1 - 1);
      const float* p = (APPEND && row >= P) ? vn + (long)(row - P) * n_sn : v_cache + base + (long)row * kv_ss;
#pragma unroll
      for (int hv = 0; hv < VH; ++hv) vf[i][hv] = *(const float4*)(p + r16 * 4 + 64 * hv);
    }
  };
  int ti = wave;
  // The first tile's K, the queries, its V: the scores need the first two only. (Unconditional, so that the compiler knows how many
  // loads stand behind each: a wavefront without a tile takes the chunk's last row for all of its own, one line per load. us, before these
  // loads were unconditional / with the last tile / now: 1 x 12 heads of 14 keys, one node, D = 128, 5.7 / 6.2 / 5.9, 8 x 32 of 12-14, 2, 6.1 /
  // 6.5 / 6.2; 32 x 32 of 20, 8, D = 64, 9.0 / 9.5 / 9.3; 3 x 12 of 40-60, 2, D = 128, 7.0 / 6.4 / 6.4.)
  const int first = ti < n_tiles ? c0 + ti * F32_TK : c1 - 1;
  const long first_base = tile_base(first);
  load_k(first, first_base);
  float4 qf[NT][KJ];
  int node[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int qi = min(qg * QT + nt * 16 + r16, M - 1);
    node[nt] = qi % N;
    const float* p = q + query_off(qi);
#pragma unroll
    for (int j = 0; j < KJ; ++j) qf[nt][j] = *(const float4*)(p + (4 * j + g) * 4);
  }
  load_v(first, first_base);
  const bool touches_tree = c1 > P;
  // one workgroup per request owns the final outputs' validity: every workgroup of a single chunk checks the tree; with
  // several chunks only those that reach it do (the combine step gives a malformed request its zeros)
  if (touches_tree) {
    if (t < N) {
      s_tree.parent[t] = my_parent;
      s_tree.depth[t] = my_depth;
    }
    f32_lds_barrier();
    if (wave == 0) {
      const bool bad = tree_masks_by_wave(s_tree, N, lane, my_parent, my_depth);
      if (lane == 0) s_tree.bad[0] = bad;
    }
    f32_lds_barrier();
    if (s_tree.bad[0]) {
      if (APPEND && qg == 0) {   // the chunk's new rows go to the cache all the same
        const int r0 = max(P, c0);
        for (int i = t; i < (c1 - r0) * (D / 4); i += NTHREADS) {
          const int row = r0 + i / (D / 4), c = (i % (D / 4)) * 4;
          bool blk_ok;
          const long dst = cache_row_offset(pg, b, row, kv_sb, kv_ss, &blk_ok) + hk * kv_sh + c;
          if (!blk_ok && c == 0) set_status(status, b, SPEC_ST_BAD_BLOCK);
          if (blk_ok) {
            *(float4*)(k_cache + dst) = *(const float4*)(kn + (long)(row - P) * n_sn + c);
            *(float4*)(v_cache + dst) = *(const float4*)(vn + (long)(row - P) * n_sn + c);
          }
        }
      }
      fail(SPEC_ST_BAD_TREE);
      return;
    }
  }

  f32x4 O[NT][VH * 4];
  float m_run[NT], l_run[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    m_run[nt] = -INFINITY;
    l_run[nt] = 0.f;
#pragma unroll
    for (int x = 0; x < VH * 4; ++x) O[nt][x] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }

  // ---- tiles of this wavefront. The next tile's K is requested when this tile's scores are done, its V when this tile's output
  // products are: each load has the other product's time to arrive. With and without a next tile are two bodies: behind a branch
  // around the requests the compiler would wait for more than it has to.
  auto step = [&](const int ti, auto refill_tag) {
    constexpr bool REFILL = decltype(refill_tag)::value;
    const int k0 = c0 + ti * F32_TK;
    const int k1 = c0 + (REFILL ? ti + F32_WAVES : ti) * F32_TK;
    const long base1 = REFILL ? tile_base(k1) : 0;
    const bool masked = k0 + F32_TK > min(P, c1);
    // New rows go to the cache from the tile's registers (a row of a block outside the pool is not written).
    bool dst_ok = false;
    const long dst = APPEND && masked && qg == 0 ? cache_row_offset(pg, b, k0, kv_sb, kv_ss, &dst_ok) - k0 * kv_ss + hk * kv_sh : 0;
    if (APPEND && dst_ok) {
      const int row = k0 + r16;
      if (row >= P && row < c1) {
#pragma unroll
        for (int j = 0; j < KJ; ++j) *(float4*)(k_cache + dst + (long)row * kv_ss + (4 * j + g) * 4) = kf[j];
      }
    }
    f32x4 sc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {   // (one query tile after the other: eight sums at once do not fit the registers)
      f32x4 part[4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int j = 0; j < KJ; ++j) {
        const float a[4] = {kf[j].x, kf[j].y, kf[j].z, kf[j].w};
        const float bq[4] = {qf[nt][j].x, qf[nt][j].y, qf[nt][j].z, qf[nt][j].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) part[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], bq[e], part[e], 0, 0, 0);
      }
      sc[nt] = (part[0] + part[1]) + (part[2] + part[3]);
    }
    if (REFILL) load_k(k1, base1);
    float p[NT][4];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      float s[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) s[i] = sc[nt][i] * scale_log2;
      if (masked) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int key = k0 + 4 * g + i, rel = key - P;
          bool vis = key < c1;
          if (vis && rel >= 0) vis = (s_tree.anc[node[nt]][rel >> 6] >> (rel & 63)) & 1ull;
          if (!vis) s[i] = -INFINITY;
        }
      }
      // Lazy running maximum (identical in the four lanes of a query): refreshed, with the exact cross-lane maximum and
      // the rescaling of l and O, only when a score exceeds it by more than 2^16 in the exp2 domain.
      float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
      if (__any(mx > m_run[nt] + 16.f)) {
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m_run[nt], mx);
        const float alpha = __builtin_amdgcn_exp2f(m_run[nt] - (m_new == -INFINITY ? 0.f : m_new));
        m_run[nt] = m_new;
        l_run[nt] *= alpha;
#pragma unroll
        for (int x = 0; x < VH * 4; ++x) O[nt][x] *= alpha;
      }
      const float m_use = m_run[nt] == -INFINITY ? 0.f : m_run[nt];
#pragma unroll
      for (int i = 0; i < 4; ++i) p[nt][i] = __builtin_amdgcn_exp2f(s[i] - m_use);
      l_run[nt] += (p[nt][0] + p[nt][1]) + (p[nt][2] + p[nt][3]);
    }
    if (APPEND && dst_ok) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = k0 + 4 * g + i;
        if (row >= P && row < c1) {
#pragma unroll
          for (int hv = 0; hv < VH; ++hv) *(float4*)(v_cache + dst + (long)row * kv_ss + r16 * 4 + 64 * hv) = vf[i][hv];
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int hv = 0; hv < VH; ++hv) {
        const float a[4] = {vf[i][hv].x, vf[i][hv].y, vf[i][hv].z, vf[i][hv].w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
            O[nt][hv * 4 + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], p[nt][i], O[nt][hv * 4 + e], 0, 0, 0);
      }
    if (REFILL) load_v(k1, base1);
  };
  for (; ti + F32_WAVES < n_tiles; ti += F32_WAVES) step(ti, std::true_type{});
  if (ti < n_tiles) step(ti, std::false_type{});

  // ---- merge of the four wavefronts: each scales its state to the common maximum, then all threads add the rows
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    float l = l_run[nt];
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (g == 0) {
      s_m[wave][nt * 16 + r16] = m_run[nt];
      s_l[wave][nt * 16 + r16] = l;
    }
  }
  f32_lds_barrier();
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    float m_all = s_m[0][nt * 16 + r16];
#pragma unroll
    for (int w = 1; w < F32_WAVES; ++w) m_all = fmaxf(m_all, s_m[w][nt * 16 + r16]);
    const float f = m_run[nt] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run[nt] - m_all);
#pragma unroll
    for (int hv = 0; hv < VH; ++hv)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *(float4*)&s_o[wave][nt * 16 + r16][(4 * g + i) * 4 + 64 * hv] =
            make_float4(O[nt][hv * 4][i] * f, O[nt][hv * 4 + 1][i] * f, O[nt][hv * 4 + 2][i] * f, O[nt][hv * 4 + 3][i] * f);
  }
  f32_lds_barrier();
  for (int i = t; i < QT * (D / 4); i += NTHREADS) {
    const int row = i / (D / 4), c = (i % (D / 4)) * 4;
    const int qi = qg * QT + row;
    if (qi >= M) break;
    float m_all = s_m[0][row];
#pragma unroll
    for (int w = 1; w < F32_WAVES; ++w) m_all = fmaxf(m_all, s_m[w][row]);
    float l = 0.f;
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < F32_WAVES; ++w) {
      const float mw = s_m[w][row];
      if (mw != -INFINITY) l += s_l[w][row] * __builtin_amdgcn_exp2f(mw - m_all);
      const float4 ow = *(const float4*)&s_o[w][row][c];
      o.x += ow.x; o.y += ow.y; o.z += ow.z; o.w += ow.w;
    }
    if (n_splits == 1) {
      const float inv = 1.f / l;
      o.x *= inv; o.y *= inv; o.z *= inv; o.w *= inv;
      *(float4*)(out + query_off(qi) + c) = o;
    } else {
      const long slot = partial_row<false>(b, hk * group + qi / N, split, B, H, N, n_splits) + qi % N;
      *(float4*)(ws_o + slot * D + c) = o;
      if (c == 0) {
        ws_ml[slot * 2 + 0] = m_all;
        ws_ml[slot * 2 + 1] = partial_sum(l, c1 == len);
      }
    }
  }
}

// Merge of the partials of one (request, head): out = sum_s O_s 2^(m_s - M) / sum_s l_s 2^(m_s - M),
// M = max_s m_s. grid = (H, B, ceil(N * D/4 / 256)), 256 threads; a thread owns 4 consecutive d of one
// query. A pair has a block of N rows in each of `slots` slots, filled from 0; which is the last, whether the tree was malformed
// and whether the output is there already, the partials themselves say (see partial_sum). Also the place where a malformed
// request gets its defined result (zeros) and its status bit. Bound by its launch and one trip to memory, and in large batches by
// reading the filled slots once. (With a tree check, two barriers and under the balanced plans the deal in front of the merge: 32
// layers of one request, 32 heads, 1024 keys, a pass 487 us, 476 now; 4 x 32 heads of 8192 to 16384 keys 137.3, 136.3.)
template <bool BF16, bool BAL, int CH>   // CH: partial slots fetched together
__global__ void __launch_bounds__(256) attn_combine_kernel(const float* __restrict__ ws_o, const float* __restrict__ ws_ml,
                                                           const int32_t* __restrict__ prefix_len, void* __restrict__ out,
                                                           int32_t* status, int B, int N, int H, int D, int S_cap, int chunk_keys,
                                                           int slots, long q_sb, long q_sn, long q_sh) {
  const int h = blockIdx.x, b = blockIdx.y, t = threadIdx.x;
  const int CG = D / 4;
  const int idx = blockIdx.z * 256 + t;
  if (idx >= N * CG) return;
  const int n = idx / CG, cg = idx % CG;
  const long base = partial_row<BAL>(b, h, 0, B, H, N, slots) + n, slot_rows = BAL ? (long)B * H * N : N;
  // The first slots are fetched before anything is known about the request (every slot exists in the
  // workspace, whatever it holds): of fixed chunks up to eight, which a request near the stated maximum has filled (1 request of
  // 8000 keys on 8 K/V heads, 31 slots: 23.3 -> 21.9 us with attention; 5 slots: 13.6 -> 13.5), of a balanced deal two, as most
  // pairs have no more (a third is 17 MB for 32 requests x 64 heads x 16 nodes).
  float m_s[CH], l_s[CH];
  float4 o_s[CH];
  auto fetch = [&](int s0, int take) {
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      if (j < take) {
        const long row = base + min(s0 + j, slots - 1) * slot_rows;
        const float2 ml = *(const float2*)(ws_ml + row * 2);
        m_s[j] = ml.x;
        l_s[j] = ml.y;
        o_s[j] = *(const float4*)(ws_o + row * D + cg * 4);
      }
    }
  };
  int take = BAL ? 2 : CH;
  fetch(0, take);
  const int P = prefix_len[b];
  const bool cap_ok = (P >= 0) && (P <= S_cap - N);
  // fixed chunks: known from the length; balanced: until a slot says that it is the last
  const int ns = !cap_ok ? 0 : BAL ? slots : min(slots, uniform_div(P + N + chunk_keys - 1, chunk_keys));
  int bit = cap_ok ? 0 : SPEC_ST_CAPACITY;
  // online merge over groups of slots (those behind the last one hold nothing meaningful)
  float M = -INFINITY, l = 0.f;
  float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s0 = 0; s0 < ns;) {
    if (s0 > 0) fetch(s0, take);
    int filled = min(take, ns - s0);
    bool last = false;
#pragma unroll
    for (int j = 0; j < CH; ++j)
      if (j < filled && uniform((int)(BAL ? partial_ends(m_s[j], l_s[j]) : m_s[j] != m_s[j])) != 0) {   // the same for a pair's rows
        if (uniform((int)(m_s[j] != m_s[j])) != 0) {
          if (BAL && l_s[j] == PARTIAL_FINAL) return;
          bit = SPEC_ST_BAD_TREE;
        }
        filled = j + 1;   // (the slots behind it are not looked at any more)
        last = true;
      }
    if (bit != 0) break;
    float Mc = M;
#pragma unroll
    for (int j = 0; j < CH; ++j)
      if (j < filled) Mc = fmaxf(Mc, m_s[j]);
    const float keep = (M == -INFINITY) ? 0.f : exp2f(M - Mc);   // Mc = -inf only while nothing carried mass
    l *= keep;
    o.x *= keep; o.y *= keep; o.z *= keep; o.w *= keep;
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      if (j < filled && m_s[j] != -INFINITY) {   // an all-masked partial carries nothing
        const float w = exp2f(m_s[j] - Mc);
        l = fmaf(fabsf(l_s[j]), w, l);
        o.x = fmaf(o_s[j].x, w, o.x); o.y = fmaf(o_s[j].y, w, o.y); o.z = fmaf(o_s[j].z, w, o.z); o.w = fmaf(o_s[j].w, w, o.w);
      }
    }
    M = Mc;
    if (last) break;
    s0 += take;
    if (BAL && s0 >= 4) take = CH;
  }
  if (bit != 0) {
    if (h == 0 && idx == 0) set_status(status, b, bit);
    l = 0.f;
    o = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  const float inv = (l > 0.f) ? 1.f / l : 0.f;
  o.x *= inv; o.y *= inv; o.z *= inv; o.w *= inv;
  const long off = b * q_sb + n * q_sn + h * q_sh + cg * 4;
  if (BF16) {
    __hip_bfloat16* ob = (__hip_bfloat16*)out + off;
    union { uint2 u; __hip_bfloat16 h4[4]; } pk;
    pk.h4[0] = __float2bfloat16(o.x); pk.h4[1] = __float2bfloat16(o.y);
    pk.h4[2] = __float2bfloat16(o.z); pk.h4[3] = __float2bfloat16(o.w);
    *(uint2*)ob = pk.u;
  } else {
    *(float4*)((float*)out + off) = o;
  }
}

hipError_t launch_tree_attention_f32(const spec_attn_desc_t& d, const AttnPlan& plan, const Pages& pg, const float* q,
                                     float* k_cache, float* v_cache, const float* k_new, const float* v_new,
                                     const int32_t* parent, const int32_t* depth, const int32_t* prefix_len, float* out,
                                     void* ws, int32_t* status, hipStream_t s) {
  const float scale = (d.softmax_scale != 0.f ? d.softmax_scale : 1.0f / sqrtf((float)d.D)) * kLog2e;
  float* ws_o = ws ? (float*)((char*)ws + plan.ws_o_off) : nullptr;
  float* ws_ml = ws ? (float*)((char*)ws + plan.ws_ml_off) : nullptr;
  const int nt = f32_query_tiles(d), n_qg = f32_query_groups(d);
  const NewStrides ns = attn_new_strides(d);
  const long chunks = (long)d.B * d.H_kv * plan.n_splits;
  const long wgs = (chunks + 7) / 8 * 8 * n_qg;
  if (wgs > 0x7fffffffL) return hipErrorInvalidConfiguration;
#define SPEC_F32(DD, NTT, APP)                                                                                            \
  hipLaunchKernelGGL((tree_attention_f32_kernel<DD, NTT, APP>), dim3((unsigned)wgs), dim3(F32_WAVES * 64), 0, s, q, k_cache, \
                     v_cache, k_new, v_new, parent, depth, prefix_len, out, ws_o, ws_ml, status, d.B, d.N, d.H, d.H_kv,     \
                     d.S_cap, n_qg, plan.chunk_keys, plan.n_splits, (long)d.q_stride_b, (long)d.q_stride_n,                 \
                     (long)d.q_stride_h, ns.b, ns.n, ns.h, (long)d.kv_stride_b, (long)d.kv_stride_h, (long)d.kv_stride_s,   \
                     scale, pg)
#define SPEC_F32_APP(DD, NTT)                                \
  if (k_new != nullptr) { SPEC_F32(DD, NTT, true); }         \
  else { SPEC_F32(DD, NTT, false); }
#define SPEC_F32_NT(DD)                                      \
  if (nt == 1) { SPEC_F32_APP(DD, 1); }                      \
  else { SPEC_F32_APP(DD, 2); }
  if (d.D == 64) { SPEC_F32_NT(64); } else { SPEC_F32_NT(128); }
#undef SPEC_F32_NT
#undef SPEC_F32_APP
#undef SPEC_F32
  return hipGetLastError();
}

hipError_t launch_attn_combine(const spec_attn_desc_t& d, const AttnPlan& plan, const int32_t* prefix_len, const void* ws,
                               void* out, int32_t* status, hipStream_t s) {
  const float* ws_o = (const float*)((const char*)ws + plan.ws_o_off);
  const float* ws_ml = (const float*)((const char*)ws + plan.ws_ml_off);
  const int items = d.N * (d.D / 4);
  dim3 grid(d.H, d.B, (items + 255) / 256);
#define SPEC_COMBINE(BF, BL, CH)                                                                                              \
  hipLaunchKernelGGL((attn_combine_kernel<BF, BL, CH>), grid, dim3(256), 0, s, ws_o, ws_ml, prefix_len, out, status, d.B, d.N, \
                     d.H, d.D, d.S_cap, plan.chunk_keys, plan.n_splits, (long)d.q_stride_b, (long)d.q_stride_n, (long)d.q_stride_h)
  const bool many = plan.n_splits > 4;
  if (plan.balanced_wgs > 0) { SPEC_COMBINE(true, true, 4); }   // (bf16 only)
  else if (d.dtype == SPEC_BF16 && many) { SPEC_COMBINE(true, false, 8); }
  else if (d.dtype == SPEC_BF16) { SPEC_COMBINE(true, false, 4); }
  else if (many) { SPEC_COMBINE(false, false, 8); }
  else { SPEC_COMBINE(false, false, 4); }
#undef SPEC_COMBINE
  return hipGetLastError();
}

}  // namespace spec
