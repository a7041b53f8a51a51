// C ABI of libspectree: host-side argument checks and kernel launches. Every entry point validates
// what the host can see, enqueues its kernels on the caller's stream and returns; nothing here
// allocates or synchronises.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>

#include "spec_internal.h"

// Scratch of spec_tree_attention_append_static: the split plans' float32 partial results, for callers that can
// neither allocate nor bring a workspace. Part of the code object, so every GPU that loads the library holds
// its own copy at its own address. In host code this name is only a handle for hipGetSymbolAddress; the
// device address it returns is what kernels and copies take.
static __device__ __align__(256) unsigned char scratch[SPEC_STATIC_SCRATCH_BYTES];

namespace spec {

// Device address of `scratch` on the current device, looked up once per device.
static int static_scratch(void** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* ptr[kMaxDevices] = {};
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SPEC_ERR_HIP;
  std::lock_guard<std::mutex> lock(mu);
  if (ptr[dev] == nullptr) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return SPEC_ERR_HIP;
    ptr[dev] = p;
  }
  *out = ptr[dev];
  return SPEC_OK;
}

static inline int elem_bytes(int dtype) { return dtype == SPEC_F32 ? 4 : 2; }
static inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
static inline size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Host-checkable part of the attention descriptor. Returns SPEC_OK or an error code.
static int check_desc(const spec_attn_desc_t* d) {
  if (d == nullptr) return SPEC_ERR_INVALID_ARG;
  if (d->B <= 0 || d->H <= 0 || d->H_kv <= 0 || d->N <= 0 || d->S_cap <= 0 || d->D <= 0) return SPEC_ERR_INVALID_ARG;
  if (d->plan_chunk_keys < 0 || d->plan_balanced_wgs < -1 || d->plan_heads_per_wg < 0) return SPEC_ERR_INVALID_ARG;
  if (d->dtype != SPEC_F32 && d->dtype != SPEC_BF16) return SPEC_ERR_UNSUPPORTED;
  if (d->D != 64 && d->D != 128) return SPEC_ERR_UNSUPPORTED;
  if (d->N > SPEC_MAX_TREE_NODES) return SPEC_ERR_UNSUPPORTED;
  if (d->H % d->H_kv != 0) return SPEC_ERR_UNSUPPORTED;
  {
    const bool none = d->new_stride_b == 0 && d->new_stride_n == 0 && d->new_stride_h == 0;
    if (!none && (d->new_stride_b <= 0 || d->new_stride_n <= 0 || d->new_stride_h < d->D)) return SPEC_ERR_INVALID_ARG;
  }
  if (d->N > d->S_cap) return SPEC_ERR_CAPACITY;
  if (d->max_prefix_len < 0 || (long)d->max_prefix_len + d->N > d->S_cap) return SPEC_ERR_CAPACITY;
  if (!(d->softmax_scale >= 0.f) || std::isinf(d->softmax_scale)) return SPEC_ERR_INVALID_ARG;
  const int per16 = 16 / elem_bytes(d->dtype);
  const int64_t strides[6] = {d->q_stride_b, d->q_stride_n, d->q_stride_h, d->kv_stride_b, d->kv_stride_h, d->kv_stride_s};
  for (int64_t s : strides)
    if (s <= 0 || s % per16 != 0) return SPEC_ERR_INVALID_ARG;
  const int64_t new_strides[3] = {d->new_stride_b, d->new_stride_n, d->new_stride_h};
  for (int64_t s : new_strides)
    if (s % per16 != 0) return SPEC_ERR_INVALID_ARG;
  if (d->q_stride_h < d->D || d->kv_stride_s < d->D) return SPEC_ERR_INVALID_ARG;
  // the kernels compute row offsets inside one (request, head) span (paged: one block) in 32 bits
  if ((double)d->S_cap * (double)d->kv_stride_s * elem_bytes(d->dtype) >= 4294967296.0) return SPEC_ERR_UNSUPPORTED;
  return SPEC_OK;
}

// k_new / v_new cannot share q's layout when there are fewer K/V heads than query heads.
static bool new_strides_missing(const spec_attn_desc_t* d) {
  return d->H_kv != d->H && d->new_stride_b == 0 && d->new_stride_n == 0 && d->new_stride_h == 0;
}

// Host-checkable part of a paged-cache description; fills the form the kernels take.
static int check_pages(const spec_attn_desc_t* d, const spec_kv_pages_t* p, Pages* out) {
  if (p == nullptr || p->block_table == nullptr || p->max_blocks <= 0 || p->n_blocks <= 0) return SPEC_ERR_INVALID_ARG;
  const int bt = p->block_tokens;
  if (bt < 64 || bt > 65536 || (bt & (bt - 1)) != 0) return SPEC_ERR_UNSUPPORTED;
  if ((long)d->S_cap > (long)p->max_blocks * bt) return SPEC_ERR_CAPACITY;
  int lg = 0;
  while ((1 << lg) < bt) ++lg;
  *out = Pages{p->block_table, p->max_blocks, lg, p->n_blocks};
  return SPEC_OK;
}

// Compute units of the current device (256 when no device can be queried, e.g. sizing a workspace on a
// machine without a GPU). Asked on every call: the answer belongs to the device that is current now.
int compute_units() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) == hipSuccess &&
      hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
    return n;
  return 256;
}

AttnPlan make_attn_plan(const spec_attn_desc_t& d, bool paged) {
  AttnPlan p;
  p.balanced_wgs = 0;
  p.contiguous = false;
  p.heads_per_wg = 1;
  p.m32 = false;
  const int max_prefix = d.max_prefix_len > 0 ? d.max_prefix_len : d.S_cap - d.N;
  const int max_len = max_prefix + d.N;
  // bf16: one workgroup serves all query heads of a K/V head; float32: one per one or two query tiles
  const QueryGroups qg = attn_query_groups(d);
  const int virtual_heads = d.H_kv * qg.n_qgroups;
  const long groups = (long)d.B * (d.dtype == SPEC_BF16 ? virtual_heads : d.H_kv * f32_query_groups(d));
  const int tiles = qg.tiles_per_wg;   // 16-query tiles per workgroup
  // The few-query kernel serves one query tile per K/V head with k_new / v_new laid out like q; everything
  // else in bf16 runs on the wide kernel.
  const NewStrides ns = attn_new_strides(d);
  p.wide = d.dtype == SPEC_BF16 &&
           (tiles > 1 || ns.b != d.q_stride_b || ns.n != d.q_stride_n || ns.h != d.q_stride_h);
  int chunk = d.plan_chunk_keys;   // caller's hint; 0 = chosen below
  // Five to eight query tiles: four wavefronts of 32 queries unless the caller asks for several heads per
  // workgroup, which only the eight-wavefront shape serves.
  p.m32 = p.wide && tiles > 4 && d.D == 128 && d.plan_heads_per_wg == 0;
  // workgroups the device holds at once: four-wavefront shapes of the wide kernel run two per compute unit
  const long resident = (long)compute_units() * ((p.wide && (tiles <= 4 || p.m32)) ? 2 : 1);
  const int tile = p.wide ? SPEC_WIDE_TILE_KEYS : SPEC_SMALL_TILE_KEYS;
  if (chunk <= 0 && d.dtype == SPEC_BF16) {
    // Several requests with few (request, head) pairs and long key ranges (long-context serving, ragged lengths): the
    // bf16 kernels cut every pair's key tiles into as many equal chunks as its length asks for, about as many in all as
    // the device holds workgroups, so the stream is balanced whatever the individual lengths are. Against fixed chunks of
    // the stated maximum the deal costs 1 to 3 us of reading prefix_len[] first, and saves what unequal lengths leave
    // idle (8 requests of 512 to 16384 keys: 257 us uncut, 195 us dealt to 512 chunks; 4 requests of 8192 to 16384: 138
    // us either way): it is used for at least 2048 keys per chunk at the stated maximum length, where 3 us are small
    // next to either. One request has no lengths to balance: fixed chunks.
    int wgs = d.plan_balanced_wgs;   // caller's hint: > 0 that many workgroups, -1 never, 0 = chosen here
    if (wgs < 0) {
      wgs = 0;
    } else if (wgs == 0) {
      const long max_tiles = groups * ((max_len + tile - 1) / tile);
      long cand = (max_tiles * tile / resident >= 2048) ? resident : 0;
      // every workgroup writes (and the combine step reads back) float32 partials for all queries of its
      // pair: keep that traffic under three fifths of the K/V stream (it matters with grouped-query heads,
      // where a pair has many queries and the batch few pairs; a quarter left too few chunks to balance: 2 x 64/8 heads of 16000
      // keys, trees of 128, 408 us, 178 now), as long as the partials fit the library's own scratch array; a quarter where they
      // would not.
      const double stream_bytes = (double)d.B * d.H_kv * max_len * d.D * 2.0 * 2.0;
      const double partial_bytes_per_wg = 2.0 * (double)qg.heads_per_wg * d.N * (d.D + 2) * 4.0;
      const double slot_bytes = (double)d.B * d.H * d.N * (d.D + 2) * 4.0;
      const long fitting = ((long)(((double)SPEC_STATIC_SCRATCH_BYTES - 512.0) / slot_bytes) - 1) * virtual_heads;
      cand = std::min<long>(cand, std::max<long>((long)(0.25 * stream_bytes / partial_bytes_per_wg),
                                                 std::min<long>((long)(0.6 * stream_bytes / partial_bytes_per_wg), fitting)));
      // every workgroup reads prefix_len[0..B) first, a wavefront's worth at a time
      wgs = (cand > groups && d.B > 1 && d.B <= 64) ? (int)cand : 0;
      // Chunks are whole fractions of a pair: with fewer than two per pair on average most pairs stay whole beside a few
      // halved ones. Twice as many then, in two rounds, on the kernels that run two workgroups per compute unit (9 requests
      // x 40 heads of 4100 keys, trees of 20: 149 -> 142 us), as long as the partials still fit the library's own scratch
      // array; the few-query kernel takes contiguous shares instead (see contiguous_deal).
      const long twice = std::min<long>(2 * resident, (long)(0.25 * stream_bytes / partial_bytes_per_wg));
      const double slots = (double)((twice + virtual_heads - 1) / virtual_heads + 1);
      if (p.wide && wgs > 0 && wgs < 2 * groups && twice > wgs &&
          (double)d.B * d.H * slots * d.N * (d.D + 2) * 4.0 + 512.0 <= (double)SPEC_STATIC_SCRATCH_BYTES)
        wgs = (int)twice;
    }
    if (wgs > 0) {
      p.balanced_wgs = wgs;
      p.contiguous = !p.wide && wgs < 2 * groups;
      p.chunk_keys = 0;
      p.n_splits = (wgs + virtual_heads - 1) / virtual_heads + 1;   // a pair has at most this many chunks
    }
  }
  if (chunk <= 0 && d.dtype == SPEC_F32) {
    // float32: two workgroups fit a compute unit, and the matrix unit is as busy as the memory: the key range is cut
    // until there are two workgroups per compute unit, in chunks of at least 128 keys (two tiles per wavefront), where
    // that saves more than the merge launch costs (from 256 keys on; never with a workgroup per compute unit already).
    // Measured, us at the chosen cut / uncut: 4 requests x 32 heads, 300-1000 keys, trees of 24: 38 / 53; 1 x 32, 400
    // keys, 16: 14 / 19.5; 1 x 32, 800 keys: 15 / 29; 8 x 32, 512 keys: cut in two 40.9, uncut (the choice) 37.4. The
    // partials of 512 workgroups of 32 queries are 9 MB at most.
    const long want = 2L * compute_units() / std::max<long>(1, groups);
    const long splits =
        (max_len < 256 || groups >= compute_units()) ? 1 : std::max<long>(1, std::min<long>(want, max_len / 128));
    chunk = (int)((max_len + splits - 1) / splits);
    chunk = std::max(128, (int)round_up((size_t)chunk, 64));
  }
  if (p.balanced_wgs == 0) {
    if (chunk <= 0) {
      // One workgroup per (request, head, query group) streams its whole key range when that already
      // gives every compute unit a workgroup: a workgroup's fixed cost (first loads, tree set-up, final
      // merge, and the extra combine launch) outweighs any gain from more parallel slack. With fewer pairs
      // the key range is cut into as many equal chunks as fill the device once, of at least 256 keys
      // (measured on one to four requests of 32 heads, 1024 to 16384 keys: 13 us instead of 22 for one
      // request of 1024 keys, 50 instead of 57 for 16384).
      const long max_splits = std::max<long>(1, max_len / 256);
      // The wide kernels hold two workgroups per compute unit, but where one per compute unit nearly fills the device (four
      // fifths) a cut for that many is the better one: half the partials, or none and no merge, and no two workgroups that
      // compete for a compute unit. Measured, us, two per compute unit / one: 32/8 heads of 7000 keys, trees of 33, 31.4 / 25.5;
      // 32/8 of 16000, 10, 30.3 / 25.8; 2 x 32 of 1500, 60, 27.6 / 24.3; 4 x 32/8 of 3000, 32, 32.7 / 27.5; uncut 8 x 32 heads of 600, 100, 43.0 / 31.4; 6 x 40 of 1000, 100, 48.4 / 41.0; 4 x 64 of 600, 30, 26.1
      // / 20.7; 7 x 32 of 2000, 60, 55.9 / 52.2. Uncut, a lone workgroup's two tiles in flight and the idle fifth tell in the end
      // (28 x 64/8 heads of 3000, 16, 83.1 / 85.8; D = 64: 20 x 12 of 3000, 30, 38.8 / 42.4, but 8 x 32 of 700, 50, 22.7 / 17.6):
      // only up to 20 D keys. Cut, several requests of unequal lengths lose more to the longer chunks than that saves: chunks of
      // up to 8 D keys, or 20 D of one request (16 x 64/8 of 8000 in two, 111 / 125, of 4000-8000 98 / 115; 4 x 32/8 of 12000 in
      // eight, 46.4 / 45.0, of 6000-12000 41.3 / 43.9), the 32-query kernel up to 6 D (2 x 32 of 1688-3374, 101, 35.7 / 37.8; 2 x 64 of 751-1500,
      // 90, 35.0 / 37.1; but 4 x 32/8 of 6000, 32, 38.8 / 35.2, 2 x 12 of 2001-4000, 100, 29.1 / 27.5). Pairs of many query groups are bound by arithmetic and want both (64/8
      // heads of 4000 keys, trees of 128, 42 / 47). Pairs of up to two query tiles: with D = 128 one per unit (32 heads
      // of 3152 keys, trees of 20, 20.7 / 18.7; 64 of 999, 29, 19.1 / 16.4; 40 of 9728, 28, 42.0 / 38.6; 4 x 12 of 1044-2086, 29, 19.7 / 17.9;
      // 2 x 64 of 556-1111, 17, 20.5 / 19.4), with D = 64 two (64 heads of 3225 keys, 20, 17.6 / 18.3; 40 of 4407, 20, 16.9 / 17.7; 2 x 64
      // of 784, 23, 13.0 / 13.1; 40 of 2092, 17, 12.6 / 11.9).
      const long per_unit = compute_units() / std::max<long>(1, groups);
      // Longest chunk for that, in halves of D. Paged, the wide kernel's tiles wait for their blocks' numbers first, which a second
      // workgroup hides: shorter chunks only (us, two / one: cut, 4 x 32 heads of 600-1200 keys, trees of 50, 29.2 / 31.3; 64 of 3000, 40,
      // 33.2 / 34.8; 32 of 12000, 24, 42.2 / 44.9; but 32 of 3100, 20, 22.4 / 19.8, 4 x 12 of 1044-2086, 29, 21.2 / 19.7; uncut 8 x 32
      // of 1200-2400, 60, 69.0 / 71.9, of 750-1500 52.3 / 50.2).
      const int half_d = p.m32 ? (per_unit == 1 ? 40 : d.B > 1 ? 12 : paged ? 24 : 40)
                               : paged ? (per_unit == 1 ? 28 : 7) : (per_unit == 1 || d.B == 1) ? 40 : 16;
      const bool one_per_unit = p.wide && (per_unit == 1 || tiles > 2 || d.D == 128) && qg.n_qgroups <= 2 && per_unit <= max_splits &&
                                groups * per_unit * 5 >= 4 * compute_units() &&
                                max_len / per_unit <= half_d * d.D / 2;
      const long hold = one_per_unit ? compute_units() : resident;
      long splits = std::max<long>(1, hold / std::max<long>(1, groups));
      if (splits > max_splits) splits = max_splits;
      // Three query tiles and more per workgroup (grouped heads, wide trees) make a tile of keys dearer: where few pairs leave
      // most of the device idle the cuts go down to 128 keys, up to eight of them and half a workgroup per compute unit
      // (beyond that the partials cost what it saves). Measured, us, by 256 and by 128 keys: 12 heads of 400 keys, trees of 100,
      // 24.3 / 18.4; 2 x 32/8 heads, 700 keys, 16.9 / 12.6; 4 x 64/8, 500 keys, 20.7 / 17.7; 32 heads of 400 keys, trees of 40,
      // 18.0 / 14.1. Two cuts alone only pay where there are few pairs and a head dimension of 128 (32/8 heads, 250 keys, 14.2 /
      // 12.0; but 64 heads of 300 keys, trees of 50, 15.1 / 16.1, and 3 x 12 heads of 260 keys, D = 64, 10.4 / 11.5); two query
      // tiles do not gain (40 heads of 300 keys, trees of 24, 13.3 / 14.7).
      if (p.wide && tiles > 2 && splits <= 4) {   // (2 x 24/6 heads, 2032 keys, in seven or in eight: 12.0 / 12.7)
        const long room = compute_units() / 2 / std::max<long>(1, groups);
        const long finer = std::min<long>({room, (long)max_len / 128, 8});
        if (finer > 2 || (finer == 2 && room > 2 && d.D == 128)) splits = std::max(splits, finer);
      }
      chunk = (int)((max_len + splits - 1) / splits);
      if (chunk < 128) chunk = 128;
      // Where there is room for one chunk more per pair, the prefix alone is cut, at multiples of the kernel's tile: the tree
      // then has a short chunk of its own instead of standing behind a full one, and no chunk starts inside a tile (one
      // request, 32 heads, us: 1024 keys, trees of 40: 18.5 -> 15.2; trees of 24: 14.7 -> 13.6; 512 keys,
      // trees of 16: 14.5 -> 12.1). Not for the 32-query kernel, whose partials cost what that saves (21.6 -> 23.5).
      // The few-query kernel's tile has 32 keys. Its chunks are rounded up to 64 all the same where the last one, which the
      // tree's own tile makes about 64 keys longer, would otherwise be the longest: 12 heads of 1589 keys, trees of 3, in
      // chunks of 288 (the last of 152) 24.0, of 320 (the last of 312) 26.4; 40 heads of 1704 keys in chunks of 288 (the last of
      // 265) 22.1, of 320 (the last of 105) 21.2; two layers each.
      if (splits > 1 && !p.m32) {
        const int per = (max_prefix + (int)splits - 1) / (int)splits;
        auto rounded = [&](int to) { return std::max(128, (int)round_up((size_t)per, (size_t)to)); };
        auto fits = [&](int c) { return groups * ((max_len + c - 1) / c) <= hold; };
        auto longest = [&](int c) { return std::max(c, max_len - (max_len - 1) / c * c + 64); };
        if (!p.wide) {
          chunk = fits(rounded(tile)) ? rounded(tile) : (int)round_up((size_t)chunk, tile);
          if (fits(rounded(64)) && longest(rounded(64)) < longest(chunk)) chunk = rounded(64);
        } else if (fits(rounded(tile))) {
          // (in tiles: the longest chunk, or the last with the tree's masked tiles behind it. With workgroups to spare only that
          // counts: 2 requests x 8 K/V heads of 2191 keys, trees of 5, in chunks of 288, the last of 180: 15.2 us, of 320, the
          // last of 276: 15.7. With a workgroup per compute unit and more, fewer chunks do less in all: 32 heads of 4432 keys,
          // trees of 20, two layers: 49.3 / 45.3.)
          auto steps = [&](int c) { return std::max((c + 63) / 64, (max_len - (max_len - 1) / c * c + 63) / 64 + 1); };
          const int equal = (int)round_up((size_t)chunk, paged ? 64 : 32);
          if (groups * ((max_len + equal - 1) / equal) > resident / 2 || steps(rounded(tile)) <= steps(equal)) chunk = rounded(tile);
        }
      }
    }
    // chunks start at tile boundaries (with paged caches a tile must not straddle two blocks)
    chunk = (int)round_up((size_t)chunk, (paged && p.wide) ? SPEC_WIDE_TILE_KEYS : 32);
    p.chunk_keys = chunk;
    p.n_splits = (max_len + chunk - 1) / chunk;
  }
  if (p.wide && p.n_splits <= 1 && p.balanced_wgs == 0 && qg.n_qgroups == 1 && tiles > 4 && !p.m32) {
    // Eight-wavefront workgroups (one per compute unit) and more (request, head) pairs than compute units: a
    // workgroup then serves several heads of a request in a row, which costs one prologue and one tree set-up
    // instead of one per head (measured: 3 % on 512 pairs of 640 keys; no gain for the four-wavefront shape,
    // where two workgroups per compute unit already overlap each other's prologues). Chosen to minimise
    // (rounds of workgroups) x (heads in a row + the fixed cost of a workgroup, about a third of a head).
    int best = 1;
    double best_cost = 1e30;
    for (int nh = 1; nh <= 8 && nh <= d.H_kv; ++nh) {
      const long wgs = (long)d.B * ((d.H_kv + nh - 1) / nh);
      const double cost = (double)((wgs + resident - 1) / resident) * (nh + 0.35);
      if (cost < best_cost - 1e-9) { best_cost = cost; best = nh; }
    }
    p.heads_per_wg = d.plan_heads_per_wg > 0 ? d.plan_heads_per_wg : best;
    if (p.heads_per_wg < 1) p.heads_per_wg = 1;
    if (p.heads_per_wg > d.H_kv) p.heads_per_wg = d.H_kv;
  }
  if (p.n_splits <= 1 && p.balanced_wgs == 0) {
    p.n_splits = 1;
    p.ws_o_off = p.ws_ml_off = 0;
    p.ws_bytes = 0;
  } else {
    const size_t rows = (size_t)d.B * d.H * p.n_splits * d.N;
    p.ws_o_off = 0;
    p.ws_ml_off = round_up(rows * d.D * sizeof(float), 256);
    p.ws_bytes = p.ws_ml_off + round_up(rows * 2 * sizeof(float), 256);
  }
  return p;
}

}  // namespace spec

using namespace spec;

extern "C" {

int spec_version(void) { return 100; }

const char* spec_strerror(int code) {
  switch (code) {
    case SPEC_OK: return "ok";
    case SPEC_ERR_INVALID_ARG: return "invalid argument (null pointer, non-positive size, bad stride or alignment)";
    case SPEC_ERR_UNSUPPORTED: return "unsupported shape or dtype";
    case SPEC_ERR_CAPACITY: return "tree does not fit the cache capacity";
    case SPEC_ERR_HIP: return "HIP runtime error";
    case SPEC_ERR_WORKSPACE: return "workspace missing or too small";
    default: return "unknown error code";
  }
}

// Every cache-touching entry point exists in a contiguous and a paged form; `pages` is NULL in the first.
static int kv_append_impl(const spec_attn_desc_t* desc, const spec_kv_pages_t* pages, bool paged, const void* k_new,
                          const void* v_new, void* k_cache, void* v_cache, const int32_t* prefix_len, int32_t* status,
                          void* hip_stream) {
  int rc = check_desc(desc);
  if (rc != SPEC_OK) return rc;
  Pages pg = no_pages();
  if (paged && (rc = check_pages(desc, pages, &pg)) != SPEC_OK) return rc;
  if (!k_new || !v_new || !k_cache || !v_cache || !prefix_len) return SPEC_ERR_INVALID_ARG;
  if (!aligned16(k_new) || !aligned16(v_new) || !aligned16(k_cache) || !aligned16(v_cache)) return SPEC_ERR_INVALID_ARG;
  if (new_strides_missing(desc)) return SPEC_ERR_INVALID_ARG;
  return launch_kv_append(*desc, pg, k_new, v_new, k_cache, v_cache, prefix_len, status, (hipStream_t)hip_stream) ==
                 hipSuccess
             ? SPEC_OK
             : SPEC_ERR_HIP;
}

int spec_kv_append(const spec_attn_desc_t* desc, const void* k_new, const void* v_new, void* k_cache, void* v_cache,
                   const int32_t* prefix_len, int32_t* status, void* hip_stream) {
  return kv_append_impl(desc, nullptr, false, k_new, v_new, k_cache, v_cache, prefix_len, status, hip_stream);
}

int spec_kv_append_paged(const spec_attn_desc_t* desc, const spec_kv_pages_t* pages, const void* k_new, const void* v_new,
                         void* k_cache, void* v_cache, const int32_t* prefix_len, int32_t* status, void* hip_stream) {
  return kv_append_impl(desc, pages, true, k_new, v_new, k_cache, v_cache, prefix_len, status, hip_stream);
}

static int kv_append_rope_impl(const spec_attn_desc_t* desc, const spec_kv_pages_t* pages, bool paged, const void* k_new,
                               const void* v_new, void* k_cache, void* v_cache, const int32_t* tree_depth,
                               const int32_t* prefix_len, const float* rope_cos, const float* rope_sin, int32_t rope_len,
                               int32_t* status, void* hip_stream, void* q = nullptr, bool with_q = false) {
  if (with_q && (q == nullptr || !aligned16(q))) return check_desc(desc) != SPEC_OK ? check_desc(desc) : SPEC_ERR_INVALID_ARG;
  int rc = check_desc(desc);
  if (rc != SPEC_OK) return rc;
  Pages pg = no_pages();
  if (paged && (rc = check_pages(desc, pages, &pg)) != SPEC_OK) return rc;
  if (!k_new || !v_new || !k_cache || !v_cache || !prefix_len || !tree_depth || !rope_cos || !rope_sin) return SPEC_ERR_INVALID_ARG;
  if (rope_len <= 0 || new_strides_missing(desc)) return SPEC_ERR_INVALID_ARG;
  if (!aligned16(k_new) || !aligned16(v_new) || !aligned16(k_cache) || !aligned16(v_cache)) return SPEC_ERR_INVALID_ARG;
  return launch_kv_append_rope(*desc, pg, k_new, v_new, k_cache, v_cache, tree_depth, prefix_len, rope_cos, rope_sin,
                               rope_len, status, (hipStream_t)hip_stream, q) == hipSuccess
             ? SPEC_OK
             : SPEC_ERR_HIP;
}

int spec_qk_rope_append(const spec_attn_desc_t* desc, void* q, const void* k_new, const void* v_new, void* k_cache,
                        void* v_cache, const int32_t* tree_depth, const int32_t* prefix_len, const float* rope_cos,
                        const float* rope_sin, int32_t rope_len, int32_t* status, void* hip_stream) {
  return kv_append_rope_impl(desc, nullptr, false, k_new, v_new, k_cache, v_cache, tree_depth, prefix_len, rope_cos,
                             rope_sin, rope_len, status, hip_stream, q, true);
}

int spec_qk_rope_append_paged(const spec_attn_desc_t* desc, const spec_kv_pages_t* pages, void* q, const void* k_new,
                              const void* v_new, void* k_cache, void* v_cache, const int32_t* tree_depth,
                              const int32_t* prefix_len, const float* rope_cos, const float* rope_sin, int32_t rope_len,
                              int32_t* status, void* hip_stream) {
  return kv_append_rope_impl(desc, pages, true, k_new, v_new, k_cache, v_cache, tree_depth, prefix_len, rope_cos, rope_sin,
                             rope_len, status, hip_stream, q, true);
}

int spec_kv_append_rope(const spec_attn_desc_t* desc, const void* k_new, const void* v_new, void* k_cache, void* v_cache,
                        const int32_t* tree_depth, const int32_t* prefix_len, const float* rope_cos, const float* rope_sin,
                        int32_t rope_len, int32_t* status, void* hip_stream) {
  return kv_append_rope_impl(desc, nullptr, false, k_new, v_new, k_cache, v_cache, tree_depth, prefix_len, rope_cos,
                             rope_sin, rope_len, status, hip_stream);
}

int spec_kv_append_rope_paged(const spec_attn_desc_t* desc, const spec_kv_pages_t* pages, const void* k_new,
                              const void* v_new, void* k_cache, void* v_cache, const int32_t* tree_depth,
                              const int32_t* prefix_len, const float* rope_cos, const float* rope_sin, int32_t rope_len,
                              int32_t* status, void* hip_stream) {
  return kv_append_rope_impl(desc, pages, true, k_new, v_new, k_cache, v_cache, tree_depth, prefix_len, rope_cos, rope_sin,
                             rope_len, status, hip_stream);
}

size_t spec_tree_attention_workspace_bytes(const spec_attn_desc_t* desc) {
  if (check_desc(desc) != SPEC_OK) return 0;
  return make_attn_plan(*desc).ws_bytes;
}

size_t spec_tree_attention_paged_workspace_bytes(const spec_attn_desc_t* desc, const spec_kv_pages_t* pages) {
  Pages pg;
  if (check_desc(desc) != SPEC_OK || check_pages(desc, pages, &pg) != SPEC_OK) return 0;
  return make_attn_plan(*desc, true).ws_bytes;
}

// Shared body of spec_tree_attention (k_new == NULL) and spec_tree_attention_append.
static int tree_attention_impl(const spec_attn_desc_t* desc, const spec_kv_pages_t* pages, bool paged, const void* q,
                               const void* k_new, const void* v_new, void* k_cache, void* v_cache,
                               const int32_t* tree_parent, const int32_t* tree_depth, const int32_t* prefix_len, void* out,
                               void* workspace, size_t workspace_bytes, int32_t* status, void* hip_stream,
                               const Rope& rope = no_rope()) {
  int rc = check_desc(desc);
  if (rc != SPEC_OK) return rc;
  Pages pg = no_pages();
  if (paged && (rc = check_pages(desc, pages, &pg)) != SPEC_OK) return rc;
  if (!q || !k_cache || !v_cache || !tree_parent || !tree_depth || !prefix_len || !out) return SPEC_ERR_INVALID_ARG;
  if (!aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(out)) return SPEC_ERR_INVALID_ARG;
  const bool append = k_new != nullptr || v_new != nullptr;
  if (append && (!k_new || !v_new || !aligned16(k_new) || !aligned16(v_new) || new_strides_missing(desc)))
    return SPEC_ERR_INVALID_ARG;
  const AttnPlan plan = make_attn_plan(*desc, paged);
  if (plan.ws_bytes > 0) {
    if (workspace == nullptr || workspace_bytes < plan.ws_bytes) return SPEC_ERR_WORKSPACE;
    if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return SPEC_ERR_INVALID_ARG;
  }
  // The launch plan covers keys up to max_prefix_len + N. A request whose prefix_len exceeds the stated
  // maximum must not be attended over a truncated key range: the kernels treat the stated maximum as the
  // capacity, so such a request is flagged SPEC_ST_CAPACITY like one that does not fit the cache.
  spec_attn_desc_t d = *desc;
  if (d.max_prefix_len > 0) d.S_cap = d.max_prefix_len + d.N;   // <= S_cap (checked above); strides are unchanged
  // Rotary tables: they must cover every position of a tree of N nodes, so their length bounds the capacity too.
  if (rope.cos != nullptr && rope.len < d.S_cap) d.S_cap = rope.len;
  hipStream_t s = (hipStream_t)hip_stream;
  hipError_t e;
  if (d.dtype == SPEC_BF16) {
    e = launch_tree_attention_bf16(d, plan, pg, q, k_cache, v_cache, k_new, v_new, tree_parent, tree_depth, prefix_len, out,
                                   workspace, status, s, rope);
  } else {
    e = launch_tree_attention_f32(d, plan, pg, (const float*)q, (float*)k_cache, (float*)v_cache, (const float*)k_new,
                                  (const float*)v_new, tree_parent, tree_depth, prefix_len, (float*)out, workspace, status, s);
  }
  if (e != hipSuccess) return SPEC_ERR_HIP;
  if (plan.n_splits > 1 || plan.balanced_wgs > 0) {
    e = launch_attn_combine(d, plan, prefix_len, workspace, out, status, s);
    if (e != hipSuccess) return SPEC_ERR_HIP;
  }
  return SPEC_OK;
}

int spec_tree_attention(const spec_attn_desc_t* desc, const void* q, const void* k_cache, const void* v_cache,
                        const int32_t* tree_parent, const int32_t* tree_depth, const int32_t* prefix_len, void* out,
                        void* workspace, size_t workspace_bytes, int32_t* status, void* hip_stream) {
  return tree_attention_impl(desc, nullptr, false, q, nullptr, nullptr, const_cast<void*>(k_cache),
                             const_cast<void*>(v_cache), tree_parent, tree_depth, prefix_len, out, workspace,
                             workspace_bytes, status, hip_stream);
}

int spec_tree_attention_paged(const spec_attn_desc_t* desc, const spec_kv_pages_t* pages, const void* q,
                              const void* k_cache, const void* v_cache, const int32_t* tree_parent,
                              const int32_t* tree_depth, const int32_t* prefix_len, void* out, void* workspace,
                              size_t workspace_bytes, int32_t* status, void* hip_stream) {
  return tree_attention_impl(desc, pages, true, q, nullptr, nullptr, const_cast<void*>(k_cache),
                             const_cast<void*>(v_cache), tree_parent, tree_depth, prefix_len, out, workspace,
                             workspace_bytes, status, hip_stream);
}

int spec_tree_attention_append(const spec_attn_desc_t* desc, const void* q, const void* k_new, const void* v_new,
                               void* k_cache, void* v_cache, const int32_t* tree_parent, const int32_t* tree_depth,
                               const int32_t* prefix_len, void* out, void* workspace, size_t workspace_bytes,
                               int32_t* status, void* hip_stream) {
  if (!k_new || !v_new) return check_desc(desc) != SPEC_OK ? check_desc(desc) : SPEC_ERR_INVALID_ARG;
  return tree_attention_impl(desc, nullptr, false, q, k_new, v_new, k_cache, v_cache, tree_parent, tree_depth,
                             prefix_len, out, workspace, workspace_bytes, status, hip_stream);
}

static int rope_args(const spec_attn_desc_t* desc, const void* k_new, const void* v_new, const float* rope_cos,
                     const float* rope_sin, int32_t rope_len) {
  const int rc = check_desc(desc);
  if (rc != SPEC_OK) return rc;
  if (!k_new || !v_new || !rope_cos || !rope_sin || rope_len <= 0) return SPEC_ERR_INVALID_ARG;
  if (desc->dtype != SPEC_BF16) return SPEC_ERR_UNSUPPORTED;
  return SPEC_OK;
}

int spec_tree_attention_append_rope(const spec_attn_desc_t* desc, const void* q, const void* k_new, const void* v_new,
                                    void* k_cache, void* v_cache, const int32_t* tree_parent, const int32_t* tree_depth,
                                    const int32_t* prefix_len, const float* rope_cos, const float* rope_sin,
                                    int32_t rope_len, void* out, void* workspace, size_t workspace_bytes,
                                    int32_t* status, void* hip_stream) {
  const int rc = rope_args(desc, k_new, v_new, rope_cos, rope_sin, rope_len);
  if (rc != SPEC_OK) return rc;
  return tree_attention_impl(desc, nullptr, false, q, k_new, v_new, k_cache, v_cache, tree_parent, tree_depth,
                             prefix_len, out, workspace, workspace_bytes, status, hip_stream,
                             Rope{rope_cos, rope_sin, rope_len});
}

int spec_tree_attention_append_rope_paged(const spec_attn_desc_t* desc, const spec_kv_pages_t* pages, const void* q,
                                          const void* k_new, const void* v_new, void* k_cache, void* v_cache,
                                          const int32_t* tree_parent, const int32_t* tree_depth,
                                          const int32_t* prefix_len, const float* rope_cos, const float* rope_sin,
                                          int32_t rope_len, void* out, void* workspace, size_t workspace_bytes,
                                          int32_t* status, void* hip_stream) {
  const int rc = rope_args(desc, k_new, v_new, rope_cos, rope_sin, rope_len);
  if (rc != SPEC_OK) return rc;
  return tree_attention_impl(desc, pages, true, q, k_new, v_new, k_cache, v_cache, tree_parent, tree_depth, prefix_len,
                             out, workspace, workspace_bytes, status, hip_stream, Rope{rope_cos, rope_sin, rope_len});
}

int spec_tree_attention_append_static(const spec_attn_desc_t* desc, const void* q, const void* k_new, const void* v_new,
                                      void* k_cache, void* v_cache, const int32_t* tree_parent,
                                      const int32_t* tree_depth, const int32_t* prefix_len, void* out, int32_t* status,
                                      void* hip_stream) {
  const int rc = check_desc(desc);
  if (rc != SPEC_OK) return rc;
  if (!k_new || !v_new) return SPEC_ERR_INVALID_ARG;
  // the plan of the contiguous call decides how much scratch the launch needs
  const size_t need = make_attn_plan(*desc).ws_bytes;
  if (need > (size_t)SPEC_STATIC_SCRATCH_BYTES) return SPEC_ERR_WORKSPACE;
  void* ws = nullptr;
  if (need > 0) {
    const int src = static_scratch(&ws);
    if (src != SPEC_OK) return src;
  }
  return tree_attention_impl(desc, nullptr, false, q, k_new, v_new, k_cache, v_cache, tree_parent, tree_depth,
                             prefix_len, out, ws, need, status, hip_stream);
}

int spec_tree_attention_append_paged(const spec_attn_desc_t* desc, const spec_kv_pages_t* pages, const void* q,
                                     const void* k_new, const void* v_new, void* k_cache, void* v_cache,
                                     const int32_t* tree_parent, const int32_t* tree_depth, const int32_t* prefix_len,
                                     void* out, void* workspace, size_t workspace_bytes, int32_t* status,
                                     void* hip_stream) {
  if (!k_new || !v_new) return check_desc(desc) != SPEC_OK ? check_desc(desc) : SPEC_ERR_INVALID_ARG;
  return tree_attention_impl(desc, pages, true, q, k_new, v_new, k_cache, v_cache, tree_parent, tree_depth, prefix_len,
                             out, workspace, workspace_bytes, status, hip_stream);
}

static int check_verify_common(int32_t B, int32_t N, int32_t V, int32_t logits_dtype, const void* logits,
                               const int32_t* tree_token, const int32_t* tree_parent, int32_t Lmax,
                               const int32_t* accepted_path, const int32_t* accepted_len, const int32_t* out_tokens) {
  if (B <= 0 || N <= 0 || V <= 0 || Lmax <= 0) return SPEC_ERR_INVALID_ARG;
  if (N > SPEC_MAX_TREE_NODES) return SPEC_ERR_UNSUPPORTED;
  if (logits_dtype != SPEC_F32 && logits_dtype != SPEC_BF16) return SPEC_ERR_UNSUPPORTED;
  if (!logits || !tree_token || !tree_parent || !accepted_path || !accepted_len || !out_tokens) return SPEC_ERR_INVALID_ARG;
  if (!aligned16(logits)) return SPEC_ERR_INVALID_ARG;
  return SPEC_OK;
}

int spec_tree_expand_topk(int32_t B, int32_t F, int32_t V, int32_t logits_dtype, const void* ssm_logits, int32_t k,
                          const int32_t* child_slot, int32_t N, int32_t* tree_token, int32_t* status, void* hip_stream) {
  if (B <= 0 || F <= 0 || V <= 0 || N <= 0 || k <= 0) return SPEC_ERR_INVALID_ARG;
  if (k > V || k > SPEC_MAX_TOPK || N > SPEC_MAX_TREE_NODES) return SPEC_ERR_UNSUPPORTED;
  if (logits_dtype != SPEC_F32 && logits_dtype != SPEC_BF16) return SPEC_ERR_UNSUPPORTED;
  if (!ssm_logits || !child_slot || !tree_token) return SPEC_ERR_INVALID_ARG;
  return launch_expand_topk(B, F, V, logits_dtype, ssm_logits, k, child_slot, N, tree_token, status,
                            (hipStream_t)hip_stream) == hipSuccess
             ? SPEC_OK
             : SPEC_ERR_HIP;
}

int spec_tree_merge(int32_t B, int32_t M, int32_t Nin, const int32_t* in_parent, const int32_t* in_token,
                    const int32_t* in_size, int32_t Nout, int32_t* out_parent, int32_t* out_depth, int32_t* out_token,
                    int32_t* out_ssm, int32_t* out_size, int32_t* node_map, int32_t* status, void* hip_stream) {
  if (B <= 0 || M <= 0 || Nin <= 0 || Nout <= 0) return SPEC_ERR_INVALID_ARG;
  if ((long)M * Nin > SPEC_MAX_MERGE_INPUT_NODES || Nout > SPEC_MAX_TREE_NODES) return SPEC_ERR_UNSUPPORTED;
  if (!in_parent || !in_token || !in_size || !out_parent || !out_depth || !out_token || !out_ssm || !out_size)
    return SPEC_ERR_INVALID_ARG;
  return launch_tree_merge(B, M, Nin, in_parent, in_token, in_size, Nout, out_parent, out_depth, out_token, out_ssm,
                           out_size, node_map, status, (hipStream_t)hip_stream) == hipSuccess
             ? SPEC_OK
             : SPEC_ERR_HIP;
}

int spec_verify_greedy(int32_t B, int32_t N, int32_t V, int32_t logits_dtype, const void* logits_llm,
                       const int32_t* tree_token, const int32_t* tree_parent, int32_t Lmax, int32_t* accepted_path,
                       int32_t* accepted_len, int32_t* out_tokens, int32_t* node_argmax, void* workspace,
                       size_t workspace_bytes, int32_t* status, void* hip_stream) {
  const int rc = check_verify_common(B, N, V, logits_dtype, logits_llm, tree_token, tree_parent, Lmax, accepted_path,
                                     accepted_len, out_tokens);
  if (rc != SPEC_OK) return rc;
  if (node_argmax == nullptr) {
    if (workspace == nullptr || workspace_bytes < (size_t)B * N * sizeof(int32_t)) return SPEC_ERR_WORKSPACE;
    node_argmax = (int32_t*)workspace;
  }
  hipStream_t s = (hipStream_t)hip_stream;
  if (launch_node_stats(B, N, V, logits_dtype, logits_llm, 1.0f, node_argmax, nullptr, nullptr, s) != hipSuccess)
    return SPEC_ERR_HIP;
  if (launch_greedy_walk(B, N, node_argmax, tree_token, tree_parent, Lmax, accepted_path, accepted_len, out_tokens,
                         status, s) != hipSuccess)
    return SPEC_ERR_HIP;
  return SPEC_OK;
}

size_t spec_lm_head_argmax_workspace_bytes(int32_t M, int32_t V) {
  if (M <= 0 || V <= 0) return 0;
  // the partials, then room for node_argmax when the caller of spec_verify_greedy_lm_head does not want it
  return lm_head_partials_bytes(M, V) + round_up((size_t)M * sizeof(int32_t), 256);
}

static int check_lm_head(int32_t M, int32_t K, int32_t V, const void* hidden, const void* weight, const void* workspace,
                         size_t workspace_bytes) {
  if (M <= 0 || K <= 0 || V <= 0) return SPEC_ERR_INVALID_ARG;
  if (K % 256 != 0) return SPEC_ERR_UNSUPPORTED;
  if (!hidden || !weight || !aligned16(hidden) || !aligned16(weight)) return SPEC_ERR_INVALID_ARG;
  if (workspace == nullptr || workspace_bytes < spec_lm_head_argmax_workspace_bytes(M, V)) return SPEC_ERR_WORKSPACE;
  if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return SPEC_ERR_INVALID_ARG;
  return SPEC_OK;
}

int spec_lm_head_argmax(int32_t M, int32_t K, int32_t V, const void* hidden, const void* weight, int32_t* node_argmax,
                        float* node_max, void* workspace, size_t workspace_bytes, void* hip_stream) {
  const int rc = check_lm_head(M, K, V, hidden, weight, workspace, workspace_bytes);
  if (rc != SPEC_OK) return rc;
  if (!node_argmax) return SPEC_ERR_INVALID_ARG;
  return launch_lm_head_argmax(M, K, V, hidden, weight, node_argmax, node_max, workspace, (hipStream_t)hip_stream) ==
                 hipSuccess
             ? SPEC_OK
             : SPEC_ERR_HIP;
}

int spec_verify_greedy_lm_head(int32_t B, int32_t N, int32_t K, int32_t V, const void* hidden, const void* weight,
                               const int32_t* tree_token, const int32_t* tree_parent, int32_t Lmax,
                               int32_t* accepted_path, int32_t* accepted_len, int32_t* out_tokens, int32_t* node_argmax,
                               void* workspace, size_t workspace_bytes, int32_t* status, void* hip_stream) {
  if (B <= 0 || N <= 0 || Lmax <= 0) return SPEC_ERR_INVALID_ARG;
  if (N > SPEC_MAX_TREE_NODES) return SPEC_ERR_UNSUPPORTED;
  if ((long)B * N > 0x7fffffffL) return SPEC_ERR_UNSUPPORTED;
  const int M = B * N;
  const int rc = check_lm_head(M, K, V, hidden, weight, workspace, workspace_bytes);
  if (rc != SPEC_OK) return rc;
  if (!tree_token || !tree_parent || !accepted_path || !accepted_len || !out_tokens) return SPEC_ERR_INVALID_ARG;
  if (node_argmax == nullptr) node_argmax = (int32_t*)((char*)workspace + lm_head_partials_bytes(M, V));
  hipStream_t s = (hipStream_t)hip_stream;
  if (launch_lm_head_argmax(M, K, V, hidden, weight, node_argmax, nullptr, workspace, s) != hipSuccess) return SPEC_ERR_HIP;
  if (launch_greedy_walk(B, N, node_argmax, tree_token, tree_parent, Lmax, accepted_path, accepted_len, out_tokens,
                         status, s) != hipSuccess)
    return SPEC_ERR_HIP;
  return SPEC_OK;
}

size_t spec_verify_naive_workspace_bytes(int32_t B, int32_t N, int32_t V) {
  if (B <= 0 || N <= 0 || V <= 0) return 0;
  // node max, then the sampled tokens when the caller does not want them
  return round_up((size_t)B * N * sizeof(float), 256) + round_up((size_t)B * N * sizeof(int32_t), 256);
}

int spec_verify_naive(int32_t B, int32_t N, int32_t V, int32_t logits_dtype, const void* logits_llm,
                      const int32_t* tree_token, const int32_t* tree_parent, const float* u_sample, float temperature,
                      int32_t Lmax, int32_t* accepted_path, int32_t* accepted_len, int32_t* out_tokens,
                      int32_t* node_sample, void* workspace, size_t workspace_bytes, int32_t* status,
                      void* hip_stream) {
  const int rc = check_verify_common(B, N, V, logits_dtype, logits_llm, tree_token, tree_parent, Lmax, accepted_path,
                                     accepted_len, out_tokens);
  if (rc != SPEC_OK) return rc;
  if (!u_sample) return SPEC_ERR_INVALID_ARG;
  if (!(temperature > 0.f) || std::isinf(temperature)) return SPEC_ERR_INVALID_ARG;
  if (workspace == nullptr || workspace_bytes < spec_verify_naive_workspace_bytes(B, N, V)) return SPEC_ERR_WORKSPACE;
  if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return SPEC_ERR_INVALID_ARG;
  float* node_max = (float*)workspace;
  if (node_sample == nullptr) node_sample = (int32_t*)((char*)workspace + round_up((size_t)B * N * sizeof(float), 256));
  hipStream_t s = (hipStream_t)hip_stream;
  const float inv_temp = 1.0f / temperature;
  if (launch_node_stats(B, N, V, logits_dtype, logits_llm, inv_temp, nullptr, node_max, nullptr, s) != hipSuccess)
    return SPEC_ERR_HIP;
  if (launch_node_sample(B, N, V, logits_dtype, logits_llm, inv_temp, node_max, u_sample, node_sample, s) != hipSuccess)
    return SPEC_ERR_HIP;
  if (launch_greedy_walk(B, N, node_sample, tree_token, tree_parent, Lmax, accepted_path, accepted_len, out_tokens,
                         status, s) != hipSuccess)
    return SPEC_ERR_HIP;
  return SPEC_OK;
}

size_t spec_verify_stochastic_workspace_bytes(int32_t B, int32_t N, int32_t V) {
  if (B <= 0 || N <= 0 || V <= 0) return 0;
  // node max + node sum-exp, then two residual buffers of V floats per request
  return round_up((size_t)B * N * 2 * sizeof(float), 256) + round_up((size_t)2 * B * V * sizeof(float), 256);
}

int spec_verify_stochastic(int32_t B, int32_t N, int32_t V, int32_t logits_dtype, const void* logits_llm,
                           const float* probs_ssm, int32_t R, const int32_t* ssm_row, const int32_t* tree_token,
                           const int32_t* tree_parent, const float* u_accept, const float* u_order,
                           const float* u_final, float temperature, int32_t Lmax, int32_t* accepted_path,
                           int32_t* accepted_len, int32_t* out_tokens, void* workspace, size_t workspace_bytes,
                           int32_t* status, void* hip_stream) {
  const int rc = check_verify_common(B, N, V, logits_dtype, logits_llm, tree_token, tree_parent, Lmax, accepted_path,
                                     accepted_len, out_tokens);
  if (rc != SPEC_OK) return rc;
  if (!ssm_row || !u_accept || !u_order || !u_final) return SPEC_ERR_INVALID_ARG;
  if (R < 0 || (R > 0 && probs_ssm == nullptr)) return SPEC_ERR_INVALID_ARG;
  if (!(temperature > 0.f) || std::isinf(temperature)) return SPEC_ERR_INVALID_ARG;
  const size_t need = spec_verify_stochastic_workspace_bytes(B, N, V);
  if (workspace == nullptr || workspace_bytes < need) return SPEC_ERR_WORKSPACE;
  if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return SPEC_ERR_INVALID_ARG;
  float* node_max = (float*)workspace;
  float* node_sumexp = node_max + (size_t)B * N;
  float* resid = (float*)((char*)workspace + round_up((size_t)B * N * 2 * sizeof(float), 256));
  const float inv_temp = 1.0f / temperature;
  hipStream_t s = (hipStream_t)hip_stream;
  const int own_levels = stochastic_own_levels(B, N, V, logits_dtype, Lmax);
  if (own_levels >= std::min(Lmax, N)) {   // no walk visits more nodes, whatever the tree
    node_max = node_sumexp = nullptr;
  } else if (launch_node_stats(B, N, V, logits_dtype, logits_llm, inv_temp, nullptr, node_max, node_sumexp, s,
                               own_levels > 0 ? tree_parent : nullptr, own_levels) != hipSuccess) {
    return SPEC_ERR_HIP;
  }
  if (launch_stochastic_walk(B, N, V, logits_dtype, logits_llm, probs_ssm, R, ssm_row, tree_token, tree_parent, u_accept,
                             u_order, u_final, inv_temp, node_max, node_sumexp, resid, Lmax, accepted_path, accepted_len,
                             out_tokens, status, s, own_levels) != hipSuccess)
    return SPEC_ERR_HIP;
  return SPEC_OK;
}

size_t spec_lm_head_logits_stats_workspace_bytes(int32_t M, int32_t V) {
  if (M <= 0 || V <= 0) return 0;
  return 3 * (lm_head_partials_bytes(M, V) / 2);   // (max, arg-max, sum) per row and vocabulary tile
}

int spec_lm_head_logits_stats(int32_t M, int32_t K, int32_t V, const void* hidden, const void* weight, float temperature,
                              void* logits, int32_t* node_argmax, float* node_max, float* node_sumexp, void* workspace,
                              size_t workspace_bytes, void* hip_stream) {
  if (M <= 0 || K <= 0 || V <= 0) return SPEC_ERR_INVALID_ARG;
  if (K % 256 != 0) return SPEC_ERR_UNSUPPORTED;
  if (!hidden || !weight || !aligned16(hidden) || !aligned16(weight)) return SPEC_ERR_INVALID_ARG;
  if (!logits || !node_max || !node_sumexp || (reinterpret_cast<uintptr_t>(logits) & 7u)) return SPEC_ERR_INVALID_ARG;
  if (!(temperature > 0.f) || std::isinf(temperature)) return SPEC_ERR_INVALID_ARG;
  if (workspace == nullptr || workspace_bytes < spec_lm_head_logits_stats_workspace_bytes(M, V)) return SPEC_ERR_WORKSPACE;
  if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return SPEC_ERR_INVALID_ARG;
  return launch_lm_head(M, K, V, hidden, weight, logits, 1.0f / temperature, node_argmax, node_max, node_sumexp, workspace,
                        (hipStream_t)hip_stream) == hipSuccess
             ? SPEC_OK
             : SPEC_ERR_HIP;
}

size_t spec_verify_stochastic_stats_workspace_bytes(int32_t B, int32_t V) {
  if (B <= 0 || V <= 0) return 0;
  return round_up((size_t)2 * B * V * sizeof(float), 256);   // two residual buffers of V floats per request
}

int spec_verify_stochastic_stats(int32_t B, int32_t N, int32_t V, int32_t logits_dtype, const void* logits_llm,
                                 const float* node_max, const float* node_sumexp, const float* probs_ssm, int32_t R,
                                 const int32_t* ssm_row, const int32_t* tree_token, const int32_t* tree_parent,
                                 const float* u_accept, const float* u_order, const float* u_final, float temperature,
                                 int32_t Lmax, int32_t* accepted_path, int32_t* accepted_len, int32_t* out_tokens,
                                 void* workspace, size_t workspace_bytes, int32_t* status, void* hip_stream) {
  const int rc = check_verify_common(B, N, V, logits_dtype, logits_llm, tree_token, tree_parent, Lmax, accepted_path,
                                     accepted_len, out_tokens);
  if (rc != SPEC_OK) return rc;
  if (!ssm_row || !u_accept || !u_order || !u_final || !node_max || !node_sumexp) return SPEC_ERR_INVALID_ARG;
  if (R < 0 || (R > 0 && probs_ssm == nullptr)) return SPEC_ERR_INVALID_ARG;
  if (!(temperature > 0.f) || std::isinf(temperature)) return SPEC_ERR_INVALID_ARG;
  if (workspace == nullptr || workspace_bytes < spec_verify_stochastic_stats_workspace_bytes(B, V)) return SPEC_ERR_WORKSPACE;
  if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return SPEC_ERR_INVALID_ARG;
  return launch_stochastic_walk(B, N, V, logits_dtype, logits_llm, probs_ssm, R, ssm_row, tree_token, tree_parent, u_accept,
                                u_order, u_final, 1.0f / temperature, node_max, node_sumexp, (float*)workspace, Lmax,
                                accepted_path, accepted_len, out_tokens, status, (hipStream_t)hip_stream) == hipSuccess
             ? SPEC_OK
             : SPEC_ERR_HIP;
}

static int kv_commit_impl(const spec_attn_desc_t* desc, const spec_kv_pages_t* pages, bool paged, int32_t n_layers,
                          void* const* k_caches, void* const* v_caches, const int32_t* accepted_path, int32_t Lmax,
                          const int32_t* accepted_len, const int32_t* prefix_len, int32_t* prefix_len_out, int32_t* status,
                          void* hip_stream) {
  int rc = check_desc(desc);
  if (rc != SPEC_OK) return rc;
  Pages pg = no_pages();
  if (paged && (rc = check_pages(desc, pages, &pg)) != SPEC_OK) return rc;
  if (n_layers <= 0 || Lmax <= 0) return SPEC_ERR_INVALID_ARG;
  if (n_layers > SPEC_MAX_COMMIT_LAYERS) return SPEC_ERR_UNSUPPORTED;
  if (!k_caches || !v_caches || !accepted_path || !accepted_len || !prefix_len || !prefix_len_out) return SPEC_ERR_INVALID_ARG;
  if (prefix_len_out == prefix_len) return SPEC_ERR_INVALID_ARG;
  for (int l = 0; l < n_layers; ++l)
    if (!k_caches[l] || !v_caches[l] || !aligned16(k_caches[l]) || !aligned16(v_caches[l])) return SPEC_ERR_INVALID_ARG;
  return launch_kv_commit(*desc, pg, n_layers, k_caches, v_caches, accepted_path, Lmax, accepted_len, prefix_len,
                          prefix_len_out, status, (hipStream_t)hip_stream) == hipSuccess
             ? SPEC_OK
             : SPEC_ERR_HIP;
}

int spec_kv_commit(const spec_attn_desc_t* desc, int32_t n_layers, void* const* k_caches, void* const* v_caches,
                   const int32_t* accepted_path, int32_t Lmax, const int32_t* accepted_len, const int32_t* prefix_len,
                   int32_t* prefix_len_out, int32_t* status, void* hip_stream) {
  return kv_commit_impl(desc, nullptr, false, n_layers, k_caches, v_caches, accepted_path, Lmax, accepted_len, prefix_len,
                        prefix_len_out, status, hip_stream);
}

int spec_kv_commit_paged(const spec_attn_desc_t* desc, const spec_kv_pages_t* pages, int32_t n_layers,
                         void* const* k_caches, void* const* v_caches, const int32_t* accepted_path, int32_t Lmax,
                         const int32_t* accepted_len, const int32_t* prefix_len, int32_t* prefix_len_out, int32_t* status,
                         void* hip_stream) {
  return kv_commit_impl(desc, pages, true, n_layers, k_caches, v_caches, accepted_path, Lmax, accepted_len, prefix_len,
                        prefix_len_out, status, hip_stream);
}

}  // extern "C"
