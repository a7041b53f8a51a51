"""The balanced deal's arithmetic on the host: which (K/V head, chunk, query group) a workgroup gets is a permutation, chunks
cover a request's tiles, and in the order of their sizes every chunk of every request is found once. The functions are the kernels'
own (csrc/spec_internal.h), compiled for the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cmath>
#include <cstdlib>
#include <vector>
#include "spec_internal.h"
using namespace spec;
static void check(bool ok, const char* what, int a, int b, int c) {
  if (!ok) { printf("%s: %d %d %d\n", what, a, b, c); exit(1); }
}
int main() {
  for (int n_qg = 1; n_qg <= 9; ++n_qg)
    for (int units = 1; units <= 130; ++units) {
      std::vector<int> at(units * n_qg, -1);
      for (int r = 0; r < units * n_qg; ++r) {
        const DealUnit u = deal_unit(r, n_qg, units);
        check(u.unit >= 0 && u.unit < units && u.qg >= 0 && u.qg < n_qg, "range", r, n_qg, units);
        int& place = at[u.unit * n_qg + u.qg];
        check(place < 0, "twice", r, n_qg, units);
        place = r;
      }
      for (int u = 0; u < units / 8 * 8; ++u)      // the groups of a unit in a whole block: on one of the eight XCDs
        for (int g = 1; g < n_qg; ++g)
          check((at[u * n_qg + g] - at[u * n_qg]) % 8 == 0, "XCD", u, n_qg, units);
    }
  for (int tb = 1; tb <= 400; ++tb)
    for (int share = 1; share <= 90; ++share) {
      const int chunks = deal_chunks(tb, share), per = deal_chunk_tiles(tb, chunks), used = deal_chunks(tb, per);
      check(per >= 1 && per <= share, "share", tb, share, per);
      check(used <= chunks && (used > 1) == (chunks > 1), "count", tb, share, used);
      // (a workgroup whose request has one chunk writes the output, so one must be all that is used; the workgroup of a request's
      // last key signs its partial, so no slot below it may be empty)
      check(per * (used - 1) < tb && tb <= per * used, "cover", tb, share, per);
    }
  for (int cus : {1, 3, 256})   // every chunk once; two workgroups of a compute unit take chunks whose places add up to the same
    for (long count : {1L, 2L, 5L, 6L, 7L, 255L, 256L, 257L, 400L, 511L, 512L, 513L, 1500L}) {
      std::vector<int> seen(count, 0);
      for (long id = 0; id < count; ++id) {
        const long at = deal_place(id, count, cus);
        check(at >= 0 && at < count && !seen[at]++, "place", (int)id, (int)count, cus);
        if (count <= 2l * cus && id >= cus) check(at + deal_place(id - cus, count, cus) == count - 1, "pair", (int)id, (int)count, cus);
      }
    }
  // Batches of up to 64 requests in descending order of their chunks' sizes, as deal_find numbers them: the requests that come before
  // a lane's own are added up by deal_before. Lengths all equal, few different ones, with requests that do not fit (no tiles).
  unsigned seed = 1;
  auto random = [&](int n) { return (int)((seed = seed * 1664525u + 1013904223u) >> 8) % n; };
  for (int B : {1, 2, 3, 17, 40, 63, 64})
    for (int kinds : {1, 2, 5, 200})
      for (int share : {1, 3, 8, 300})
        for (int n_qg : {1, 3}) {
          const int kv_heads = 2, H = kv_heads * n_qg;
          std::vector<int> tb(B), v(B), size(B), incl(B);
          for (int b = 0; b < B; ++b) {
            tb[b] = random(7) == 0 ? 0 : 1 + random(kinds);
            v[b] = deal_chunks(tb[b], share);
            size[b] = v[b] > 0 ? deal_chunk_tiles(tb[b], v[b]) : 0;
          }
          long count = 0;
          for (int b = 0; b < B; ++b) {
            incl[b] = v[b];
            for (int i = 0; i < B; ++i) incl[b] += deal_before(size[i], i, size[b], b) ? v[i] : 0;
            count += v[b] * H;
          }
          bool equal = true;   // chunks of one size are numbered as the requests stand
          for (int b = 0, some = 0; b < B; ++b) {
            if (size[b] > 0 && some > 0) equal = equal && size[b] == some;
            some = size[b] > 0 ? size[b] : some;
          }
          for (int b = 0, sum = 0; b < B; ++b) {
            sum += v[b];
            if (equal && v[b] > 0) check(incl[b] == sum, "as they stand", b, B, share);
          }
          std::vector<std::vector<int>> seen(B);
          for (int b = 0; b < B; ++b) seen[b].assign(H * v[b], 0);
          int before = 1 << 30;
          for (long id = 0; id < count; ++id) {
            int b = -1, hits = 0;
            for (int i = 0; i < B; ++i)
              if ((long)incl[i] * H > id && (long)(incl[i] - v[i]) * H <= id) b = i, ++hits;
            check(hits == 1, "one request", (int)id, B, share);
            check(size[b] <= before, "descending", (int)id, B, share);
            before = size[b];
            const int r = (int)(id - (long)(incl[b] - v[b]) * H);
            check(r >= 0 && r < H * v[b], "number in the request", r, B, share);
            const DealUnit u = deal_unit(r, n_qg, kv_heads * v[b]);
            check(!seen[b][u.unit * n_qg + u.qg]++, "chunk", (int)id, b, share);
          }
        }
  // the kernels' division: float32 reciprocal (one unit off either way included) and one correction
  auto by_reciprocal = [](int a, int b, int ulp) {
    float rcp = 1.0f / (float)b;
    for (int i = 0; i < abs(ulp); ++i) rcp = nextafterf(rcp, ulp > 0 ? 2.0f : 0.0f);
    const int q = (int)((float)a * rcp), rest = a - q * b;
    return q + (rest >= b) - (rest < 0);
  };
  for (int b : {1, 2, 3, 7, 22, 64, 255, 1000, 4095, 65537, 1048575, 16777217, 0x3ffffffe, 0x3fffffff})
    for (long q : {0L, 1L, 2L, 63L, 1000L, 65535L, 1048576L, 2097151L})
      for (long d = -2; d <= 2; ++d) {
        const long a = q * b + d;
        if (a < 0 || a > 0x7fffffffL || a / b >= 1 << 22) continue;
        for (int ulp = -1; ulp <= 1; ++ulp) check(by_reciprocal((int)a, b, ulp) == a / b, "division", (int)a, b, ulp);
        check(deal_quotient((int)a, b) == a / b, "quotient", (int)a, b, 0);
      }
  check(request_tiles(-1, 16, 100, 64) == 0 && request_tiles(85, 16, 100, 64) == 0 && request_tiles(84, 16, 100, 64) == 2 &&
        request_tiles(0, 1, 1, 32) == 1, "tiles", 0, 0, 0);
  puts("ok");
}
"""


def cut_into(lens, N, virtual_heads, tile, wgs):
    """Chunks per (request, virtual head) pair of a deal that aims at `wgs` chunks, as the kernels find them."""
    tiles = [-(-(p + N) // tile) for p in lens]
    cap = max(wgs, virtual_heads * len(tiles))
    share = max(1, -(-sum(tiles) * virtual_heads // cap))
    while virtual_heads * sum(-(-t // share) for t in tiles) > cap:
        share = max(share + 1, share * virtual_heads * sum(-(-t // share) for t in tiles) // cap)
    return [-(-t // -(-t // -(-t // share))) for t in tiles]


def query_groups(H, H_kv, N):
    """Query groups per K/V head in the bf16 kernels: whole heads, eight 16-query tiles a workgroup at most."""
    group, per_head = H // H_kv, -(-N // 16)
    return -(-group // min(group, max(1, 8 // per_head)))


def test_deal_is_a_permutation_and_covers_every_tile(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("needs a host compiler and the HIP headers")
    src, exe = tmp_path / "deal.cc", tmp_path / "deal"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2305_09781_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout


def test_small_hints_leave_pairs_whole():
    """A pair is cut only if the hint leaves room for it: tests that mean to cut pairs check it with cut_into."""
    assert cut_into([40, 170, 300], 32, 2, 64, 7) == [1, 1, 1]
    assert cut_into([40, 170, 300], 32, 2, 64, 24) == [2, 4, 6]
    assert query_groups(32, 2, 16) == 2 and query_groups(12, 2, 40) == 3 and query_groups(32, 32, 128) == 1
