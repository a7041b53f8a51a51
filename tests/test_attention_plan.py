"""The launch plans that spec_tree_attention chooses without hints, read from the size of the workspace it asks for (float32
partials [n_splits][B][H][N][D + 2]). Without a GPU the library plans for 256 compute units."""
import ctypes

import pytest
import torch

from paper_2305_09781_amd import binding

pytestmark = pytest.mark.skipif(torch.cuda.is_available() and torch.cuda.get_device_properties(0).multi_processor_count != 256,
                                reason="expectations are for 256 compute units")


def _slots(B, H, D, N, P, H_kv=None, dtype=binding.SPEC_BF16, wgs=0, chunk=0, block=0):
    H_kv = H_kv or H
    S = P + N
    d = binding.AttnDesc(B=B, H=H, H_kv=H_kv, D=D, N=N, S_cap=S, dtype=dtype, max_prefix_len=P, q_stride_b=N * H * D, q_stride_n=H * D,
                         q_stride_h=D, kv_stride_b=H_kv * S * D, kv_stride_h=S * D, kv_stride_s=D, new_stride_b=N * H_kv * D,
                         new_stride_n=H_kv * D, new_stride_h=D, softmax_scale=0.0, plan_chunk_keys=chunk, plan_balanced_wgs=wgs,
                         plan_heads_per_wg=0)
    if block:
        d.S_cap = -(-S // block) * block
        d.kv_stride_b, d.kv_stride_h = H_kv * block * D, block * D
        pages = binding.KvPages(256, d.S_cap // block, block, B * d.S_cap // block)
        got = binding.spec_tree_attention_paged_workspace_bytes(d, pages)
    else:
        got = binding.load().spec_tree_attention_workspace_bytes(ctypes.byref(d))
    up = lambda x: (x + 255) // 256 * 256  # noqa: E731
    for n in range(1, 600):
        rows = B * H * n * N
        if n > 1 and up(rows * D * 4) + up(rows * 8) == got:
            return n
    assert got == 0
    return 1


@pytest.mark.parametrize("B,H,H_kv,D,N,P,chunks", [
    # few-query kernel: chunks of the prefix at multiples of 32 keys
    (1, 12, 12, 128, 3, 1589, 6),       # 288 keys, the last chunk 152 (chunks of 320 would end in one of 312)
    (2, 12, 12, 128, 1, 1874, 7),
    (2, 12, 12, 64, 2, 1883, 7),
    # ... at multiples of 64 where the last one would be as long as the others
    (1, 32, 32, 64, 3, 1414, 5),        # 320, the last 137 (288 would end in 265)
    (1, 12, 12, 128, 12, 554, 2),
    # wide kernel: multiples of its 64-key tile
    (2, 32, 8, 128, 3, 4825, 16),
    (1, 24, 6, 128, 7, 3205, 11),
    (1, 32, 32, 128, 40, 1024, 5),      # the tree in a chunk of its own
    (1, 32, 32, 64, 20, 4432, 14),
    # ... for one workgroup per compute unit where two query tiles share a head dimension of 128 (14 chunks: 23.8 us, 8: 21.4)
    (1, 32, 32, 128, 20, 4432, 8),
    (4, 32, 32, 128, 21, 769, 2),
    (1, 64, 64, 64, 20, 3225, 8),
    # ... and for three tiles and more, from four fifths of the compute units on
    (4, 52, 52, 128, 40, 600, 1),
    (4, 51, 51, 128, 40, 600, 2),
    # ... uncut up to 20 D keys
    (8, 32, 32, 128, 60, 2500, 1),
    (8, 32, 32, 128, 60, 2501, 2),
    (8, 32, 32, 64, 60, 1221, 2),
    # ... cut up to 8 D keys a chunk of several requests, 20 D of one
    (4, 32, 32, 128, 40, 2009, 2),
    (4, 32, 32, 128, 40, 2010, 4),
    (1, 32, 32, 128, 40, 20447, 8),
    (1, 32, 32, 128, 40, 20448, 16),
    # ... down to 128 keys where most of the device is idle: up to half a workgroup per compute unit, up to eight chunks (and one of
    # the tree's own), two only of few pairs with a head dimension of 128
    (1, 32, 32, 128, 40, 400, 3),
    (1, 12, 12, 128, 60, 963, 6),
    (1, 12, 12, 128, 60, 964, 8),
    (1, 12, 12, 128, 60, 1000, 9),
    (1, 12, 12, 128, 60, 300, 2),
    (1, 12, 12, 64, 60, 300, 1),
    (1, 64, 64, 128, 50, 300, 1),
    # ... unless the last of them would be the longest, where there are workgroups to spare
    (2, 32, 8, 128, 5, 2191, 8),
    (1, 32, 8, 64, 2, 3477, 13),
    # the 32-query kernel keeps equal chunks of everything
    (1, 32, 32, 128, 100, 1024, 4),
    # one workgroup per pair
    (8, 32, 32, 128, 16, 1024, 1),
    (1, 4, 4, 64, 8, 128, 1),
])
def test_fixed_chunks(B, H, H_kv, D, N, P, chunks):
    assert _slots(B, H, D, N, P, H_kv) == chunks


@pytest.mark.parametrize("B,H,H_kv,D,N,P,chunks,contiguous", [
    # (chunks of whole 64-key tiles) wide kernel: one workgroup per compute unit for chunks of up to 3.5 D keys, uncut up to 14 D
    (1, 32, 32, 128, 20, 3100, 7, 8),
    (4, 12, 12, 128, 29, 2086, 5, 5),
    (1, 32, 32, 128, 24, 12000, 16, 8),
    (4, 32, 32, 128, 50, 1200, 4, 2),
    (8, 32, 32, 128, 60, 1732, 1, 1),
    (8, 32, 32, 128, 60, 1733, 2, 1),
    # 32-query kernel: chunks of up to 6 D of several requests, 12 D of one (20 D contiguous)
    (2, 32, 32, 128, 101, 2974, 4, 4),
    (2, 32, 32, 128, 101, 2975, 7, 8),
    (1, 32, 32, 128, 100, 12195, 8, 8),
    (1, 32, 32, 128, 100, 12196, 15, 8),
])
def test_fixed_chunks_paged(B, H, H_kv, D, N, P, chunks, contiguous):
    assert (_slots(B, H, D, N, P, H_kv, block=64), _slots(B, H, D, N, P, H_kv)) == (chunks, contiguous)
