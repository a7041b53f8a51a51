"""The balanced deal over up to as many and over more requests than a wavefront has lanes (lengths are read 64 requests at a time;
the wide kernels take the chunks of up to 64 requests by size), with requests that contribute no tiles, on every bf16 kernel, pairs
whole and cut, chunks on some, on most and on more than all of the compute units. Bar: that of the other attention tests."""
import numpy as np
import pytest
import torch

from paper_2305_09781_amd import workloads as wl
from test_gpu_parity import _balanced_wgs, _check_attention, _oracle_append_attention, _run_append_attention

pytestmark = pytest.mark.gpu


def _check_deal(spec, inp, out_of_range, wgs):
    B = inp["prefix_len"].numel()
    ref, _, _ = _oracle_append_attention(inp)
    for b in out_of_range:              # no room for the tree: flagged, zero outputs, no tiles in the deal
        inp["prefix_len"][b] = 201
    status = torch.zeros(B, dtype=torch.int32, device="cuda:0")
    with _balanced_wgs(wgs):
        out, _, _ = _run_append_attention(spec, inp, status=status, fused=True)
    st = status.cpu().numpy()
    assert [b for b in range(B) if st[b]] == out_of_range and (st[out_of_range] == spec.ST_CAPACITY).all()
    ok = [b for b in range(B) if b not in out_of_range]
    assert (out[out_of_range] == 0).all()
    _check_attention(out[ok], ref[ok], torch.bfloat16)


@pytest.mark.parametrize("B,N,wgs", [(63, 5, 17), (64, 5, 200), (65, 20, 31), (130, 5, 300), (70, 70, 90), (30, 5, 130), (70, 16, 300),
                                     (65, 20, 300), (70, 70, 320), (66, 100, 330),
                                     (30, 20, 90), (63, 70, 320), (64, 20, 300), (64, 70, 140), (40, 100, 300), (64, 100, 600), (30, 100, 70)])
def test_deal_over_many_requests(spec, B, N, wgs):
    cfg = wl.Config(91, "deal", "bf16", B=B, H=2, D=128, P=(0, 200), N=N, tree="random_branching")
    inp = wl.make_attention_inputs(cfg, seed=4000 + B, S_cap=200 + N)
    _check_deal(spec, inp, [3, B - 1], wgs)


@pytest.mark.parametrize("B,N,wgs,out_of_range", [(25, 20, 150, []), (25, 20, 150, [0, 7, 24]), (40, 100, 300, [0]), (64, 70, 300, [63]), (5, 20, 2, [0])])
def test_deal_over_equal_lengths(spec, B, N, wgs, out_of_range):
    """Chunks of one size are numbered without being ordered; the requests without tiles among them, the first one too."""
    cfg = wl.Config(92, "deal", "bf16", B=B, H=2, D=128, P=(150, 150), N=N, tree="random_branching")
    _check_deal(spec, wl.make_attention_inputs(cfg, seed=4100 + B, S_cap=200 + N), out_of_range, wgs)
