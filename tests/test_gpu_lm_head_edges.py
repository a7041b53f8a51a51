"""LM head at the edges of its tiles: rows of hidden around 32, 64, 128 and 256, vocabularies around 64 and 128 rows and where
the tile changes, K of four stages (fewer than the ring holds) and of many, logits at an address that is only 8-byte aligned,
equal rows of W in different workgroups. Bars: those of the other LM head tests (float32 accumulation, worst case)."""
import numpy as np
import pytest
import torch

from test_gpu_lm_head import DEV, _check_rows, _dev, _inputs, _stats_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,V", [(32, 256, 64), (33, 256, 65), (64, 512, 63), (65, 512, 128), (128, 256, 16384), (31, 512, 16385),
                                   (255, 256, 1000), (256, 1024, 129), (257, 512, 513), (600, 256, 200)])
def test_lm_head_tile_edges(spec, M, K, V):
    h, w = _inputs(M, K, V, seed=M * 7 + V)
    arg, mx = spec.spec_lm_head_argmax(_dev(h), _dev(w), want_max=True)
    torch.cuda.synchronize()
    _check_rows(arg.cpu().numpy(), mx.cpu().numpy().astype(np.float64), h, w)
    _stats_case(spec, M, K, V, 0.9, seed=M * 7 + V)


@pytest.mark.parametrize("M,V,K", [(12, 20000, 1024), (70, 20001, 1024), (130, 9000, 1024), (12, 20000, 2048), (70, 16385, 4096),
                                   (100, 20001, 2048), (200, 20000, 2048)])
def test_equal_rows_of_the_weight_matrix_give_equal_logits(spec, M, V, K):
    """The same row of W at places of different lanes, wavefronts and workgroups (that start with different parts of K): bit-equal
    logits, so the lowest token wins whatever its workgroup."""
    h, w = _inputs(M, K, V, seed=V)
    places = [V - 1, 5, 40, 70, 133, 2100, 5000, 5001]
    w[places] = w[17] * 40      # the largest logit of about half of the rows
    logits, arg, _, _ = spec.spec_lm_head_logits_stats(_dev(h), _dev(w))
    arg2, mx = spec.spec_lm_head_argmax(_dev(h), _dev(w), want_max=True)
    torch.cuda.synchronize()
    got = logits.view(torch.int16)[:, places].cpu().numpy()
    assert (got == got[:, :1]).all()
    for a in (arg.cpu().numpy(), arg2.cpu().numpy()):
        hit = np.isin(a, places)
        assert hit.mean() > 0.1 and (a[hit] == 5).all()


def test_logits_at_an_eight_byte_aligned_address(spec):
    M, K, V = 40, 512, 1000
    h, w = _inputs(M, K, V, seed=9)
    want, arg, mx, se = spec.spec_lm_head_logits_stats(_dev(h), _dev(w))
    buf = torch.empty(M * V + 4, dtype=torch.bfloat16, device=DEV)
    out = (buf[4:].view(M, V), torch.empty_like(arg), torch.empty_like(mx), torch.empty_like(se))
    spec.spec_lm_head_logits_stats(_dev(h), _dev(w), out=out)
    torch.cuda.synchronize()
    assert torch.equal(out[0], want) and torch.equal(out[1], arg) and torch.equal(out[3], se)


@pytest.mark.parametrize("K,V", [(768, 1000), (1024, 8000), (512, 16384), (512, 16385), (768, 20000), (2048, 16385), (4096, 17000)])
def test_a_row_has_the_same_logits_in_a_batch_of_any_size(spec, K, V):
    """Every tile of `hidden` and of the vocabulary sums a logit in the same order: bit-equal maxima before rounding, logits and
    arg-max, from one row to three slices."""
    M = 300
    h, w = _inputs(M, K, V, seed=V + 1)
    h, w = _dev(h), _dev(w)
    arg, mx = spec.spec_lm_head_argmax(h, w, want_max=True)
    logits, _, _, _ = spec.spec_lm_head_logits_stats(h, w)
    for m in (1, 16, 32, 33, 64, 65, 128, 129, 256, 257):
        a, x = spec.spec_lm_head_argmax(h[:m], w, want_max=True)
        lo, _, _, _ = spec.spec_lm_head_logits_stats(h[:m], w)
        torch.cuda.synchronize()
        assert torch.equal(x, mx[:m]) and torch.equal(a, arg[:m]) and torch.equal(lo, logits[:m]), m


def test_short_sums_over_a_large_vocabulary_keep_the_stream_up(spec):
    """Four workgroups' worth of starts and ends per compute unit: one row against 128256 x 256 reads W at 3.9 TB/s where they
    overlap, at 2.7 where they do not (four different W in turn, so that none is left in a cache)."""
    K, V = 256, 128256
    g = torch.Generator(device=DEV).manual_seed(2)
    ws = [torch.randn((V, K), generator=g, device=DEV, dtype=torch.bfloat16) for _ in range(4)]
    h = torch.randn((1, K), generator=g, device=DEV, dtype=torch.bfloat16)
    scratch = torch.empty(spec.spec_lm_head_argmax_workspace_bytes(1, V), dtype=torch.uint8, device=DEV)
    spec.spec_lm_head_argmax(h, ws[0], workspace=scratch)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for i in range(20):
            spec.spec_lm_head_argmax(h, ws[i % 4], workspace=scratch)
    times = []
    for _ in range(7):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        graph.replay()
        end.record()
        torch.cuda.synchronize()
        times.append(start.elapsed_time(end) / 20 * 1e-3)
    rate = V * K * 2 / sorted(times)[3]
    assert rate > 3.2e12, rate
