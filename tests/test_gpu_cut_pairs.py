"""Balanced plans that cut (request, K/V head) pairs into chunks, on every bf16 kernel, with one to six query groups per K/V head
(numbered eight apart where eight chunks of a request make a block), contiguous and paged, with malformed trees and requests that
do not fit. Every case checks that its hint does cut. Bars: those of the other attention tests."""
import numpy as np
import pytest
import torch

from oracle import spec_oracle as orc
from paper_2305_09781_amd import workloads as wl
from test_balanced_deal import cut_into, query_groups
from test_gpu_paged import _paged_inputs
from test_gpu_parity import (DEV, _balanced_wgs, _check_attention, _dev, _f64, _oracle_append_attention, _plan,
                             _run_append_attention)

pytestmark = pytest.mark.gpu

CASES = [
    # B, H, H_kv, D, (P lo, hi), N, workgroups
    (3, 2, 2, 128, (40, 300), 16, 24),       # few-query kernel
    (3, 2, 2, 128, (40, 300), 32, 24),       # two query tiles
    (2, 2, 2, 64, (100, 700), 32, 17),
    (2, 4, 2, 64, (100, 700), 16, 12),       # two heads of one tile
    (2, 3, 3, 128, (100, 700), 64, 30),      # four query tiles
    (2, 2, 2, 128, (60, 700), 100, 20),      # 32-query kernel
    (1, 2, 2, 128, (900, 900), 128, 11),
    (1, 2, 2, 64, (900, 900), 128, 13),      # eight wavefronts
    # several query groups; (K/V heads x chunks) of a request below eight, eight, above and not a multiple of it
    (2, 32, 2, 128, (30, 700), 16, 24),      # 2 groups
    (1, 32, 2, 128, (640, 640), 16, 24),
    (1, 32, 4, 128, (250, 250), 32, 16),
    (2, 12, 2, 128, (100, 700), 40, 66),     # 3 groups of two heads
    (2, 36, 3, 64, (100, 500), 16, 72),      # 2 groups, the second one short
    (1, 48, 1, 64, (900, 900), 16, 50),      # 6 groups of one K/V head
    (3, 9, 3, 128, (0, 900), 90, 120),       # a group per query head
]


def _lens_are_cut(lens, H, H_kv, N, wgs):
    n_qg = query_groups(H, H_kv, N)
    few = N <= 16 and H == H_kv
    chunks = cut_into([int(p) for p in lens], N, H_kv * n_qg, 32 if few else 64, wgs)
    assert max(chunks) > 1
    return n_qg, chunks


@pytest.mark.parametrize("case", CASES, ids=lambda c: "B%d-H%d/%d-D%d-P%d-N%d-wg%d" % (c[0], c[1], c[2], c[3], c[4][1], c[5], c[6]))
def test_cut_pairs(spec, case):
    B, H, H_kv, D, P, N, wgs = case
    cfg = wl.Config(95, "cut", "bf16", B=B, H=H, D=D, P=P if P[0] != P[1] else P[0], N=N, tree="random_branching", H_kv=H_kv)
    inp = wl.make_attention_inputs(cfg, seed=9000 + N + H + B, S_cap=P[1] + N + 5)
    _lens_are_cut(inp["prefix_len"], H, H_kv, N, wgs)
    ref, kco, vco = _oracle_append_attention(inp)
    for fused in (False, True):
        status = torch.zeros(B, dtype=torch.int32, device=DEV)
        if fused or H == H_kv:
            with _balanced_wgs(wgs):
                out, kc, vc = _run_append_attention(spec, inp, status=status, fused=fused)
            _check_attention(out, ref, cfg.torch_dtype)
            assert (status.cpu().numpy() == 0).all()
            assert np.array_equal(kc.double().cpu().numpy(), kco) and np.array_equal(vc.double().cpu().numpy(), vco), fused


def test_the_cases_reach_whole_blocks_of_eight_chunks_and_what_is_left_over():
    """What the numbering of query groups can do: no whole block, whole blocks only, and both."""
    seen = set()
    for B, H, H_kv, D, P, N, wgs in CASES:
        if query_groups(H, H_kv, N) > 1 and P[0] == P[1]:
            units = H_kv * cut_into([P[0]] * B, N, H_kv * query_groups(H, H_kv, N), 64, wgs)[0]
            seen.add((units >= 8, units % 8 != 0))
    assert seen >= {(True, True), (True, False)}


@pytest.mark.parametrize("B,H,H_kv,D,P,N,wgs,bt", [(3, 2, 2, 128, (40, 300), 16, 24, 64), (2, 2, 2, 128, (60, 700), 100, 20, 128),
                                                    (2, 32, 2, 128, (30, 700), 16, 40, 64), (2, 12, 2, 64, (100, 700), 40, 66, 256),
                                                    (2, 4, 2, 128, (100, 700), 32, 24, 64)])
def test_cut_pairs_of_a_paged_cache(spec, B, H, H_kv, D, P, N, wgs, bt):
    cfg, inp, kp, vp, table = _paged_inputs("bf16", B, H, H_kv, D, P, N, "random_branching", bt, seed=700 + N + bt, unused_entry=1 << 30)
    pl, par = inp["prefix_len"].numpy(), inp["tree_parent"].numpy()
    _lens_are_cut(pl, H, H_kv, N, wgs)
    kpo, vpo = _f64(kp), _f64(vp)
    orc.kv_append_paged(kpo, vpo, table.numpy(), bt, table.shape[1] * bt, _f64(inp["k_new"][0]), _f64(inp["v_new"][0]), pl)
    ref = orc.tree_attention_paged(_f64(inp["q"][0]), kpo, vpo, table.numpy(), bt, par, pl)
    kpd, vpd = _dev(kp), _dev(vp)
    status = torch.zeros(B, dtype=torch.int32, device=DEV)
    with _balanced_wgs(wgs):
        out = spec.spec_tree_attention_append_paged(_dev(inp["q"][0]), _dev(inp["k_new"][0]), _dev(inp["v_new"][0]), kpd, vpd, _dev(table),
                                                    _dev(inp["tree_parent"]), _dev(inp["tree_depth"]), _dev(inp["prefix_len"]),
                                                    status=status, max_prefix_len=int(pl.max()), plan=_plan())
    torch.cuda.synchronize()
    assert (status.cpu().numpy() == 0).all()
    assert np.array_equal(kpd.double().cpu().numpy(), kpo) and np.array_equal(vpd.double().cpu().numpy(), vpo)
    _check_attention(out, ref, torch.bfloat16)


@pytest.mark.parametrize("H,H_kv,D,N,wgs", [(2, 2, 128, 16, 40), (2, 2, 128, 40, 40), (2, 2, 128, 100, 40), (2, 2, 64, 100, 40),
                                            (32, 2, 128, 16, 80)])
def test_malformed_trees_on_cut_pairs(spec, H, H_kv, D, N, wgs):
    """Zeros and a status bit for a malformed tree whose pairs are cut, for one that is wrong in its depths only, and for a
    request that does not fit (no tiles in the deal); the others are unaffected."""
    cfg = wl.Config(91, "bad", "bf16", B=4, H=H, D=D, P=500, N=N, tree="random_parent", H_kv=H_kv)
    inp = wl.make_attention_inputs(cfg, seed=5, S_cap=500 + N)
    inp["tree_parent"][1, 5] = 9
    inp["tree_depth"][2, 7] += 1
    inp["prefix_len"][3] = 501
    _lens_are_cut([500, 500, 500], H, H_kv, N, wgs)
    ref, _, _ = _oracle_append_attention(inp, bsel=[0])
    for fused in (False, True):
        if not fused and H != H_kv:
            continue
        status = torch.zeros(4, dtype=torch.int32, device=DEV)
        with _balanced_wgs(wgs):
            out, _, _ = _run_append_attention(spec, inp, status=status, fused=fused)
        assert status.cpu().tolist() == [0, orc.ST_BAD_TREE, orc.ST_BAD_TREE, orc.ST_CAPACITY]
        assert (out[1:].float() == 0).all()
        _check_attention(out[:1], ref, torch.bfloat16)


@pytest.mark.parametrize("B,H,N,P,slots", [(2, 65, 16, 4100, 5), (2, 129, 20, 4200, 9)])
def test_deals_that_are_chosen_without_a_hint(spec, B, H, N, P, slots):
    """Fewer than two chunks per pair at the stated maximum: contiguous shares of the few-query kernel (256 workgroups for 130 pairs)
    and twice the resident workgroups of the wide one (1024 for 258 pairs), read from the size of the workspace. The requests are shorter than the maximum."""
    D = 64
    cfg = wl.Config(96, "default", "bf16", B=B, H=H, D=D, P=(150, P), N=N, tree="random_branching")
    inp = wl.make_attention_inputs(cfg, seed=N, S_cap=P + N)
    q, kc, vc = _dev(inp["q"][0]), _dev(inp["k_cache"][0]), _dev(inp["v_cache"][0])
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        rows = B * H * slots * N
        up = lambda x: (x + 255) // 256 * 256  # noqa: E731
        assert spec.spec_tree_attention_workspace_bytes(spec.make_desc(q, kc, P)) == up(rows * D * 4) + up(rows * 8)
    status = torch.zeros(B, dtype=torch.int32, device=DEV)
    out = spec.spec_tree_attention_append(q, _dev(inp["k_new"][0]), _dev(inp["v_new"][0]), kc, vc, _dev(inp["tree_parent"]),
                                          _dev(inp["tree_depth"]), _dev(inp["prefix_len"]), status=status, max_prefix_len=P)
    torch.cuda.synchronize()
    assert (status.cpu().numpy() == 0).all()
    out_h = out.cpu()
    for b in range(B):
        ref, _, _ = _oracle_append_attention(inp, bsel=[b])
        _check_attention(out_h[b:b + 1], ref, torch.bfloat16)
