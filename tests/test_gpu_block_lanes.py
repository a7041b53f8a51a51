"""Block numbers of a paged request in the lanes of a wavefront: chunks that reach past the 64 blocks the lanes hold (needs an
MI355X), from a request's start and from its middle, over one head and over several in a row, with and without the rotary embedding.
The same tiles in the same order as in a contiguous cache, so the outputs agree bit for bit; entries outside the pool are flagged
wherever they lie among the blocks a request uses, and nowhere else."""
import numpy as np
import pytest
import torch

from oracle import spec_oracle as orc
from paper_2305_09781_amd import workloads as wl
from test_balanced_deal import cut_into, query_groups
from test_gpu_paged import _paged_inputs
from test_gpu_parity import DEV, _bits, _dev

pytestmark = pytest.mark.gpu

CASES = [
    # D, H, H_kv, N: the few-query kernel, the wide kernel's three shapes, the 32-query kernel
    (128, 2, 2, 9), (64, 2, 2, 16), (128, 2, 2, 20), (128, 4, 1, 14), (64, 2, 1, 100), (128, 2, 2, 100), (128, 8, 1, 12),
]


def _paged_like_contiguous(spec, D, H, H_kv, N, P, plan, bad_blocks, rope=False):
    """The fused call over a paged cache of 64-row blocks and over a contiguous one: outputs and caches bit for bit; then with one
    block number outside the pool at a time."""
    cfg, inp, kp, vp, table = _paged_inputs("bf16", 1, H, H_kv, D, (P, P), N, "random_branching", 64, seed=P + N, unused_entry=1 << 30)
    rest = (_dev(inp["tree_parent"]), _dev(inp["tree_depth"]), _dev(inp["prefix_len"]))
    q, kn, vn = (_dev(inp[k][0]) for k in ("q", "k_new", "v_new"))
    angles = tuple(_dev(t) for t in wl.make_rope_tables(P + N, D))

    def call(kc, vc, tab, status):
        kw = dict(status=status, max_prefix_len=P, plan=plan)
        if rope:
            return spec.spec_tree_attention_append_rope(q, kn, vn, kc, vc, *rest, *angles, block_table=tab, **kw)
        if tab is not None:
            return spec.spec_tree_attention_append_paged(q, kn, vn, kc, vc, tab, *rest, **kw)
        return spec.spec_tree_attention_append(q, kn, vn, kc, vc, *rest, **kw)

    kcd, vcd = _dev(inp["k_cache"][0]), _dev(inp["v_cache"][0])
    out_c = call(kcd, vcd, None, None)
    for bad in (None, *bad_blocks):
        tab = table.clone()
        if bad is not None:
            tab[0, bad] = kp.shape[0] + 7
        kpd, vpd = _dev(kp), _dev(vp)
        status = torch.zeros(1, dtype=torch.int32, device=DEV)
        out = call(kpd, vpd, _dev(tab), status)
        torch.cuda.synchronize()
        assert status.cpu().tolist() == [0 if bad is None else orc.ST_BAD_BLOCK], bad
        if bad is None:
            assert np.array_equal(_bits(out_c), _bits(out))
            n = np.array([P + N])
            for pool, cache in ((kpd, kcd), (vpd, vcd)):
                got = orc.paged_gather(_bits(pool), tab.numpy(), 64, n)
                assert np.array_equal(got[0, :, :P + N], _bits(cache)[0, :, :P + N])
    if not rope:
        kco = inp["k_cache"][0].clone()
        kco[0, :, P:P + N] = inp["k_new"][0][0].transpose(0, 1)
        assert np.array_equal(_bits(kcd)[0, :, :P + N], _bits(kco)[0, :, :P + N])


@pytest.mark.parametrize("D,H,H_kv,N", CASES)
@pytest.mark.parametrize("P", [4095 - 64, 4096, 8192 + 130])
def test_chunks_past_the_blocks_in_the_lanes(spec, D, H, H_kv, N, P):
    blocks = (P + N + 63) // 64
    _paged_like_contiguous(spec, D, H, H_kv, N, P, (16384, -1, 0), (0, min(63, blocks - 1), min(64, blocks - 1), blocks - 1))


@pytest.mark.parametrize("D,N,heads", [(64, 100, 2), (64, 128, 3), (128, 70, 2), (128, 100, 3)])
def test_several_heads_of_a_workgroup_past_the_blocks_in_the_lanes(spec, D, N, heads):
    """The lanes go back to the first block at the border between two heads, beside the last tile of the head before."""
    P = 4096 + 700
    _paged_like_contiguous(spec, D, 3, 3, N, P, (16384, -1, heads), (0, 64, (P + N - 1) // 64))


@pytest.mark.parametrize("D,H,H_kv,N", [(128, 2, 2, 9), (128, 2, 2, 16), (64, 2, 2, 12), (128, 2, 2, 30), (128, 2, 2, 100)])
@pytest.mark.parametrize("P", [4096, 8192 + 130])
def test_rotary_calls_past_the_blocks_in_the_lanes(spec, D, H, H_kv, N, P):
    _paged_like_contiguous(spec, D, H, H_kv, N, P, (16384, -1, 0), (0, 64, (P + N - 1) // 64), rope=True)


@pytest.mark.parametrize("D,H,H_kv,N", CASES)
@pytest.mark.parametrize("rope", [False, True])
def test_chunks_of_the_deal_past_the_blocks_in_the_lanes(spec, D, H, H_kv, N, rope):
    """Two chunks a pair and more, each of more than 64 blocks: all but the first start at a block of their own."""
    P = 16384 + 100
    pairs = H_kv * query_groups(H, H_kv, N)
    chunks = cut_into([P], N, pairs, 32 if N <= 16 and H == H_kv else 64, 2 * pairs)[0]
    assert chunks > 1 and (P // 64) // chunks > 64
    last = (P + N - 1) // 64
    _paged_like_contiguous(spec, D, H, H_kv, N, P, (0, 2 * pairs, 0), (0, last // 2 + 3, last // 2 + 70, last), rope=rope)
