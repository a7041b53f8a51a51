"""Block numbers of a paged request in the lanes of a wavefront: chunks that reach past the 64 blocks the lanes hold (needs an
MI355X). The same tiles in the same order as in a contiguous cache, so the outputs agree bit for bit; entries outside the pool
are flagged wherever they lie among the blocks a request uses, and nowhere else."""
import numpy as np
import pytest
import torch

from oracle import spec_oracle as orc
from test_gpu_paged import _paged_inputs
from test_gpu_parity import DEV, _bits, _dev

pytestmark = pytest.mark.gpu

CASES = [
    # D, H, H_kv, N: the few-query kernel, the wide kernel's three shapes, the 32-query kernel
    (128, 2, 2, 9), (64, 2, 2, 16), (128, 2, 2, 20), (128, 4, 1, 14), (64, 2, 1, 100), (128, 2, 2, 100), (128, 8, 1, 12),
]


@pytest.mark.parametrize("D,H,H_kv,N", CASES)
@pytest.mark.parametrize("P", [4095 - 64, 4096, 8192 + 130])
def test_chunks_past_the_blocks_in_the_lanes(spec, D, H, H_kv, N, P):
    cfg, inp, kp, vp, table = _paged_inputs("bf16", 1, H, H_kv, D, (P, P), N, "random_branching", 64, seed=P + N, unused_entry=1 << 30)
    rest = (_dev(inp["tree_parent"]), _dev(inp["tree_depth"]), _dev(inp["prefix_len"]))
    q, kn, vn = (_dev(inp[k][0]) for k in ("q", "k_new", "v_new"))
    plan = (16384, -1, 0)   # one chunk
    out_c = spec.spec_tree_attention_append(q, kn, vn, _dev(inp["k_cache"][0]), _dev(inp["v_cache"][0]), *rest, max_prefix_len=P, plan=plan)
    blocks = (P + N + 63) // 64
    for bad in (None, 0, min(63, blocks - 1), min(64, blocks - 1), blocks - 1):
        tab = table.clone()
        if bad is not None:
            tab[0, bad] = kp.shape[0] + 7
        kpd, vpd = _dev(kp), _dev(vp)
        status = torch.zeros(1, dtype=torch.int32, device=DEV)
        out = spec.spec_tree_attention_append_paged(q, kn, vn, kpd, vpd, _dev(tab), *rest, status=status, max_prefix_len=P, plan=plan)
        torch.cuda.synchronize()
        assert status.cpu().tolist() == [0 if bad is None else orc.ST_BAD_BLOCK]
        if bad is None:
            assert np.array_equal(_bits(out_c), _bits(out))
            n = np.array([P + N])
            got = orc.paged_gather(_bits(kpd), tab.numpy(), 64, n)
            kco, vco = inp["k_cache"][0].clone(), inp["v_cache"][0].clone()
            kco[0, :, P:P + N] = inp["k_new"][0][0].transpose(0, 1)
            assert np.array_equal(got[0, :, :P + N], _bits(kco)[0, :, :P + N])
