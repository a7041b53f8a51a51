"""Partials that say themselves where they end (needs an MI355X): whatever a workspace held before a call - zeros, all bits set, the
mark of a pair without partials in every row, another batch's partials - the outputs are the same bits and agree with the oracle, on
every kernel that cuts a pair, under fixed chunks and under the balanced plans, with requests of one chunk and of many, a malformed
tree in each and a request that does not fit."""
import numpy as np
import pytest
import torch

from oracle import spec_oracle as orc
from paper_2305_09781_amd import workloads as wl
from test_gpu_parity import DEV, _check_attention, _dev, _oracle_append_attention

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, H, H_kv, D, N, plan (chunk_keys, balanced_wgs, heads_per_wg)
    ("bf16", 2, 2, 128, 16, (128, -1, 0)),     # few-query kernel: seven chunks of the longest request (eight fetched together)
    ("bf16", 2, 2, 64, 5, (320, -1, 0)),       # three (four fetched together)
    ("bf16", 2, 2, 128, 16, (0, 12, 0)),       # contiguous shares
    ("bf16", 2, 2, 128, 16, (0, 40, 0)),       # balanced deal
    ("bf16", 2, 2, 128, 40, (128, -1, 0)),     # wide kernel
    ("bf16", 2, 2, 128, 30, (0, 40, 0)),
    ("bf16", 12, 2, 128, 40, (0, 90, 0)),      # three query groups of two heads
    ("bf16", 2, 2, 64, 100, (0, 30, 0)),       # eight wavefronts; the tree spans two chunks
    ("bf16", 2, 2, 64, 100, (192, -1, 0)),     # ... under fixed chunks
    ("bf16", 2, 2, 128, 100, (128, -1, 0)),    # 32-query kernel
    ("bf16", 32, 2, 128, 16, (0, 80, 0)),      # two query groups
    ("f32", 4, 2, 128, 20, (128, 0, 0)),
    ("f32", 2, 2, 64, 8, (256, 0, 0)),
]


@pytest.mark.parametrize("dtype,H,H_kv,D,N,plan", CASES, ids=lambda v: "-".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_what_a_workspace_held_before_does_not_matter(spec, dtype, H, H_kv, D, N, plan):
    P = [830, 3, 500, 17, 831, 64]
    cfg = wl.Config(93, "partials", dtype, B=6, H=H, D=D, P=830, N=N, tree="random_branching", H_kv=H_kv)
    inp = wl.make_attention_inputs(cfg, seed=31 + N, S_cap=900 + N)
    inp["prefix_len"] = torch.tensor(P, dtype=torch.int32)
    inp["tree_parent"][2, 3] = 4               # malformed, of several chunks and of one; the fifth request does not fit
    inp["tree_depth"][3, 2] += 1
    good = [0, 1, 5]
    ref, _, _ = _oracle_append_attention(inp, bsel=good)
    q, kn, vn = (_dev(inp[k][0]) for k in ("q", "k_new", "v_new"))
    par, dep = _dev(inp["tree_parent"]), _dev(inp["tree_depth"])

    def run(pl, ws):
        status = torch.zeros(6, dtype=torch.int32, device=DEV)
        out = spec.spec_tree_attention_append(q, kn, vn, _dev(inp["k_cache"][0]), _dev(inp["v_cache"][0]), par, dep, pl, workspace=ws,
                                              status=status, max_prefix_len=830, plan=plan)
        torch.cuda.synchronize()
        return out, status.cpu().tolist()

    d = spec.make_desc(q, _dev(inp["k_cache"][0]), 830, k_new=kn, plan=plan)
    need = spec.spec_tree_attention_workspace_bytes(d)
    assert need > 0
    pl = _dev(inp["prefix_len"])
    final = torch.tensor([float("nan"), -1.0], device=DEV).repeat((need + 7) // 8).view(torch.uint8)[:need].clone()
    other = torch.zeros(need, dtype=torch.uint8, device=DEV)
    run(pl.flip(0).contiguous(), other)
    first = None
    for ws in (torch.zeros(need, dtype=torch.uint8, device=DEV), torch.full((need,), 255, dtype=torch.uint8, device=DEV), final, other):
        out, status = run(pl, ws)
        assert status == [0, 0, orc.ST_BAD_TREE, orc.ST_BAD_TREE, orc.ST_CAPACITY, 0]
        assert (out[2:5].float() == 0).all()
        first = out if first is None else first
        assert torch.equal(out.view(torch.int16 if dtype == "bf16" else torch.int32), first.view(torch.int16 if dtype == "bf16" else torch.int32))
    _check_attention(first[good], ref, cfg.torch_dtype)
