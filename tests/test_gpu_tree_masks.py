"""Ancestor masks of trees whose nodes fill one 64-node half, or two: chains through the border, nodes of the upper half that hang
on the lower one at once or by way of others, and malformed words in either half. Against the oracle, on the kernel for more
than four query tiles (D = 128), the eight-wavefront one (D = 64), up to 64 nodes the one for fewer queries, and up to 16 the
few-query kernel, whose tail wavefront reads the words by groups of four, which end with the tree above eight nodes."""
import numpy as np
import pytest
import torch

from oracle import spec_oracle as orc
from paper_2305_09781_amd import workloads as wl
from test_gpu_parity import DEV, _check_attention, _oracle_append_attention, _run_append_attention

pytestmark = pytest.mark.gpu


def _trees(N, rng):
    v = np.arange(N)
    return np.stack([
        v - 1,                                                                    # a chain
        np.where(v == 0, -1, np.where(v < 64, 0, np.maximum(v - 64, 1))),         # upper nodes below one lower node each
        np.where(v == 0, -1, np.where(v <= 64, (v - 1) // 2, v - 1)),             # upper chain hanging on a lower node
        np.where(v == 0, -1, np.maximum(v - 3, 0)),                               # three chains through the border
        np.array([-1] + [int(rng.integers(0, u)) for u in range(1, N)]),
        np.where(v == 0, -1, (v - 1) // 3),
    ]).astype(np.int32)


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("N", [1, 3, 4, 5, 8, 9, 10, 11, 12, 13, 14, 15, 16, 33, 63, 64, 65, 66, 96, 127, 128])
def test_masks_of_either_half(spec, N, D):
    rng = np.random.default_rng(N + D)
    trees = _trees(N, rng)
    B = len(trees)
    inp = wl.make_attention_inputs(wl.Config(97, "masks", "bf16", B=B, H=2, D=D, P=(20, 90), N=N, tree="random_parent"), seed=N + D)
    inp["tree_parent"] = torch.from_numpy(trees)
    inp["tree_depth"] = torch.from_numpy(np.stack([wl.depth_of(p) for p in trees]).astype(np.int32))
    for p, d in zip(inp["tree_parent"].numpy(), inp["tree_depth"].numpy()):
        assert orc.tree_status(p, d) == 0
    status = torch.zeros(B, dtype=torch.int32, device=DEV)
    out, _, _ = _run_append_attention(spec, inp, status=status, fused=True)
    ref, _, _ = _oracle_append_attention(inp)
    _check_attention(out, ref, torch.bfloat16)
    assert (status == 0).all()

    if N < 8:
        return
    bad = {k: (x.clone() if isinstance(x, torch.Tensor) else x) for k, x in inp.items()}
    bad["tree_parent"][0, 0] = 0                      # a root with a parent
    bad["tree_parent"][1, N - 1] = N - 1              # its own parent
    bad["tree_depth"][2, N // 2] += 1
    bad["tree_depth"][3, N - 1] = 0
    bad["tree_parent"][5, min(N - 1, 64)] = 1 << 30
    status.zero_()
    got, _, _ = _run_append_attention(spec, bad, status=status, fused=True)
    assert (status.cpu().numpy() == np.array([orc.ST_BAD_TREE] * 4 + [0, orc.ST_BAD_TREE])).all()
    assert (got[[0, 1, 2, 3, 5]] == 0).all() and torch.equal(got[4], out[4])
