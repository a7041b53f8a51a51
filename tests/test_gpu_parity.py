"""GPU-vs-oracle parity through the C ABI (needs an MI355X: `pytest -m gpu`).

Bars: attention max-abs 1e-5 for float32 inputs, |g-o| <= 2e-2 + 1e-2*|o| for bf16 inputs (oracle in
float64, not rounded); append, commit, verification decisions, paths and tokens bit-exact.
"""
import ctypes
import dataclasses

import numpy as np
import pytest
import torch

from oracle import spec_oracle as orc
from oracle import vetting
from paper_2305_09781_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _dev(x):
    if isinstance(x, np.ndarray):
        x = torch.from_numpy(np.ascontiguousarray(x))
    return x.to(DEV)


def _f64(t):
    return t.double().numpy()


def _bits(t):
    """Raw element bits as integers (bit-exact comparison of copies)."""
    t = t.cpu().contiguous()
    return t.view(torch.int16 if t.element_size() == 2 else torch.int32).numpy()


def _check_attention(out_gpu, ref64, dtype):
    g = out_gpu.double().cpu().numpy()
    err = np.abs(g - ref64)
    if dtype == torch.float32:
        assert err.max() <= 1e-5, f"max abs err {err.max():.3e}"
    else:
        bound = 2e-2 + 1e-2 * np.abs(ref64)
        worst = (err - bound).max()
        assert worst <= 0, f"bf16 tolerance exceeded by {worst:.3e} (max abs err {err.max():.3e})"
    return float(err.max())


_PLAN = [0, 0, 0]   # launch-plan hints the helpers below put into the descriptor: chunk keys, balanced workgroups, heads


class _plan_hint:
    """Sets one of the descriptor's launch-plan hints for the calls made inside the block."""

    def __init__(self, slot, n):
        self.slot, self.n = slot, n

    def __enter__(self):
        self.old = _PLAN[self.slot]
        _PLAN[self.slot] = int(self.n) if self.n else 0

    def __exit__(self, *a):
        _PLAN[self.slot] = self.old


def _plan():
    return tuple(_PLAN)


def _chunk_keys(n):
    """Forces the number of keys per workgroup so that small inputs span several chunks."""
    return _plan_hint(0, n)


def _balanced_wgs(n):
    """Forces the balanced plan on small inputs: pairs cut into n chunks in all, or left whole if there are not many fewer pairs
    than n (the few-query kernel then takes n equal contiguous shares of all tiles)."""
    return _plan_hint(1, n)


def _heads_per_wg(n):
    """Forces the number of consecutive heads one workgroup of the eight-wavefront shape serves."""
    return _plan_hint(2, n)


def _run_append_attention(spec, inp, layer=0, status=None, fused=False):
    """append + attention on the GPU for one layer of `inp` (two calls, or the fused entry point);
    returns (out, k_cache, v_cache) device tensors."""
    kc, vc = _dev(inp["k_cache"][layer]), _dev(inp["v_cache"][layer])
    pl = _dev(inp["prefix_len"])
    mp = min(int(inp["prefix_len"].max()), kc.shape[2] - inp["q"][layer].shape[1])
    kn, vn = _dev(inp["k_new"][layer]), _dev(inp["v_new"][layer])
    if fused:
        out = spec.spec_tree_attention_append(_dev(inp["q"][layer]), kn, vn, kc, vc, _dev(inp["tree_parent"]),
                                              _dev(inp["tree_depth"]), pl, status=status, max_prefix_len=mp, plan=_plan())
    else:
        spec.spec_kv_append(kn, vn, kc, vc, pl, status=status)
        out = spec.spec_tree_attention(_dev(inp["q"][layer]), kc, vc, _dev(inp["tree_parent"]), _dev(inp["tree_depth"]),
                                       pl, status=status, max_prefix_len=mp, plan=_plan())
    torch.cuda.synchronize()
    return out, kc, vc


def _oracle_append_attention(inp, layer=0, bsel=None, hsel=None):
    """Oracle on a (request, head) subset; caches are converted to float64 for the subset only."""
    bsel = list(range(inp["q"][layer].shape[0])) if bsel is None else bsel
    hsel = list(range(inp["q"][layer].shape[2])) if hsel is None else hsel
    if inp["k_cache"][layer].shape[1] != inp["q"][layer].shape[2]:
        assert hsel == list(range(inp["q"][layer].shape[2])), "head subsets are for multi-head inputs"
        ksel = list(range(inp["k_cache"][layer].shape[1]))
    else:
        ksel = hsel
    kc = _f64(inp["k_cache"][layer][bsel][:, ksel])
    vc = _f64(inp["v_cache"][layer][bsel][:, ksel])
    q = _f64(inp["q"][layer][bsel][:, :, hsel])
    kn = _f64(inp["k_new"][layer][bsel][:, :, ksel])
    vn = _f64(inp["v_new"][layer][bsel][:, :, ksel])
    pl = inp["prefix_len"].numpy()[bsel]
    st = orc.kv_append(kc, vc, kn, vn, pl)
    assert (st == 0).all()
    return orc.tree_attention(q, kc, vc, inp["tree_parent"].numpy()[bsel], pl), kc, vc


# ------------------------------------------------------------------------------------------------
# attention + append
# ------------------------------------------------------------------------------------------------

def test_config1_fp32_attention_and_append(spec):
    cfg = wl.CONFIGS[1]
    inp = wl.make_attention_inputs(cfg)
    for chunk in (0, 32, 64):
        with _chunk_keys(chunk):
            out, kc, vc = _run_append_attention(spec, inp, fused=(chunk == 32))
        ref, kco, vco = _oracle_append_attention(inp)
        _check_attention(out, ref, torch.float32)
        assert np.array_equal(kc.cpu().numpy().astype(np.float64), kco)
        assert np.array_equal(vc.cpu().numpy().astype(np.float64), vco)


SMALL = [
    # dtype, B, H, D, (P lo, hi), N, tree, forced chunk
    ("bf16", 2, 3, 128, (70, 200), 16, "expansion", 64),
    ("bf16", 2, 2, 128, (0, 5), 16, "random_parent", 0),
    ("bf16", 3, 2, 128, (33, 97), 7, "random_parent", 32),
    ("bf16", 2, 2, 128, (130, 300), 32, "random_branching", 96),
    ("bf16", 2, 2, 128, (130, 300), 17, "random_branching", 0),
    ("bf16", 2, 2, 64, (0, 300), 25, "random_parent", 64),
    ("bf16", 2, 2, 128, (130, 300), 33, "random_branching", 128),
    ("bf16", 1, 2, 128, (250, 250), 64, "random_branching", 64),
    ("bf16", 2, 2, 128, (100, 260), 100, "random_branching", 160),
    ("bf16", 1, 2, 128, (190, 190), 128, "random_branching", 0),
    ("bf16", 2, 3, 64, (60, 220), 16, "random_parent", 64),
    ("bf16", 2, 2, 64, (60, 220), 50, "random_branching", 96),
    ("f32", 2, 2, 128, (40, 150), 16, "random_parent", 64),
    ("f32", 1, 2, 64, (100, 100), 128, "random_branching", 96),
    ("f32", 2, 2, 128, (0, 3), 1, "random_parent", 0),
    ("bf16", 2, 2, 128, (0, 70), 1, "random_parent", 32),
]


@pytest.mark.parametrize("case", SMALL, ids=[f"{c[0]}-B{c[1]}H{c[2]}D{c[3]}P{c[4][0]}-{c[4][1]}N{c[5]}-{c[6]}-ck{c[7]}" for c in SMALL])
def test_small_shapes_attention_and_append(spec, case):
    dtype, B, H, D, P, N, tree, chunk = case
    cfg = wl.Config(90, "small", dtype, B=B, H=H, D=D, P=P if P[0] != P[1] else P[0], N=N, tree=tree,
                    widths=wl.EXPANSION_EVAL * 2)
    inp = wl.make_attention_inputs(cfg, seed=1000 + N + D + B, S_cap=P[1] + N + 5)
    ref, kco, vco = _oracle_append_attention(inp)
    for fused in (False, True):
        with _chunk_keys(chunk):
            out, kc, vc = _run_append_attention(spec, inp, fused=fused)
        _check_attention(out, ref, cfg.torch_dtype)
        # append is a bit copy: compare the whole cache (float64 conversion of either dtype is exact)
        assert np.array_equal(kc.double().cpu().numpy(), kco) and np.array_equal(vc.double().cpu().numpy(), vco), fused


def _shaped_tree(kind, N):
    """Extremes of the topology-aware mask (Section 4.2): a chain (every node sees all nodes before it), a star
    (a node sees the root and itself), and a comb (a chain of every 8th node, seven leaves hanging off each)."""
    par = np.full(N, -1, dtype=np.int32)
    for i in range(1, N):
        par[i] = {"chain": i - 1, "star": 0, "comb": (i - 8 if i % 8 == 0 else i - i % 8)}[kind]
    par[0] = -1
    return par


@pytest.mark.parametrize("kind", ["chain", "star", "comb"])
@pytest.mark.parametrize("N,P", [(16, 45), (48, 0), (64, 97), (96, 64), (128, 33), (128, 160), (65, 31)])
def test_extreme_tree_shapes(spec, kind, N, P):
    """Chains, stars and combs on every bf16 kernel, with prefixes that end inside a key stage: the masks of whole
    stages are all-visible, all-hidden or mixed, and the wavefronts that may skip a stage must skip exactly those."""
    cfg = wl.Config(91, "shaped", "bf16", B=2, H=2, D=128, P=P, N=N, tree="random_parent")
    inp = wl.make_attention_inputs(cfg, seed=77 + N + P, S_cap=P + N + 3)
    par = _shaped_tree(kind, N)
    inp["tree_parent"] = torch.from_numpy(np.stack([par, par]))
    inp["tree_depth"] = torch.from_numpy(np.stack([wl.depth_of(par), wl.depth_of(par)]).astype(np.int32))
    ref, kco, vco = _oracle_append_attention(inp)
    for fused in (False, True):
        out, kc, vc = _run_append_attention(spec, inp, fused=fused)
        _check_attention(out, ref, cfg.torch_dtype)
        assert np.array_equal(kc.double().cpu().numpy(), kco) and np.array_equal(vc.double().cpu().numpy(), vco), fused


@pytest.mark.parametrize("case", [("bf16", 3, 4, 128, (30, 200), 16, "expansion"), ("bf16", 2, 3, 64, (0, 90), 40, "random_branching"),
                                  ("f32", 2, 2, 64, (5, 60), 9, "random_parent"), ("f32", 1, 2, 128, (100, 100), 128, "random_branching")])
def test_kv_append_with_rotary_embedding(spec, case):
    """K rotated at position prefix_len + depth on the way into the cache: within one unit in the last place
    of the storage type of the float64 oracle (the kernel rotates in float32), V a bit copy."""
    dtype, B, H, D, P, N, tree = case
    cfg = wl.Config(96, "rope", dtype, B=B, H=H, D=D, P=P if P[0] != P[1] else P[0], N=N, tree=tree,
                    widths=wl.EXPANSION_EVAL * 2)
    inp = wl.make_attention_inputs(cfg, seed=300 + N, S_cap=P[1] + N + 2)
    cos, sin = wl.make_rope_tables(P[1] + N + 2, D)
    kco, vco = _f64(inp["k_cache"][0]), _f64(inp["v_cache"][0])
    st_ref = orc.kv_append_rope(kco, vco, _f64(inp["k_new"][0]), _f64(inp["v_new"][0]), inp["prefix_len"].numpy(),
                                inp["tree_depth"].numpy(), cos.numpy(), sin.numpy(), dtype)
    assert (st_ref == 0).all()
    kc, vc = _dev(inp["k_cache"][0]), _dev(inp["v_cache"][0])
    status = torch.zeros(B, dtype=torch.int32, device=DEV)
    spec.spec_kv_append_rope(_dev(inp["k_new"][0]), _dev(inp["v_new"][0]), kc, vc, _dev(inp["tree_depth"]),
                             _dev(inp["prefix_len"]), _dev(cos), _dev(sin), status=status)
    torch.cuda.synchronize()
    assert (status.cpu().numpy() == 0).all()
    assert np.array_equal(vc.double().cpu().numpy(), vco)
    got = kc.double().cpu().numpy()
    ulp = 2.0 ** -7 if dtype == "bf16" else 2.0 ** -21      # one unit in the last place, relative, at worst
    assert (np.abs(got - kco) <= ulp * np.abs(kco) + 1e-6).all()   # + float32 cancellation noise of x1 cos - x2 sin
    if dtype == "bf16":
        assert (got != kco).mean() < 0.02                   # flips of the last bit are rare
    # tables too short for one request: that request is untouched and flagged, the others are done
    short = int(inp["prefix_len"].max())
    kc2 = _dev(inp["k_cache"][0])
    status.zero_()
    spec.spec_kv_append_rope(_dev(inp["k_new"][0]), _dev(inp["v_new"][0]), kc2, _dev(inp["v_cache"][0]), _dev(inp["tree_depth"]),
                             _dev(inp["prefix_len"]), _dev(cos[:short].contiguous()), _dev(sin[:short].contiguous()), status=status)
    torch.cuda.synchronize()
    kref = _f64(inp["k_cache"][0])
    st2 = orc.kv_append_rope(kref, _f64(inp["v_cache"][0]), _f64(inp["k_new"][0]), _f64(inp["v_new"][0]),
                             inp["prefix_len"].numpy(), inp["tree_depth"].numpy(), cos[:short].numpy(), sin[:short].numpy(), dtype)
    assert np.array_equal(status.cpu().numpy(), st2) and (st2 != 0).any()
    for b in np.nonzero(st2)[0]:
        assert np.array_equal(_bits(kc2[b]), _bits(inp["k_cache"][0][b]))


@pytest.mark.parametrize("case", [("bf16", 3, 8, 2, 128, (30, 200), 16, "expansion"), ("bf16", 2, 3, 3, 64, (0, 90), 40, "random_branching"),
                                  ("f32", 2, 4, 2, 64, (5, 60), 9, "random_parent"), ("f32", 1, 2, 2, 128, (100, 100), 128, "random_branching")])
def test_q_and_k_rotary_embedding_in_one_launch(spec, case):
    """spec_qk_rope_append: the cache as after spec_kv_append_rope (bit for bit: the same arithmetic), q rotated
    in place within one unit in the last place of the float64 oracle, skipped requests untouched on both
    sides, and tree attention on the rotated operands within the attention bar of the oracle on the same bits."""
    dtype, B, H, H_kv, D, P, N, tree = case
    cfg = wl.Config(96, "ropeq", dtype, B=B, H=H, H_kv=H_kv, D=D, P=P if P[0] != P[1] else P[0], N=N, tree=tree,
                    widths=wl.EXPANSION_EVAL * 2)
    S = P[1] + N + 2
    inp = wl.make_attention_inputs(cfg, seed=400 + N, S_cap=S)
    cos, sin = wl.make_rope_tables(S, D)
    pl, dep, par = inp["prefix_len"].numpy(), inp["tree_depth"].numpy(), inp["tree_parent"].numpy()
    kco, vco = _f64(inp["k_cache"][0]), _f64(inp["v_cache"][0])
    orc.kv_append_rope(kco, vco, _f64(inp["k_new"][0]), _f64(inp["v_new"][0]), pl, dep, cos.numpy(), sin.numpy(), dtype)
    q_ref, st_ref = orc.rope_queries(_f64(inp["q"][0]), pl, dep, cos.numpy(), sin.numpy(), S, dtype)
    assert (st_ref == 0).all()
    # the key side alone, for the bit comparison
    kc1, vc1 = _dev(inp["k_cache"][0]), _dev(inp["v_cache"][0])
    spec.spec_kv_append_rope(_dev(inp["k_new"][0]), _dev(inp["v_new"][0]), kc1, vc1, _dev(inp["tree_depth"]),
                             _dev(inp["prefix_len"]), _dev(cos), _dev(sin))
    q, kc, vc = _dev(inp["q"][0]), _dev(inp["k_cache"][0]), _dev(inp["v_cache"][0])
    status = torch.zeros(B, dtype=torch.int32, device=DEV)
    spec.spec_qk_rope_append(q, _dev(inp["k_new"][0]), _dev(inp["v_new"][0]), kc, vc, _dev(inp["tree_depth"]),
                             _dev(inp["prefix_len"]), _dev(cos), _dev(sin), status=status)
    torch.cuda.synchronize()
    assert (status.cpu().numpy() == 0).all()
    assert np.array_equal(_bits(kc), _bits(kc1)) and np.array_equal(_bits(vc), _bits(vc1))
    got = q.double().cpu().numpy()
    ulp = 2.0 ** -7 if dtype == "bf16" else 2.0 ** -21
    assert (np.abs(got - q_ref) <= ulp * np.abs(q_ref) + 1e-6).all()
    if dtype == "bf16":
        assert (got != q_ref).mean() < 0.02
    # attention on what the launch left behind against the oracle on its own rotated operands
    out = torch.empty_like(q)
    spec.spec_tree_attention(q, kc, vc, _dev(inp["tree_parent"]), _dev(inp["tree_depth"]), _dev(inp["prefix_len"]), out)
    torch.cuda.synchronize()
    # (q and the cache were compared with the oracle's rotation above, to one unit in the last place; the
    # attention is then held to its usual bar on the operands the launch left in memory)
    want = orc.tree_attention(got, kc.double().cpu().numpy(), vc.double().cpu().numpy(), par, pl)
    _check_attention(out, want, cfg.torch_dtype)
    # tables too short for one request: its q and its cache rows stay as they were, it is flagged
    short = int(pl.max())
    q2, kc2 = _dev(inp["q"][0]), _dev(inp["k_cache"][0])
    status.zero_()
    spec.spec_qk_rope_append(q2, _dev(inp["k_new"][0]), _dev(inp["v_new"][0]), kc2, _dev(inp["v_cache"][0]),
                             _dev(inp["tree_depth"]), _dev(inp["prefix_len"]), _dev(cos[:short].contiguous()),
                             _dev(sin[:short].contiguous()), status=status)
    torch.cuda.synchronize()
    _, st2 = orc.rope_queries(_f64(inp["q"][0]), pl, dep, cos[:short].numpy(), sin[:short].numpy(), S, dtype)
    assert np.array_equal(status.cpu().numpy(), st2) and (st2 != 0).any()
    for b in range(B):
        if st2[b]:
            assert np.array_equal(_bits(q2[b]), _bits(inp["q"][0][b])) and np.array_equal(_bits(kc2[b]), _bits(inp["k_cache"][0][b]))
        else:
            assert np.array_equal(_bits(q2[b]), _bits(q[b]))


def test_qk_rope_append_rejects_bad_arguments(spec):
    cfg = wl.Config(96, "ropeq", "bf16", B=1, H=2, D=64, P=10, N=4, tree="random_parent")
    inp = wl.make_attention_inputs(cfg, seed=1, S_cap=32)
    cos, sin = wl.make_rope_tables(32, 64)
    args = [_dev(inp[k][0]) for k in ("q", "k_new", "v_new", "k_cache", "v_cache")] + [_dev(inp["tree_depth"]), _dev(inp["prefix_len"])]
    with pytest.raises(ValueError):
        spec.spec_qk_rope_append(*args, _dev(cos[:, :16].contiguous()), _dev(sin[:, :16].contiguous()))
    d = spec.make_desc(args[0], args[3], k_new=args[1])
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    cs, sn = _dev(cos), _dev(sin)
    rc = spec.load().spec_qk_rope_append(ctypes.byref(d), None, *[ptr(t) for t in args[1:]], ptr(cs), ptr(sn), 32, None, None)
    assert rc != 0                                                  # q is not optional here


@pytest.mark.parametrize("case", [(1, 2, 128, 131072, 16, "expansion"), (1, 1, 128, 200000, 100, "random_branching"),
                                  (2, 1, 64, (70000, 90001), 40, "random_branching"), (1, 2, 128, 131072, 128, "random_branching")],
                         ids=lambda c: f"B{c[0]}H{c[1]}D{c[2]}P{c[3]}N{c[4]}")
def test_very_long_prefixes(spec, case):
    """Prefixes of a hundred thousand keys and more (key ranges cut into hundreds of chunks, float32 partials and
    the combine step; row offsets near the 32-bit range for one head): every output against the oracle, the
    appended rows bit for bit."""
    B, H, D, P, N, tree = case
    cfg = wl.Config(89, "long", "bf16", B=B, H=H, D=D, P=P, N=N, tree=tree, widths=wl.EXPANSION_EVAL * 16)
    inp = wl.make_attention_inputs(cfg, seed=5 + N)
    ref, kco, vco = _oracle_append_attention(inp)
    for fused in (True, False):
        out, kc, vc = _run_append_attention(spec, inp, fused=fused)
        _check_attention(out, ref, torch.bfloat16)
        pl = inp["prefix_len"].numpy()
        for b in range(B):
            rows = slice(int(pl[b]), int(pl[b]) + N)
            assert np.array_equal(kc[b, :, rows].double().cpu().numpy(), kco[b, :, rows])
            assert np.array_equal(vc[b, :, rows].double().cpu().numpy(), vco[b, :, rows])


GROUPED = [
    # dtype, B, H, H_kv, D, (P lo, hi), N, tree, forced chunk, balanced workgroups
    ("bf16", 2, 4, 2, 128, (70, 300), 16, "expansion", 0, 0),        # 2 query tiles per K/V head
    ("bf16", 2, 8, 2, 128, (70, 300), 16, "random_parent", 64, 0),   # 4 tiles
    ("bf16", 2, 8, 1, 128, (40, 200), 16, "expansion", 0, 0),        # 8 tiles, one K/V head
    ("bf16", 2, 8, 1, 64, (40, 200), 7, "random_parent", 0, 5),      # 8 partly filled tiles, balanced plan
    ("bf16", 3, 6, 3, 128, (0, 130), 40, "random_branching", 96, 0), # 2 heads x 3 tiles
    ("bf16", 2, 4, 2, 64, (100, 500), 33, "random_branching", 0, 7),
    ("bf16", 1, 16, 2, 128, (600, 600), 1, "random_parent", 0, 0),   # decode-shaped: one node, 8 heads per group
    ("f32", 2, 6, 2, 64, (30, 120), 12, "random_parent", 64, 0),
    # more than 8 query tiles per K/V head: several workgroups (query groups) per pair
    ("bf16", 2, 16, 1, 128, (40, 300), 16, "expansion", 0, 0),        # 16 heads, one K/V head: 2 query groups of 8
    ("bf16", 2, 12, 2, 128, (40, 300), 33, "random_branching", 64, 0),  # 3 tiles per head: 2 heads per workgroup, 3 groups
    ("bf16", 1, 71, 1, 64, (100, 100), 16, "expansion", 0, 0),       # multi-query attention, 71 heads: 9 groups, last one short
    ("bf16", 2, 20, 2, 64, (30, 500), 16, "random_parent", 0, 9),    # query groups under the balanced plan, pairs whole
    ("bf16", 2, 20, 2, 64, (30, 500), 16, "random_parent", 0, 40),   # ... and cut
    ("bf16", 1, 6, 1, 128, (64, 64), 128, "random_branching", 0, 4), # 8 tiles per head: one head per workgroup
    ("bf16", 1, 6, 1, 128, (64, 64), 128, "random_branching", 0, 18),
]


@pytest.mark.parametrize("case", GROUPED, ids=[f"{c[0]}-B{c[1]}H{c[2]}kv{c[3]}D{c[4]}N{c[6]}-ck{c[8]}-wg{c[9]}" for c in GROUPED])
def test_grouped_query_heads(spec, case):
    """Fewer K/V heads than query heads (an extension next to the path): the query heads of a group share
    one K/V stream; append, attention (fused and not) and status handling as for multi-head inputs."""
    dtype, B, H, H_kv, D, P, N, tree, chunk, wgs = case
    cfg = wl.Config(98, "gqa", dtype, B=B, H=H, D=D, P=P if P[0] != P[1] else P[0], N=N, tree=tree,
                    widths=wl.EXPANSION_EVAL * 2, H_kv=H_kv)
    inp = wl.make_attention_inputs(cfg, seed=3000 + N + H, S_cap=P[1] + N + 5)
    ref, kco, vco = _oracle_append_attention(inp)
    for fused in (False, True):
        with _chunk_keys(chunk), _balanced_wgs(wgs):
            out, kc, vc = _run_append_attention(spec, inp, fused=fused)
        _check_attention(out, ref, cfg.torch_dtype)
        assert np.array_equal(kc.double().cpu().numpy(), kco) and np.array_equal(vc.double().cpu().numpy(), vco), fused
    # malformed tree / request that does not fit: zeros for every query head of the group
    inp["tree_parent"][0, N - 1] = N + 3 if N > 1 else 0
    inp["prefix_len"][B - 1] = inp["k_cache"][0].shape[2] - N + 1
    status = torch.zeros(B, dtype=torch.int32, device=DEV)
    with _chunk_keys(chunk), _balanced_wgs(wgs):
        out, _, _ = _run_append_attention(spec, inp, status=status, fused=True)
    st = status.cpu().numpy()
    assert st[B - 1] == orc.ST_CAPACITY and (out[B - 1].float() == 0).all()
    if B > 1:
        assert st[0] == orc.ST_BAD_TREE and (out[0].float() == 0).all()


def test_new_rows_in_their_own_layout(spec):
    """Multi-head inputs whose k_new / v_new are not laid out like q (views into wider tensors): the
    descriptor carries their strides and the fused call still appends and attends correctly."""
    cfg = wl.Config(99, "strides", "bf16", B=2, H=3, D=128, P=(50, 260), N=16, tree="expansion", widths=wl.EXPANSION_EVAL * 2)
    inp = wl.make_attention_inputs(cfg, seed=17, S_cap=260 + 16 + 3)
    ref, kco, vco = _oracle_append_attention(inp)
    wide_k = torch.zeros((cfg.B, cfg.N, cfg.H, 2 * cfg.D), dtype=torch.bfloat16, device=DEV)
    wide_v = torch.zeros_like(wide_k)
    kn, vn = wide_k[..., :cfg.D], wide_v[..., :cfg.D]
    kn.copy_(inp["k_new"][0]); vn.copy_(inp["v_new"][0])
    assert kn.stride() != _dev(inp["q"][0]).stride()
    for wgs in (0, 3):
        kc, vc = _dev(inp["k_cache"][0]), _dev(inp["v_cache"][0])
        with _balanced_wgs(wgs):
            out = spec.spec_tree_attention_append(_dev(inp["q"][0]), kn, vn, kc, vc, _dev(inp["tree_parent"]),
                                                  _dev(inp["tree_depth"]), _dev(inp["prefix_len"]), max_prefix_len=260, plan=_plan())
        torch.cuda.synchronize()
        _check_attention(out, ref, torch.bfloat16)
        assert np.array_equal(kc.double().cpu().numpy(), kco) and np.array_equal(vc.double().cpu().numpy(), vco)
    kc, vc = _dev(inp["k_cache"][0]), _dev(inp["v_cache"][0])
    spec.spec_kv_append(kn, vn, kc, vc, _dev(inp["prefix_len"]))
    torch.cuda.synchronize()
    assert np.array_equal(kc.double().cpu().numpy(), kco) and np.array_equal(vc.double().cpu().numpy(), vco)


@pytest.mark.parametrize("seed", range(32))
def test_randomised_shapes_and_plans(spec, seed):
    """Random small shapes (heads, grouped heads, head dim, tree size, ragged prefixes down to zero, cache
    capacity exactly prefix + N) under a random launch plan, fused or not: parity and bit-exact append."""
    rng = np.random.default_rng(5000 + seed)
    dtype = "bf16" if rng.random() < 0.8 else "f32"
    D = int(rng.choice([64, 128]))
    H_kv = int(rng.integers(1, 4))
    N = int(rng.choice([1, 2, 5, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 97, 127, 128]))
    tiles_per_head = (N + 15) // 16
    group = int(rng.integers(1, 13)) if rng.random() < 0.3 else int(rng.integers(1, 4))
    H = H_kv * group
    B = int(rng.integers(1, 5))
    hi = int(rng.choice([0, 3, 40, 130, 400]))
    lo = int(rng.integers(0, hi + 1))
    tree = str(rng.choice(["random_parent", "random_branching", "expansion"]))
    cfg = wl.Config(90, "rand", dtype, B=B, H=H, D=D, P=(lo, hi) if lo != hi else hi, N=N, tree=tree,
                    widths=wl.EXPANSION_EVAL * 16, H_kv=H_kv)
    inp = wl.make_attention_inputs(cfg, seed=6000 + seed, S_cap=hi + N + int(rng.choice([0, 1, 7])))
    plan = int(rng.integers(0, 3))
    chunk = int(rng.choice([32, 64, 96, 160])) if plan == 1 else 0
    wgs = int(rng.integers(1, 12)) if plan == 2 and dtype == "bf16" else 0
    fused = bool(rng.integers(0, 2))
    ref, kco, vco = _oracle_append_attention(inp)
    with _chunk_keys(chunk), _balanced_wgs(wgs):
        out, kc, vc = _run_append_attention(spec, inp, fused=fused)
    _check_attention(out, ref, cfg.torch_dtype)
    assert np.array_equal(kc.double().cpu().numpy(), kco) and np.array_equal(vc.double().cpu().numpy(), vco)


@pytest.mark.parametrize("case", [
    # B, H, H_kv, D, (P lo, hi), N, K/V heads per workgroup, fused
    (2, 5, 5, 128, (100, 300), 128, 2, True),     # uneven: the last workgroup of a request serves one head
    (2, 6, 6, 128, (100, 300), 97, 3, False),
    (3, 4, 4, 64, (0, 20), 80, 2, True),          # two tiles per head, both masked
    (2, 4, 4, 128, (0, 0), 65, 4, True),          # empty prefix
    (1, 8, 8, 128, (500, 500), 128, 8, True),
    (2, 3, 3, 128, (64, 200), 100, 7, False),     # more heads per workgroup than heads
    (3, 24, 3, 128, (0, 48), 16, 2, True),        # grouped heads, 8 tiles per K/V head; one tile per head: the
    (3, 24, 3, 64, (0, 48), 13, 3, False),        # stream's second tile is the next head's first
    (2, 32, 4, 128, (30, 200), 16, 4, True),
], ids=lambda c: f"B{c[0]}H{c[1]}kv{c[2]}D{c[3]}P{c[4][0]}-{c[4][1]}N{c[5]}-nh{c[6]}-{'fused' if c[7] else 'two-calls'}")
def test_several_heads_per_workgroup(spec, case):
    """Wide trees on the eight-wavefront shape: a workgroup serves consecutive heads of a request as one stream
    of tiles. Forced on small inputs; parity, bit-exact append, and the defined results of flagged requests."""
    B, H, H_kv, D, P, N, nh, fused = case
    cfg = wl.Config(89, "heads", "bf16", B=B, H=H, D=D, P=P if P[0] != P[1] else P[0], N=N, tree="random_branching",
                    H_kv=H_kv)
    inp = wl.make_attention_inputs(cfg, seed=900 + N + nh, S_cap=P[1] + N + 3)
    ref, kco, vco = _oracle_append_attention(inp)
    with _heads_per_wg(nh):
        out, kc, vc = _run_append_attention(spec, inp, fused=fused)
        _check_attention(out, ref, torch.bfloat16)
        assert np.array_equal(kc.double().cpu().numpy(), kco) and np.array_equal(vc.double().cpu().numpy(), vco)
        # a malformed tree and a request that does not fit: zeros for every head, the others served
        if B >= 2:
            bad = dict(inp)
            bad["tree_parent"] = inp["tree_parent"].clone()
            bad["tree_parent"][0, N - 1] = N - 1
            bad["prefix_len"] = inp["prefix_len"].clone()
            bad["prefix_len"][1] = inp["k_cache"][0].shape[2] - N + 1
            status = torch.zeros(B, dtype=torch.int32, device=DEV)
            out2, kc2, _ = _run_append_attention(spec, bad, status=status, fused=fused)
            st = status.cpu().numpy()
            assert st[0] & orc.ST_BAD_TREE and st[1] & orc.ST_CAPACITY
            assert (out2[:2].float() == 0).all()
            assert np.array_equal(_bits(kc2[1]), _bits(inp["k_cache"][0][1]))
            if B > 2:
                _check_attention(out2[2:], ref[2:], torch.bfloat16)


@pytest.mark.parametrize("N,scale", [(16, 6.0), (40, 6.0), (128, 4.0), (16, 0.01), (64, 0.01)])
def test_peaked_and_flat_score_distributions(spec, N, scale):
    """Scores far outside the unit range (the running maximum moves by many powers of two between tiles,
    softmax weights underflow) and nearly constant scores: the online softmax stays within the bf16 bar."""
    cfg = wl.Config(89, "peaked", "bf16", B=2, H=2, D=128, P=(200, 700), N=N, tree="random_branching")
    inp = wl.make_attention_inputs(cfg, seed=71 + N, S_cap=700 + N)
    for name in ("q", "k_new", "k_cache"):
        inp[name][0] = (inp[name][0].float() * scale).to(torch.bfloat16)
    ref, kco, vco = _oracle_append_attention(inp)
    for wgs in (0, 5):
        with _balanced_wgs(wgs):
            out, kc, vc = _run_append_attention(spec, inp, fused=True)
        assert torch.isfinite(out.float()).all()
        _check_attention(out, ref, torch.bfloat16)


@pytest.mark.parametrize("N,dtype", [(16, "bf16"), (40, "bf16"), (8, "f32")])
def test_prefix_above_the_stated_maximum_is_flagged_not_truncated(spec, N, dtype):
    """max_prefix_len sizes the launch; a request whose prefix_len exceeds it must not be attended over a
    truncated key range: flagged SPEC_ST_CAPACITY, zeros, not appended; the others unaffected."""
    cfg = wl.Config(88, "hint", dtype, B=3, H=2, D=64, P=(50, 100), N=N, tree="random_parent")
    inp = wl.make_attention_inputs(cfg, seed=13, S_cap=400 + N)
    inp["prefix_len"][1] = 300                                    # fits the cache, exceeds the stated maximum
    for chunk, wgs in ((0, 0), (64, 0), (0, 4)):
        if dtype == "f32" and wgs:
            continue
        kc, vc = _dev(inp["k_cache"][0]), _dev(inp["v_cache"][0])
        status = torch.zeros(3, dtype=torch.int32, device=DEV)
        with _chunk_keys(chunk), _balanced_wgs(wgs):
            out = spec.spec_tree_attention_append(_dev(inp["q"][0]), _dev(inp["k_new"][0]), _dev(inp["v_new"][0]), kc, vc,
                                                  _dev(inp["tree_parent"]), _dev(inp["tree_depth"]), _dev(inp["prefix_len"]),
                                                  status=status, max_prefix_len=100, plan=_plan())
        torch.cuda.synchronize()
        assert status.cpu().tolist() == [0, orc.ST_CAPACITY, 0]
        assert (out[1].float() == 0).all() and np.array_equal(_bits(kc[1]), _bits(inp["k_cache"][0][1]))
        ref, _, _ = _oracle_append_attention(inp, bsel=[0, 2])
        _check_attention(out[[0, 2]], ref, cfg.torch_dtype)


BALANCED = [
    # B, H, D, (P lo, hi), N, tree, workgroups (wide kernels leave pairs whole at the small ones; cut pairs: test_gpu_cut_pairs.py)
    (3, 2, 128, (40, 300), 16, "expansion", 5),
    (3, 2, 128, (40, 300), 32, "random_branching", 7),
    (4, 3, 128, (0, 100), 7, "random_parent", 64),      # more workgroups than tiles: shares of one tile
    (2, 2, 64, (100, 400), 32, "random_branching", 3),
    (2, 2, 64, (100, 400), 16, "random_parent", 1),     # one workgroup walks every (request, head)
    (1, 2, 128, (1000, 1000), 16, "expansion", 16),
    (2, 2, 128, (100, 700), 17, "random_branching", 6),
    (2, 3, 128, (100, 500), 64, "random_branching", 7),
    (2, 2, 128, (60, 400), 100, "random_branching", 5),
    (1, 2, 64, (900, 900), 128, "random_branching", 9),
]


@pytest.mark.parametrize("case", BALANCED, ids=[f"B{c[0]}H{c[1]}D{c[2]}P{c[3][0]}-{c[3][1]}N{c[4]}-{c[5]}-wg{c[6]}" for c in BALANCED])
def test_balanced_plan_attention_and_append(spec, case):
    """The balanced plan of the bf16 kernels: contiguous shares of the few-query kernel that start and end inside a pair, cross
    pair and request boundaries, or are empty; chunks of one tile; whole pairs in more workgroups than were asked for."""
    B, H, D, P, N, tree, wgs = case
    cfg = wl.Config(92, "balanced", "bf16", B=B, H=H, D=D, P=P if P[0] != P[1] else P[0], N=N, tree=tree,
                    widths=wl.EXPANSION_EVAL * 2)
    inp = wl.make_attention_inputs(cfg, seed=2000 + N + D + B + wgs, S_cap=P[1] + N + 5)
    ref, kco, vco = _oracle_append_attention(inp)
    for fused in (False, True):
        with _balanced_wgs(wgs):
            out, kc, vc = _run_append_attention(spec, inp, fused=fused)
        _check_attention(out, ref, cfg.torch_dtype)
        assert np.array_equal(kc.double().cpu().numpy(), kco) and np.array_equal(vc.double().cpu().numpy(), vco), fused


@pytest.mark.parametrize("case", [(1, 4, 128, (700, 700), 16, "expansion"), (1, 3, 128, (1300, 1300), 40, "random_branching"),
                                  (2, 2, 128, (300, 1100), 64, "random_branching"), (1, 2, 64, (900, 900), 128, "random_branching"),
                                  (3, 2, 128, (0, 800), 16, "random_parent")])
def test_small_batches_take_the_chunked_plan_by_default(spec, case):
    """With fewer (request, head) pairs than compute units the plan itself (no override) cuts the key range
    into chunks of at least 256 keys and merges the partial results: the caller must bring a workspace, the
    result is the oracle's, and requests shorter than the stated maximum leave their trailing chunks empty."""
    B, H, D, P, N, tree = case
    cfg = wl.Config(94, "chunked", "bf16", B=B, H=H, D=D, P=P if P[0] != P[1] else P[0], N=N, tree=tree,
                    widths=wl.EXPANSION_EVAL * 2)
    inp = wl.make_attention_inputs(cfg, seed=2500 + N + B, S_cap=P[1] + N + 3)
    desc = spec.make_desc(_dev(inp["q"][0]), _dev(inp["k_cache"][0]), max_prefix_len=int(inp["prefix_len"].max()))
    assert spec.spec_tree_attention_workspace_bytes(desc) > 0
    ref, kco, vco = _oracle_append_attention(inp)
    for fused in (False, True):
        out, kc, vc = _run_append_attention(spec, inp, fused=fused)
        _check_attention(out, ref, cfg.torch_dtype)
        assert np.array_equal(kc.double().cpu().numpy(), kco) and np.array_equal(vc.double().cpu().numpy(), vco), fused


@pytest.mark.parametrize("fused", [False, True])
def test_config2_bf16_full(spec, fused):
    cfg = wl.CONFIGS[2]
    inp = wl.make_attention_inputs(cfg)
    out, kc, vc = _run_append_attention(spec, inp, fused=fused)
    ref, kco, vco = _oracle_append_attention(inp)
    _check_attention(out, ref, torch.bfloat16)
    assert np.array_equal(kc.double().cpu().numpy(), kco) and np.array_equal(vc.double().cpu().numpy(), vco)


@pytest.mark.parametrize("c,fused", [(3, True), (4, True), (4, False), (5, True)])
def test_large_configs_every_request_and_head(spec, c, fused):
    """Full-size launch (fused = the configuration the benchmark times) compared with the oracle on every
    (request, head) pair, every node and channel, and the whole cache bit for bit; the oracle runs request by
    request so that only one request's caches are in float64 at a time."""
    cfg = wl.CONFIGS[c]
    inp = wl.make_attention_inputs(cfg)
    status = torch.zeros(cfg.B, dtype=torch.int32, device=DEV)
    out, kc, vc = _run_append_attention(spec, inp, fused=fused, status=status)
    assert (status.cpu().numpy() == 0).all()
    out_h, kc_h, vc_h = out.cpu(), kc.cpu(), vc.cpu()
    worst = 0.0
    for b in range(cfg.B):
        ref, kco, vco = _oracle_append_attention(inp, bsel=[b])
        worst = max(worst, _check_attention(out_h[b:b + 1], ref, torch.bfloat16))
        assert np.array_equal(kc_h[b:b + 1].double().numpy(), kco), b
        assert np.array_equal(vc_h[b:b + 1].double().numpy(), vco), b
    print(f"config {c}: {cfg.B * cfg.H} (request, head) pairs compared, max abs err {worst:.3e}")


@pytest.mark.parametrize("N", [16, 40])
def test_attention_status_bits_and_noop(spec, N):
    """Malformed trees and requests that do not fit are flagged and produce zeros; others unaffected."""
    cfg = wl.Config(91, "bad", "bf16", B=4, H=2, D=128, P=(40, 90), N=N, tree="random_parent")
    plans = [(0, False, 0), (64, False, 0), (0, True, 0), (64, True, 0), (0, False, 5), (0, True, 3), (0, False, 24), (0, True, 24)]
    for chunk, fused, wgs in plans:
        inp = wl.make_attention_inputs(cfg, seed=5, S_cap=90 + N)
        inp["tree_parent"][1, 5] = 9            # parent after child
        inp["tree_depth"][2, 7] += 1            # depth inconsistent with parent
        inp["prefix_len"][3] = 90 + 1           # prefix + N > S_cap
        status = torch.zeros(cfg.B, dtype=torch.int32, device=DEV)
        with _chunk_keys(chunk), _balanced_wgs(wgs):
            out, kc, vc = _run_append_attention(spec, inp, status=status, fused=fused)
        st = status.cpu().numpy()
        assert st[0] == 0 and st[1] == orc.ST_BAD_TREE and st[2] == orc.ST_BAD_TREE and st[3] == orc.ST_CAPACITY
        assert (out[1:].float() == 0).all(), (chunk, fused, wgs)
        ref, _, _ = _oracle_append_attention(inp, bsel=[0])
        _check_attention(out[:1], ref, torch.bfloat16)
        assert orc.tree_status(inp["tree_parent"][1].numpy()) == orc.ST_BAD_TREE
        assert orc.tree_status(inp["tree_parent"][2].numpy(), inp["tree_depth"][2].numpy()) == orc.ST_BAD_TREE
        # the request that does not fit was not appended
        assert np.array_equal(_bits(kc[3]), _bits(inp["k_cache"][0][3]))


def test_host_side_errors(spec):
    cfg = wl.Config(92, "err", "bf16", B=1, H=2, D=128, P=20, N=16, tree="random_parent")
    inp = wl.make_attention_inputs(cfg, seed=1)
    q, kc, vc = _dev(inp["q"][0]), _dev(inp["k_cache"][0]), _dev(inp["v_cache"][0])
    par, dep, pl = _dev(inp["tree_parent"]), _dev(inp["tree_depth"]), _dev(inp["prefix_len"])
    d = spec.make_desc(q, kc)
    for field, val, code in (("D", 96, spec.ERR_UNSUPPORTED), ("N", 129, spec.ERR_UNSUPPORTED),
                             ("H_kv", 3, spec.ERR_UNSUPPORTED), ("max_prefix_len", 30, spec.ERR_CAPACITY),
                             ("q_stride_h", 100, spec.ERR_INVALID_ARG), ("dtype", 7, spec.ERR_UNSUPPORTED)):
        bad = spec.make_desc(q, kc)
        setattr(bad, field, val)
        with pytest.raises(spec.SpecError) as e:
            spec.spec_tree_attention(q, kc, vc, par, dep, pl, desc=bad)
        assert e.value.code == code, field
    with _chunk_keys(32):
        with pytest.raises(spec.SpecError) as e:
            spec.spec_tree_attention(q, kc, vc, par, dep, pl, workspace=torch.empty(256, dtype=torch.uint8, device=DEV),
                                     plan=_plan())
        assert e.value.code == spec.ERR_WORKSPACE


# ------------------------------------------------------------------------------------------------
# verification
# ------------------------------------------------------------------------------------------------

def _greedy_case(spec, cfg, seed=None, logits_dtype=torch.float32):
    inp = wl.make_verify_inputs(cfg, seed=seed, mode="greedy", logits_dtype=logits_dtype)
    path, ln, toks, am = spec.spec_verify_greedy(_dev(inp["logits"]), _dev(inp["tree_token"]), _dev(inp["tree_parent"]))
    torch.cuda.synchronize()
    lg = inp["logits"].float().numpy()
    rp, rl, rt, ra = orc.verify_greedy(lg, inp["tree_token"].numpy(), inp["tree_parent"].numpy())
    assert np.array_equal(am.cpu().numpy(), ra)
    assert np.array_equal(ln.cpu().numpy(), rl)
    assert np.array_equal(path.cpu().numpy(), rp) and np.array_equal(toks.cpu().numpy(), rt)
    return rl


@pytest.mark.parametrize("c", [1, 2, 3, 5])
def test_greedy_configs(spec, c):
    rl = _greedy_case(spec, wl.CONFIGS[c])
    assert rl.min() >= 1


def test_greedy_bf16_logits_ties_and_odd_vocab(spec):
    # bf16 logits tie often near the top (spacing 2^-4 at |x| ~ 8): lowest token id must win
    _greedy_case(spec, wl.CONFIGS[2], seed=77, logits_dtype=torch.bfloat16)
    for V in (1, 3, 63, 1001):
        cfg = wl.Config(93, "oddV", "f32", B=3, H=1, D=64, P=1, N=9, tree="random_parent", V=V)
        _greedy_case(spec, cfg, seed=V)


def test_greedy_bad_tree(spec):
    cfg = wl.Config(94, "badg", "f32", B=2, H=1, D=64, P=1, N=8, tree="random_parent", V=50)
    inp = wl.make_verify_inputs(cfg, mode="greedy")
    inp["tree_parent"][1, 3] = 3
    status = torch.zeros(2, dtype=torch.int32, device=DEV)
    path, ln, toks, am = spec.spec_verify_greedy(_dev(inp["logits"]), _dev(inp["tree_token"]), _dev(inp["tree_parent"]),
                                                 status=status)
    torch.cuda.synchronize()
    assert list(status.cpu().numpy()) == [0, orc.ST_BAD_TREE] and ln[1].item() == 0 and ln[0].item() >= 1
    assert (path[1] == -1).all()


def _stochastic_case(spec, cfg, seed=None, tau=1.2, temperature=1.0, logits_dtype=torch.float32):
    inp = wl.make_verify_inputs(cfg, seed=seed, mode="stochastic", tau=tau, logits_dtype=logits_dtype)
    lg = inp["logits"].float().numpy()
    args = (lg, inp["probs_ssm"].numpy(), inp["ssm_row"].numpy(), inp["tree_token"].numpy(), inp["tree_parent"].numpy())
    ua, uf, redraws = vetting.vet_uniforms(*args, inp["u_accept"].numpy(), inp["u_order"].numpy(), inp["u_final"].numpy(),
                                           inp["rng"], temperature=temperature)
    rp, rl, rt, rs = orc.verify_stochastic(*args, ua, inp["u_order"].numpy(), uf, temperature=temperature)
    status = torch.zeros(cfg.B, dtype=torch.int32, device=DEV)
    path, ln, toks = spec.spec_verify_stochastic(_dev(inp["logits"]), _dev(inp["probs_ssm"]), _dev(inp["ssm_row"]),
                                                 _dev(inp["tree_token"]), _dev(inp["tree_parent"]), _dev(ua),
                                                 _dev(inp["u_order"]), _dev(uf), temperature=temperature, status=status)
    torch.cuda.synchronize()
    assert np.array_equal(ln.cpu().numpy(), rl), (ln.cpu().numpy(), rl)
    assert np.array_equal(path.cpu().numpy(), rp) and np.array_equal(toks.cpu().numpy(), rt)
    assert np.array_equal(status.cpu().numpy(), rs)
    return rl, redraws


@pytest.mark.parametrize("c", [1, 2, 3])
def test_stochastic_configs(spec, c):
    rl, redraws = _stochastic_case(spec, wl.CONFIGS[c], tau=None if c == 1 else 1.2)
    print(f"config {c}: accepted lengths {rl.tolist()}, re-drawn requests {redraws}")


@pytest.mark.parametrize("seed", range(4))
def test_stochastic_many_rejections_and_temperature(spec, seed):
    """Drafts far from the LLM (many residual updates per node), wide trees, temperature != 1."""
    cfg = wl.Config(95, "rej", "f32", B=6, H=1, D=64, P=1, N=40, tree="random_branching", V=777, n_ssm=3)
    _stochastic_case(spec, cfg, seed=seed, tau=4.0, temperature=[1.0, 0.7, 1.5, 1.0][seed])
    cfg = wl.Config(96, "rej2", "f32", B=4, H=1, D=64, P=1, N=12, tree="random_parent", V=5, n_ssm=2)
    _stochastic_case(spec, cfg, seed=seed, tau=None)


def test_stochastic_bf16_logits(spec):
    _stochastic_case(spec, wl.CONFIGS[2], seed=31, logits_dtype=torch.bfloat16)


def _naive_case(spec, cfg, seed=None, temperature=1.0, logits_dtype=torch.float32, tau=1.2):
    """Naive sampling (Section 4.3) on the stochastic workload's trees (children sampled from the drafts)."""
    inp = wl.make_verify_inputs(cfg, seed=seed, mode="stochastic", tau=tau, logits_dtype=logits_dtype)
    lg = inp["logits"].float().numpy()
    us = inp["rng"].random((cfg.B, cfg.N), dtype=np.float32)
    us, redraws = vetting.vet_sample_uniforms(lg, us, inp["rng"], temperature=temperature)
    rp, rl, rt, rsamp = orc.verify_naive(lg, inp["tree_token"].numpy(), inp["tree_parent"].numpy(), us, temperature)
    status = torch.zeros(cfg.B, dtype=torch.int32, device=DEV)
    path, ln, toks, samp = spec.spec_verify_naive(_dev(inp["logits"]), _dev(inp["tree_token"]), _dev(inp["tree_parent"]),
                                                  _dev(torch.from_numpy(us)), temperature=temperature, status=status)
    torch.cuda.synchronize()
    assert np.array_equal(samp.cpu().numpy(), rsamp)          # every node's draw, visited or not
    assert np.array_equal(ln.cpu().numpy(), rl), (ln.cpu().numpy(), rl)
    assert np.array_equal(path.cpu().numpy(), rp) and np.array_equal(toks.cpu().numpy(), rt)
    assert (status.cpu().numpy() == 0).all()
    return rl, redraws


@pytest.mark.parametrize("c", [1, 2, 3])
def test_naive_sampling_configs(spec, c):
    rl, redraws = _naive_case(spec, wl.CONFIGS[c], tau=None if c == 1 else 1.2)
    print(f"config {c}: accepted lengths {rl.tolist()}, re-drawn uniforms {redraws}")


@pytest.mark.parametrize("seed", range(3))
def test_naive_sampling_odd_vocabulary_temperature_bf16(spec, seed):
    cfg = wl.Config(97, "ns", "f32", B=5, H=1, D=64, P=1, N=33, tree="random_branching", V=777, n_ssm=2)
    _naive_case(spec, cfg, seed=seed, temperature=[1.0, 0.6, 1.7][seed])
    cfg = wl.Config(98, "ns2", "f32", B=3, H=1, D=64, P=1, N=9, tree="random_parent", V=5, n_ssm=1)
    _naive_case(spec, cfg, seed=seed, tau=None)
    _naive_case(spec, wl.CONFIGS[2], seed=40 + seed, logits_dtype=torch.bfloat16)


def test_naive_sampling_flags_malformed_tree_and_checks_arguments(spec):
    cfg = wl.CONFIGS[1]
    inp = wl.make_verify_inputs(cfg, mode="greedy")
    par = inp["tree_parent"].clone()
    par[0, 3] = 5
    us = torch.rand(cfg.B, cfg.N)
    status = torch.zeros(cfg.B, dtype=torch.int32, device=DEV)
    path, ln, toks, _ = spec.spec_verify_naive(_dev(inp["logits"]), _dev(inp["tree_token"]), _dev(par), _dev(us), status=status)
    torch.cuda.synchronize()
    assert ln.cpu().numpy()[0] == 0 and status.cpu().numpy()[0] == orc.ST_BAD_TREE
    with pytest.raises(spec.SpecError) as e:
        spec.spec_verify_naive(_dev(inp["logits"]), _dev(inp["tree_token"]), _dev(inp["tree_parent"]), _dev(us), temperature=0.0)
    assert e.value.code == spec.ERR_INVALID_ARG
    with pytest.raises(spec.SpecError) as e:
        spec.spec_verify_naive(_dev(inp["logits"]), _dev(inp["tree_token"]), _dev(inp["tree_parent"]), _dev(us),
                               workspace=torch.empty(256, dtype=torch.uint8, device=DEV)[:16])
    assert e.value.code == spec.ERR_WORKSPACE


def test_multi_step_sampling_verifies_more_tokens_than_naive_sampling(spec):
    """The comparison of Table 3 on synthetic drafts: same trees (width 3 at one level, children sampled
    from drafts close to the LLM), many seeds; multi-step speculative sampling accepts at least as many
    tokens per step on average (Theorem 4.3 gives the per-node inequality)."""
    cfg = dataclasses.replace(wl.CONFIGS[2], B=64, V=512)
    tot_mss = tot_ns = 0
    for seed in range(4):
        inp = wl.make_verify_inputs(cfg, seed=900 + seed, mode="stochastic", tau=1.2)
        us = torch.from_numpy(inp["rng"].random((cfg.B, cfg.N), dtype=np.float32))
        _, ln_m, _ = spec.spec_verify_stochastic(_dev(inp["logits"]), _dev(inp["probs_ssm"]), _dev(inp["ssm_row"]),
                                                 _dev(inp["tree_token"]), _dev(inp["tree_parent"]), _dev(inp["u_accept"]),
                                                 _dev(inp["u_order"]), _dev(inp["u_final"]))
        _, ln_n, _, _ = spec.spec_verify_naive(_dev(inp["logits"]), _dev(inp["tree_token"]), _dev(inp["tree_parent"]), _dev(us))
        torch.cuda.synchronize()
        tot_mss += int(ln_m.sum())
        tot_ns += int(ln_n.sum())
    n = 4 * cfg.B
    print(f"tokens verified per step: multi-step {tot_mss / n:.3f}, naive {tot_ns / n:.3f}, ratio {tot_mss / tot_ns:.3f}")
    assert tot_mss > tot_ns


# ------------------------------------------------------------------------------------------------
# commit
# ------------------------------------------------------------------------------------------------

def _commit_case(spec, cfg, n_layers, paths=None, seed=None):
    inp = wl.make_attention_inputs(cfg, seed=seed, n_layers=n_layers)
    rng = np.random.default_rng(cfg.seed + 7)
    par = inp["tree_parent"].numpy()
    if paths is None:
        ap, al = wl.random_accepted_paths(rng, par)
    else:
        ap, al = paths
    pl = _dev(inp["prefix_len"])
    kcs, vcs = [_dev(c) for c in inp["k_cache"]], [_dev(c) for c in inp["v_cache"]]
    for l in range(n_layers):
        spec.spec_kv_append(_dev(inp["k_new"][l]), _dev(inp["v_new"][l]), kcs[l], vcs[l], pl)
    status = torch.zeros(cfg.B, dtype=torch.int32, device=DEV)
    new_len = spec.spec_kv_commit(kcs, vcs, _dev(ap), _dev(al), pl, cfg.N, status=status)
    torch.cuda.synchronize()
    # oracle on raw bits
    okc = [_bits(c).copy() for c in inp["k_cache"]]
    ovc = [_bits(c).copy() for c in inp["v_cache"]]
    for l in range(n_layers):
        orc.kv_append(okc[l], ovc[l], _bits(inp["k_new"][l]), _bits(inp["v_new"][l]), inp["prefix_len"].numpy())
    ref_len, ref_st = orc.kv_commit(okc, ovc, ap, al, inp["prefix_len"].numpy(), N=cfg.N)
    assert np.array_equal(new_len.cpu().numpy(), ref_len) and np.array_equal(status.cpu().numpy(), ref_st)
    for l in range(n_layers):
        gk, gv = _bits(kcs[l]), _bits(vcs[l])
        for b in range(cfg.B):
            n = int(ref_len[b])      # rows beyond the new prefix are unspecified
            assert np.array_equal(gk[b, :, :n], okc[l][b, :, :n]) and np.array_equal(gv[b, :, :n], ovc[l][b, :, :n])
    return ap, al


def test_commit_config4_layer_sample(spec):
    """LLaMA-65B-shaped caches, accepted paths of random length 1..9, four of the layers."""
    _commit_case(spec, wl.CONFIGS[4], n_layers=4)


def test_commit_small_all_layers_and_overlap(spec):
    cfg = wl.Config(97, "commit", "bf16", B=5, H=3, D=128, P=(10, 60), N=16, tree="expansion", widths=wl.EXPANSION_EVAL)
    par = wl.tree_expansion(wl.EXPANSION_EVAL, 16)
    # hand-made paths on parent = [-1,0,1,2,3,4,5,6,2,8,9,10,2,12,13,14]: overlapping src/dst, identity, root only
    raw = [[0, 1, 2, 8, 9], [0, 1, 2, 12, 13, 14, 15], [0, 1, 2, 3, 4, 5, 6, 7], [0], [0, 1, 2, 8, 9, 10, 11]]
    ap = np.full((5, 16), -1, dtype=np.int32)
    al = np.zeros(5, dtype=np.int32)
    for b, p in enumerate(raw):
        assert orc.path_status(p, len(p), par) == 0
        ap[b, :len(p)] = p
        al[b] = len(p)
    _commit_case(spec, cfg, n_layers=32, paths=(ap, al))
    cfg32 = wl.Config(98, "commit32", "f32", B=5, H=2, D=64, P=(10, 60), N=16, tree="expansion", widths=wl.EXPANSION_EVAL)
    _commit_case(spec, cfg32, n_layers=3, paths=(ap, al))


def test_commit_bad_paths_are_noops(spec):
    cfg = wl.Config(99, "commitbad", "bf16", B=4, H=2, D=128, P=(10, 30), N=16, tree="expansion", widths=wl.EXPANSION_EVAL)
    ap = np.full((4, 16), -1, dtype=np.int32)
    al = np.array([3, 3, 0, 2], dtype=np.int32)
    ap[0, :3] = [0, 1, 2]
    ap[1, :3] = [0, 5, 3]     # not increasing
    ap[3, :2] = [1, 2]        # does not start at the root
    _commit_case(spec, cfg, n_layers=2, paths=(ap, al))


def test_end_to_end_iteration_config5_two_layers(spec):
    """append -> attention -> greedy verify -> commit with the GPU's own accepted path, long ragged prefix."""
    cfg = wl.CONFIGS[5]
    small = wl.Config(5, cfg.name, cfg.dtype, B=2, H=4, D=128, P=(3000, 5000), N=32, tree="expansion", widths=cfg.widths,
                      V=cfg.V)
    inp = wl.make_attention_inputs(small, n_layers=2)
    ver = wl.make_verify_inputs(small, mode="greedy", parent=inp["tree_parent"].numpy())
    pl = _dev(inp["prefix_len"])
    kcs, vcs = [_dev(c) for c in inp["k_cache"]], [_dev(c) for c in inp["v_cache"]]
    par, dep = _dev(inp["tree_parent"]), _dev(inp["tree_depth"])
    outs = []
    for l in range(2):
        outs.append(spec.spec_tree_attention_append(_dev(inp["q"][l]), _dev(inp["k_new"][l]), _dev(inp["v_new"][l]),
                                                    kcs[l], vcs[l], par, dep, pl,
                                                    max_prefix_len=int(inp["prefix_len"].max())))
    path, ln, toks, _ = spec.spec_verify_greedy(_dev(ver["logits"]), _dev(ver["tree_token"]), par)
    new_len = spec.spec_kv_commit(kcs, vcs, path, ln, pl, small.N)
    torch.cuda.synchronize()
    rp, rl, rt, _ = orc.verify_greedy(ver["logits"].numpy(), ver["tree_token"].numpy(), inp["tree_parent"].numpy())
    assert np.array_equal(path.cpu().numpy(), rp) and np.array_equal(toks.cpu().numpy(), rt)
    for l in range(2):
        ref, kco, vco = _oracle_append_attention(inp, layer=l)
        _check_attention(outs[l], ref, torch.bfloat16)
        orc.kv_commit([kco], [vco], rp, rl, inp["prefix_len"].numpy(), N=small.N)
        for b in range(small.B):
            n = int(inp["prefix_len"][b]) + int(rl[b])
            assert new_len[b].item() == n
            assert np.array_equal(kcs[l][b, :, :n].double().cpu().numpy(), kco[b, :, :n])
            assert np.array_equal(vcs[l][b, :, :n].double().cpu().numpy(), vco[b, :, :n])


def test_config5_full_shape_all_32_layers_append_attention_verify_commit(spec):
    """Config 5 at its real shape (4 requests, 32 heads, ragged prefixes of 8192..16384, tree of 32) through
    fused append + attention in all 32 layers, greedy verification and one spec_kv_commit over the 32 layers'
    caches (34 GB). Layer 0 is the host-generated input; the other layers' tensors are drawn on the device
    from per-layer seeds. Compared with the oracle: the verifier's path bit for bit; in EVERY layer the
    appended rows before the commit and the committed rows after it (the oracle's kv_append / kv_commit on
    the window of tree rows, which is all either step may touch), the untouched prefix against a regenerated
    copy; the attention output of the first and the last layer on every (request, head)."""
    cfg = wl.CONFIGS[5]
    L, B, H, D, N = 32, cfg.B, cfg.H, cfg.D, cfg.N
    inp = wl.make_attention_inputs(cfg)
    pl_np, par_np = inp["prefix_len"].numpy(), inp["tree_parent"].numpy()
    ver = wl.make_verify_inputs(cfg, mode="greedy", parent=par_np)
    pl, par, dep = _dev(inp["prefix_len"]), _dev(inp["tree_parent"]), _dev(inp["tree_depth"])
    S = inp["k_cache"][0].shape[2]

    def draw(l, shape, what):
        g = torch.Generator(device=DEV)
        g.manual_seed(cfg.seed * 1000 + l * 10 + what)
        return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32).to(torch.bfloat16)

    q, kn, vn, kcs, vcs = [], [], [], [], []
    for l in range(L):
        if l == 0:
            for dst, name in ((q, "q"), (kn, "k_new"), (vn, "v_new"), (kcs, "k_cache"), (vcs, "v_cache")):
                dst.append(_dev(inp[name][0]))
        else:
            q.append(draw(l, (B, N, H, D), 0)); kn.append(draw(l, (B, N, H, D), 1)); vn.append(draw(l, (B, N, H, D), 2))
            kcs.append(draw(l, (B, H, S, D), 3)); vcs.append(draw(l, (B, H, S, D), 4))
    status = torch.zeros(B, dtype=torch.int32, device=DEV)
    mp = int(pl_np.max())
    outs = [spec.spec_tree_attention_append(q[l], kn[l], vn[l], kcs[l], vcs[l], par, dep, pl, status=status, max_prefix_len=mp)
            for l in range(L)]
    path, ln, toks, _ = spec.spec_verify_greedy(_dev(ver["logits"]), _dev(ver["tree_token"]), par, status=status)
    torch.cuda.synchronize()
    assert (status.cpu().numpy() == 0).all()
    rp, rl, rt, _ = orc.verify_greedy(ver["logits"].numpy(), ver["tree_token"].numpy(), par_np)
    assert np.array_equal(path.cpu().numpy(), rp) and np.array_equal(ln.cpu().numpy(), rl) and np.array_equal(toks.cpu().numpy(), rt)

    def window(c):   # rows [P_b, P_b + N) of every request: [B,H,N,D] raw bits on the host
        return np.stack([_bits(c[b, :, int(pl_np[b]):int(pl_np[b]) + N]) for b in range(B)])

    # attention of the first and the last layer, every (request, head), on what the launch left in the caches
    for l in (0, L - 1):
        qh, kh, vh, oh = q[l].cpu(), kcs[l].cpu(), vcs[l].cpu(), outs[l].cpu()
        for b in range(B):
            ref = orc.tree_attention(_f64(qh[b:b + 1]), _f64(kh[b:b + 1]), _f64(vh[b:b + 1]), par_np[b:b + 1], pl_np[b:b + 1])
            _check_attention(oh[b:b + 1], ref, torch.bfloat16)
    # append, every layer: the oracle's kv_append on the window (a cache of N rows behind a prefix of 0)
    zero = np.zeros(B, dtype=np.int32)
    want_k, want_v = [], []
    for l in range(L):
        wk, wv = np.zeros((B, H, N, D), dtype=np.int16), np.zeros((B, H, N, D), dtype=np.int16)
        assert (orc.kv_append(wk, wv, _bits(kn[l]), _bits(vn[l]), zero) == 0).all()
        assert np.array_equal(window(kcs[l]), wk) and np.array_equal(window(vcs[l]), wv), l
        want_k.append(wk); want_v.append(wv)
    # commit over all layers in one call
    new_len = spec.spec_kv_commit(kcs, vcs, path, ln, pl, N, status=status)
    torch.cuda.synchronize()
    assert (status.cpu().numpy() == 0).all()
    ref_len, ref_st = orc.kv_commit(want_k, want_v, rp, rl, zero, N=N)
    assert (ref_st == 0).all() and np.array_equal(new_len.cpu().numpy(), pl_np + ref_len)
    assert rl.max() > 1   # some request moves rows
    for l in range(L):
        gk, gv = window(kcs[l]), window(vcs[l])
        for b in range(B):
            n = int(ref_len[b])                     # rows beyond the new prefix are unspecified
            assert np.array_equal(gk[b, :, :n], want_k[l][b, :, :n]) and np.array_equal(gv[b, :, :n], want_v[l][b, :, :n]), (l, b)
        # the prefix rows are untouched
        k0 = _dev(inp["k_cache"][0]) if l == 0 else draw(l, (B, H, S, D), 3)
        v0 = _dev(inp["v_cache"][0]) if l == 0 else draw(l, (B, H, S, D), 4)
        for b in range(B):
            p = int(pl_np[b])
            assert torch.equal(kcs[l][b, :, :p], k0[b, :, :p]) and torch.equal(vcs[l][b, :, :p], v0[b, :, :p]), (l, b)
        del k0, v0


def test_decoding_loop_in_one_graph_with_lengths_advancing_on_the_device(spec):
    """Algorithm 2's loop: every iteration appends and attends a tree behind the current prefix, verifies it
    and commits the accepted path; prefix lengths live on the device only. Two iterations (ping-pong length
    buffers) are captured in one HIP graph and replayed; caches, lengths and the last iteration's attention
    outputs must equal the oracle's simulation of the same four iterations."""
    K, L = 4, 2
    cfg = wl.Config(87, "loop", "bf16", B=3, H=2, D=64, P=(10, 40), N=16, tree="expansion", widths=wl.EXPANSION_EVAL, V=64)
    cap = 40 + K * cfg.N + cfg.N
    inp = wl.make_attention_inputs(cfg, seed=23, n_layers=L, S_cap=cap)
    ver = wl.make_verify_inputs(cfg, seed=23, mode="greedy", parent=inp["tree_parent"].numpy())
    par, dep = _dev(inp["tree_parent"]), _dev(inp["tree_depth"])
    q, kn, vn = [_dev(x) for x in inp["q"]], [_dev(x) for x in inp["k_new"]], [_dev(x) for x in inp["v_new"]]
    kcs, vcs = [_dev(x) for x in inp["k_cache"]], [_dev(x) for x in inp["v_cache"]]
    outs = [torch.empty_like(x) for x in q]
    logits, tok = _dev(ver["logits"]), _dev(ver["tree_token"])
    pl = [_dev(inp["prefix_len"]), torch.zeros(cfg.B, dtype=torch.int32, device=DEV)]
    status = torch.zeros(cfg.B, dtype=torch.int32, device=DEV)
    desc = spec.make_desc(q[0], kcs[0], max_prefix_len=cap - cfg.N)
    ws = torch.empty(max(spec.spec_tree_attention_workspace_bytes(desc), 256), dtype=torch.uint8, device=DEV)
    vout = (torch.empty((cfg.B, cfg.N), dtype=torch.int32, device=DEV), torch.empty(cfg.B, dtype=torch.int32, device=DEV),
            torch.empty((cfg.B, cfg.N), dtype=torch.int32, device=DEV), torch.empty((cfg.B, cfg.N), dtype=torch.int32, device=DEV))

    def iteration(src, dst):
        for l in range(L):
            spec.spec_tree_attention_append(q[l], kn[l], vn[l], kcs[l], vcs[l], par, dep, pl[src], out=outs[l], workspace=ws,
                                            status=status, desc=desc)
        spec.spec_verify_greedy(logits, tok, par, status=status, out=vout)
        spec.spec_kv_commit(kcs, vcs, vout[0], vout[1], pl[src], cfg.N, prefix_len_out=pl[dst], status=status)

    # warm-up outside capture on copies of the state, then restore it
    saved = [x.clone() for x in kcs + vcs], pl[0].clone()
    iteration(0, 1)
    torch.cuda.synchronize()
    for dst_t, src_t in zip(kcs + vcs, saved[0]):
        dst_t.copy_(src_t)
    pl[0].copy_(saved[1])
    status.zero_()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        iteration(0, 1)
        iteration(1, 0)
    for dst_t, src_t in zip(kcs + vcs, saved[0]):      # capture does not execute, but keep the state explicit
        dst_t.copy_(src_t)
    pl[0].copy_(saved[1])
    for _ in range(K // 2):
        graph.replay()
    torch.cuda.synchronize()
    assert (status.cpu().numpy() == 0).all()

    # oracle: the same K iterations
    f64 = lambda t: t.double().numpy()
    kco, vco = [f64(x) for x in inp["k_cache"]], [f64(x) for x in inp["v_cache"]]
    plen = inp["prefix_len"].numpy().copy()
    rp, rl, rt, _ = orc.verify_greedy(ver["logits"].numpy(), ver["tree_token"].numpy(), inp["tree_parent"].numpy())
    assert rl.max() > 1                                  # something is accepted, so prefixes advance unevenly
    refs = None
    for it in range(K):
        refs = []
        for l in range(L):
            assert (orc.kv_append(kco[l], vco[l], f64(inp["k_new"][l]), f64(inp["v_new"][l]), plen) == 0).all()
            refs.append(orc.tree_attention(f64(inp["q"][l]), kco[l], vco[l], inp["tree_parent"].numpy(), plen))
        plen, st = orc.kv_commit(kco, vco, rp, rl, plen, N=cfg.N)
        assert (st == 0).all()
    assert np.array_equal(pl[0].cpu().numpy(), plen)
    assert np.array_equal(vout[0].cpu().numpy(), rp) and np.array_equal(vout[2].cpu().numpy(), rt)
    for l in range(L):
        _check_attention(outs[l], refs[l], torch.bfloat16)
        for b in range(cfg.B):
            assert np.array_equal(kcs[l][b, :, :plen[b]].double().cpu().numpy(), kco[l][b, :, :plen[b]])
            assert np.array_equal(vcs[l][b, :, :plen[b]].double().cpu().numpy(), vco[l][b, :, :plen[b]])


def test_hip_graph_replays_match_eager(spec):
    """The benchmark replays a captured pass; every replay must reproduce the eager results, with
    eager launches and synchronisations in between."""
    cfg = wl.Config(2, "graph", "bf16", B=2, H=4, D=128, P=(300, 500), N=16, tree="expansion", widths=wl.EXPANSION_EVAL,
                    V=3000)
    L = 3
    inp = wl.make_attention_inputs(cfg, n_layers=L)
    ver = wl.make_verify_inputs(cfg, mode="greedy", parent=inp["tree_parent"].numpy())
    pl, par, dep = _dev(inp["prefix_len"]), _dev(inp["tree_parent"]), _dev(inp["tree_depth"])
    q, kn, vn = [_dev(x) for x in inp["q"]], [_dev(x) for x in inp["k_new"]], [_dev(x) for x in inp["v_new"]]
    k0, v0 = [_dev(x) for x in inp["k_cache"]], [_dev(x) for x in inp["v_cache"]]
    kcs, vcs = [x.clone() for x in k0], [x.clone() for x in v0]
    outs = [torch.empty_like(x) for x in q]
    logits, tok = _dev(ver["logits"]), _dev(ver["tree_token"])
    desc = spec.make_desc(q[0], kcs[0], max_prefix_len=int(inp["prefix_len"].max()))
    ws = torch.empty(max(spec.spec_tree_attention_workspace_bytes(desc), 256), dtype=torch.uint8, device=DEV)
    vout = (torch.empty((2, 16), dtype=torch.int32, device=DEV), torch.empty(2, dtype=torch.int32, device=DEV),
            torch.empty((2, 16), dtype=torch.int32, device=DEV), torch.empty((2, 16), dtype=torch.int32, device=DEV))
    pl_out = torch.empty_like(pl)

    def one_pass():
        for l in range(L):
            if l == 0:
                spec.spec_kv_append(kn[l], vn[l], kcs[l], vcs[l], pl, desc=desc)
                spec.spec_tree_attention(q[l], kcs[l], vcs[l], par, dep, pl, out=outs[l], workspace=ws, desc=desc)
            else:
                spec.spec_tree_attention_append(q[l], kn[l], vn[l], kcs[l], vcs[l], par, dep, pl, out=outs[l],
                                                workspace=ws, desc=desc)
        spec.spec_verify_greedy(logits, tok, par, out=vout)
        spec.spec_kv_commit(kcs, vcs, vout[0], vout[1], pl, cfg.N, prefix_len_out=pl_out)

    def snapshot():
        torch.cuda.synchronize()
        return [o.clone() for o in outs] + [c.clone() for c in kcs] + [x.clone() for x in vout] + [pl_out.clone()]

    def reset():
        for l in range(L):
            kcs[l].copy_(k0[l])
            vcs[l].copy_(v0[l])
            outs[l].zero_()
        for x in vout:
            x.fill_(-7)
        pl_out.zero_()

    one_pass()
    want = snapshot()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        one_pass()
    for rep in range(4):
        reset()
        torch.cuda.synchronize()
        graph.replay()
        got = snapshot()
        for a, b in zip(want, got):
            assert torch.equal(a, b), f"replay {rep} differs from the eager pass"
        one_pass()                      # eager work between replays
        torch.cuda.synchronize()
