"""Top-k and merge kernels where they can go wrong: rows that are not 16-byte aligned, longer than one round of a
workgroup's loads, picks that all lie with one thread, ties, signed zeros, infinities and NaN; merges of one tree, of the
most input nodes, of chains, and of trees whose sizes differ. Bit-exact."""
import numpy as np
import pytest
import torch

from oracle import spec_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("V,k,dt,offset", [(1, 1, "f32", 0), (4096, 3, "f32", 0), (32768, 4, "f32", 0), (40004, 16, "f32", 0),
                                           (40003, 5, "f32", 0), (32000, 3, "f32", 1), (32000, 3, "bf16", 0), (70000, 16, "bf16", 0),
                                           (32004, 3, "bf16", 0), (64000, 2, "bf16", 4), (131072, 16, "f32", 0)])
def test_topk_row_lengths_and_alignments(spec, V, k, dt, offset):
    rng = np.random.default_rng(V + k)
    x = torch.from_numpy(np.round(rng.standard_normal((2, 2, V)) * 3, 1).astype(np.float32))     # coarse: many ties
    if V > 4096:
        x[0, 0, 7::4096] = 50.0 - torch.arange(x[0, 0, 7::4096].numel())      # every pick with the thread that owns element 7
        x[0, 1, 5::8192] = 60.0                                               # equal maxima: ascending ids
    x = x.to(torch.bfloat16 if dt == "bf16" else torch.float32)
    buf = torch.zeros(x.numel() + offset, dtype=x.dtype, device=DEV)
    dev = buf[offset:].view(x.shape)      # a base that is not 16-byte aligned
    dev.copy_(x)
    N = 2 * k
    slots = torch.arange(2 * k, dtype=torch.int32).view(2, k)
    tok = torch.full((2, max(N, 1)), -5, dtype=torch.int32, device=DEV)
    spec.spec_tree_expand_topk(dev, k, slots.to(DEV), tok)
    want = orc.expand_topk(x.float().numpy(), k).reshape(2, 2 * k)
    assert np.array_equal(tok.cpu().numpy(), want)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_topk_finds_the_largest_in_every_lane(spec, dt):
    """One row per thread of a workgroup, whose largest element that thread owns; the second largest lies with its neighbour."""
    vec, F = (4, 1024) if dt == "f32" else (8, 1024)
    x = torch.zeros((1, F, 1024 * vec), dtype=torch.float32)
    f = torch.arange(F)
    x[0, f, f * vec + f % vec] = 9.0
    x[0, f, (f * vec + vec) % (1024 * vec)] = 8.0
    x = x.to(torch.bfloat16 if dt == "bf16" else torch.float32)
    for f0 in range(0, F, 64):
        tok = torch.full((1, 128), -5, dtype=torch.int32, device=DEV)
        spec.spec_tree_expand_topk(x[:, f0:f0 + 64].contiguous().to(DEV), 2, torch.arange(128, dtype=torch.int32, device=DEV).view(64, 2), tok)
        n = np.arange(f0, f0 + 64)
        assert np.array_equal(tok.cpu().numpy().reshape(64, 2), np.stack([n * vec + n % vec, (n * vec + vec) % (1024 * vec)], 1))


def test_topk_zeros_infinities_and_nan(spec):
    x = torch.full((1, 4, 12), -1.0)
    x[0, 0, 3], x[0, 0, 5] = 0.0, -0.0                    # equal: the lower id first
    x[0, 1, 2], x[0, 1, 9] = -0.0, 0.0
    x[0, 2, 4], x[0, 2, 6] = float("inf"), float("nan")
    x[0, 3, :] = float("nan")
    x[0, 3, 8] = float("-inf")
    tok = torch.zeros((1, 12), dtype=torch.int32, device=DEV)
    spec.spec_tree_expand_topk(x.to(DEV), 3, torch.arange(12, dtype=torch.int32, device=DEV).view(4, 3), tok)
    assert tok.cpu().tolist() == [[3, 5, 0, 2, 9, 0, 4, 0, 1, 8, -1, -1]]


@pytest.mark.parametrize("M,Nin,Nout,chain", [(1, 1, 1, False), (1, 64, 64, True), (3, 21, 63, False), (13, 5, 65, False),
                                              (8, 128, 128, True), (2, 512, 128, False), (64, 16, 100, False)])
def test_merge_sizes(spec, M, Nin, Nout, chain):
    rng = np.random.default_rng(M * 1000 + Nin)
    B = 4
    par = np.full((B, M, Nin), -1, dtype=np.int32)
    tok = np.zeros((B, M, Nin), dtype=np.int32)
    size = np.zeros((B, M), dtype=np.int32)
    for b in range(B):
        for m in range(M):
            size[b, m] = rng.integers(max(1, Nin // 2), Nin + 1)
            for u in range(1, Nin):
                par[b, m, u] = u - 1 if chain else rng.integers(max(0, u - 4), u)
                tok[b, m, u] = rng.integers(0, 2 if b else 40)          # few tokens: many merges; many: overflow
    dev = lambda a: torch.from_numpy(a).to(DEV)  # noqa: E731
    status = torch.zeros(B, dtype=torch.int32, device=DEV)
    got = spec.spec_tree_merge(dev(par), dev(tok), dev(size), Nout, status=status)
    for b in range(B):
        for g, w in zip(list(got) + [status], orc.tree_merge(par[b], tok[b], size[b], Nout)):
            assert np.array_equal(g[b].cpu().numpy(), np.asarray(w))


def _shapes(kind, n):
    if kind == "star":
        return np.concatenate([[-1], np.zeros(n - 1)])
    if kind == "chain":
        return np.arange(-1, n - 1)
    spine = n // 2                                         # a chain whose other nodes hang on its middle and on its end
    return np.concatenate([np.arange(-1, spine - 1), np.where(np.arange(n - spine) % 2, spine // 2, spine - 1)])


@pytest.mark.parametrize("M,Nin,kind,tokens", [(8, 128, "star", 3), (8, 128, "star", 100), (1, 128, "chain", 9), (3, 100, "chain", 2),
                                               (1, 1024, "chain", 5), (1, 100, "comb", 2), (7, 61, "comb", 4), (1, 9, "star", 1),
                                               (1, 10, "star", 2), (2, 5, "star", 9)])
def test_merge_of_wide_and_narrow_levels(spec, M, Nin, kind, tokens):
    """Levels of one node, of a few and of a thousand, runs of the first next to the others, siblings that repeat tokens."""
    rng = np.random.default_rng(M * 1000 + Nin + tokens)
    B = 3
    par = np.broadcast_to(_shapes(kind, Nin), (B, M, Nin)).astype(np.int32)
    tok = rng.integers(0, tokens, size=(B, M, Nin)).astype(np.int32)
    tok[:, :, 0] = 1
    size = np.full((B, M), Nin, dtype=np.int32)
    size[1:] = rng.integers(1, Nin + 1, size=(B - 1, M))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
    status = torch.zeros(B, dtype=torch.int32, device=DEV)
    got = spec.spec_tree_merge(dev(par), dev(tok), dev(size), 128, status=status)
    for b in range(B):
        for g, w in zip(list(got) + [status], orc.tree_merge(par[b], tok[b], size[b], 128)):
            assert np.array_equal(g[b].cpu().numpy(), np.asarray(w))


@pytest.mark.parametrize("M,Nin,Nout", [(64, 1, 1), (1, 63, 63), (21, 3, 64), (4, 16, 128), (2, 32, 30), (13, 5, 128), (5, 7, 128)])
def test_merge_around_one_wavefront(spec, M, Nin, Nout):
    """Up to 64 input nodes are one wavefront's work: random trees that agree in part, sizes that leave slots unused, too many
    sequences, and one malformed tree, or root, in a batch; (13, 5) is one node more."""
    rng = np.random.default_rng(M * 100 + Nin)
    B = 24
    par = np.full((B, M, Nin), -1, dtype=np.int32)
    tok = rng.integers(0, 3, size=(B, M, Nin)).astype(np.int32)
    tok[B // 2:, :, :] = rng.integers(0, 1000, size=(B - B // 2, M, Nin))
    tok[:, :, 0] = 7
    for u in range(1, Nin):
        par[:, :, u] = rng.integers(0, u, size=(B, M))
    size = rng.integers(1, Nin + 1, size=(B, M)).astype(np.int32)
    size[0] = Nin
    size[3, M - 1], size[4, 0], tok[5, M - 1, 0] = Nin + 1, 0, 8 if M > 1 else 7
    if Nin > 1:
        size[6:9, 0] = Nin
        par[6, 0, 1], par[7, 0, Nin - 1], tok[8, 0, 1] = -1, Nin - 1, -2
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
    status = torch.zeros(B, dtype=torch.int32, device=DEV)
    got = spec.spec_tree_merge(dev(par), dev(tok), dev(size), Nout, status=status)
    for b in range(B):
        for g, w in zip(list(got) + [status], orc.tree_merge(par[b], tok[b], size[b], Nout)):
            assert np.array_equal(g[b].cpu().numpy(), np.asarray(w)), b


def test_merge_of_repeated_tokens_ends_its_comparisons_early(spec):
    """Stars of 128 nodes merged from eight trees: with three different tokens every node finds its like among the first few
    of its level, which takes half as long as comparing a thousand different ones."""
    B, M, Nin = 16, 8, 128
    par = torch.from_numpy(_shapes("star", Nin).astype(np.int32)).to(DEV).expand(B, M, Nin).contiguous()
    size = torch.full((B, M), Nin, dtype=torch.int32, device=DEV)
    us = []
    for tokens in (3, 32000):
        tok = torch.randint(0, tokens, (B, M, Nin), generator=torch.Generator(device=DEV).manual_seed(tokens), device=DEV, dtype=torch.int32)
        tok[:, :, 0] = 1
        spec.spec_tree_merge(par, tok, size, 128)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(10):
                spec.spec_tree_merge(par, tok, size, 128)
        times = []
        for _ in range(7):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            graph.replay()
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end) * 100)
        us.append(sorted(times)[3])
    assert us[0] < 0.75 * us[1], us
