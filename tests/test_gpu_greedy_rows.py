"""Arg-max rows and the one-wavefront greedy walk where they can go wrong: rows of one group, of exactly one round, past it,
and of no whole groups; few and many rows; ties, signed zeros, infinities and NaN; trees of 1, 64, 65 and 128 nodes, cut paths
and malformed trees. Bit-exact."""
import numpy as np
import pytest
import torch

from oracle import spec_oracle as orc
from paper_2305_09781_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _argmax(x):
    """Lowest index of the largest value that is not NaN; 0 when there is none above -inf."""
    y = np.where(np.isnan(x), -np.inf, x)
    return y.argmax(axis=-1).astype(np.int32)


@pytest.mark.parametrize("V", [1, 4, 8, 12, 8192, 8200, 16384, 16392, 40960, 32003])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("B,N", [(2, 5), (16, 64)])
def test_argmax_rows(spec, V, dt, B, N):
    if B * N * V > 2e7:
        N = 1200 // B if V > 8200 and B > 2 else N
    rng = np.random.default_rng(V + N)
    x = np.round(rng.standard_normal((B, N, V)).astype(np.float32) * 2)          # coarse: many ties
    x[0, 0] = -np.inf
    x[0, 1, : V // 2 + 1] = np.nan
    x[0, 2] = -0.0
    x[0, 2, V // 2] = 0.0
    x[0, 3, V - 1] = np.inf
    x[1, 0] = np.nan
    logits = torch.from_numpy(x).to(torch.bfloat16 if dt == "bf16" else torch.float32)
    par = np.stack([wl.tree_random_parent(rng, N) for _ in range(B)])
    tok = rng.integers(0, V, size=(B, N)).astype(np.int32)
    got = spec.spec_verify_greedy(logits.to(DEV), torch.from_numpy(tok).to(DEV), torch.from_numpy(par).to(DEV))
    assert np.array_equal(got[3].cpu().numpy(), _argmax(logits.float().numpy()))


@pytest.mark.parametrize("N", [1, 2, 63, 64, 65, 128])
@pytest.mark.parametrize("Lmax", [1, 3, 128, 200])
def test_walk_sizes(spec, N, Lmax):
    rng = np.random.default_rng(N * 7 + Lmax)
    B, V = 6, 40
    par = np.stack([wl.tree_random_parent(rng, N) if b % 2 else np.arange(-1, N - 1, dtype=np.int32) for b in range(B)])
    logits = rng.standard_normal((B, N, V)).astype(np.float32)
    tok = rng.integers(0, V, size=(B, N)).astype(np.int32)
    for b in range(B):                                      # most nodes carry their parent's choice: long paths, duplicates
        for v in range(1, N):
            if rng.random() < 0.8:
                tok[b, v] = logits[b, par[b, v]].argmax()
    if N > 2:
        par[5, 2] = 2                                       # malformed
    status = torch.zeros(B, dtype=torch.int32, device=DEV)
    dev = lambda a: torch.from_numpy(a).to(DEV)  # noqa: E731
    path, ln, toks, _ = spec.spec_verify_greedy(dev(logits), dev(tok), dev(par), Lmax=Lmax, status=status)
    for b in range(B):
        if N > 2 and b == 5:
            assert status[b].item() == orc.ST_BAD_TREE and ln[b].item() == 0 and (path[b] == -1).all() and (toks[b] == -1).all()
            continue
        u, want, out = 0, [0], []
        while len(want) < Lmax:                             # the walk as the paper states it
            ch = [v for v in range(N) if par[b, v] == u and tok[b, v] == logits[b, u].argmax()]
            if not ch:
                break
            u = ch[0]
            want.append(u)
            out.append(int(tok[b, u]))
        out.append(int(logits[b, u].argmax()))
        n = len(want)
        assert ln[b].item() == n and path[b, :n].tolist() == want and toks[b, :n].tolist() == out
        assert (path[b, n:] == -1).all() and (toks[b, n:] == -1).all()


@pytest.mark.parametrize("dt,rows,V", [
    # workgroups of 1024: one to five half sweeps of 16384 float32 or 32768 bfloat16, at and one group past their ends
    ("f32", 3, 16384), ("f32", 3, 16388), ("f32", 3, 32768), ("f32", 3, 32772), ("f32", 3, 65536), ("f32", 3, 65540), ("f32", 3, 81920),
    ("f32", 130, 65536), ("f32", 130, 49156), ("bf16", 3, 32768), ("bf16", 3, 32776), ("bf16", 3, 65536), ("bf16", 3, 65544),
    ("bf16", 3, 131072), ("bf16", 3, 131080),
    # of 256: halves of 4096 or 8192, in a thousand rows and more
    ("f32", 1030, 4100), ("f32", 1030, 8192), ("f32", 1030, 8196), ("f32", 1030, 12292), ("bf16", 1030, 8200), ("bf16", 1030, 16392),
    # fewer groups than threads
    ("f32", 1030, 12), ("bf16", 5, 1024)])
def test_argmax_by_whole_and_by_half_sweeps(spec, dt, rows, V):
    """The largest value in the first, a middle and the last element, and on either side of the last border of sweeps, twice in a row."""
    rng = np.random.default_rng(V + rows)
    x = rng.integers(-3, 3, size=(rows, V)).astype(np.float32)
    half = (256 if rows >= 1024 or V <= (8192 if dt == "bf16" else 4096) else 1024) * (32 if dt == "bf16" else 16)
    border = (V - 1) // half * half
    for i, at in enumerate((0, V - 1, V // 2, border, max(border - 1, 0), min(border + 1, V - 1), V - 2)):
        x[i % rows, at] = x[i % rows, min(V - 1, at + 5)] = 9.0
    x[rows - 1, -4:] = (-np.inf, np.nan, 9.0, -0.0)
    logits = torch.from_numpy(x).to(torch.bfloat16 if dt == "bf16" else torch.float32).view(rows, 1, V).to(DEV)
    one = torch.zeros((rows, 1), dtype=torch.int32, device=DEV)
    got = spec.spec_verify_greedy(logits, one, one - 1)
    assert np.array_equal(got[3].cpu().numpy()[:, 0], _argmax(x))
