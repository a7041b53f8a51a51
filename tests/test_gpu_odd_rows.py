"""Rows of vocabularies that 16-byte groups do not divide: arg-max (greedy verification), top-k and the per-node statistics,
where groups overlap at both ends of a row. Exact against numpy."""
import numpy as np
import pytest
import torch

from oracle import spec_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _rows(V, n, dt, seed):
    """Coarse values (ties in abundance), the maximum planted at the ends and around group boundaries, infinities and NaN."""
    rng = np.random.default_rng(seed)
    x = np.round(rng.standard_normal((n, V)) * 2).astype(np.float32)
    for i, at in enumerate((0, V - 1, min(V - 1, 7), min(V - 1, 8), max(0, V - 9), max(0, V - 8), V // 2)):
        x[i % n, at] = 50.0
        x[(i + 1) % n, at] = 50.0                                  # equal maxima: the lower id
    x[n - 1, :] = -np.inf
    x[n - 2, V // 3:] = np.nan
    x[n - 3, V - 1] = np.inf
    return torch.from_numpy(x).to(torch.bfloat16 if dt == "bf16" else torch.float32)


@pytest.mark.parametrize("V", [1, 3, 4, 5, 7, 8, 9, 13, 1025, 2047, 2050, 4778, 8195, 16385, 33001, 65539, 128257])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_argmax_and_topk(spec, V, dt):
    N = 12
    x = _rows(V, N, dt, V)
    f = np.where(np.isnan(x.float().numpy()), -np.inf, x.float().numpy())
    logits = x.to(DEV).view(1, N, V)
    par = torch.arange(-1, N - 1, dtype=torch.int32, device=DEV).view(1, N)
    tok = torch.zeros((1, N), dtype=torch.int32, device=DEV)
    amax = spec.spec_verify_greedy(logits, tok, par)[3].cpu().numpy()[0]
    assert np.array_equal(amax[:-1], f.argmax(1)[:-1]) and amax[-1] == 0
    k = min(5, V)
    n = N - 2                                                     # rows without NaN or only -inf
    slots = torch.arange(n * k, dtype=torch.int32, device=DEV).view(n, k)
    got = torch.full((1, n * k), -7, dtype=torch.int32, device=DEV)
    spec.spec_tree_expand_topk(logits[:, :n].contiguous(), k, slots, got)
    assert np.array_equal(got.cpu().numpy().reshape(n, k), orc.expand_topk(f[None, :n], k).reshape(n, k))


@pytest.mark.parametrize("V,N", [(1, 3), (2, 3), (5, 4), (1027, 9), (4097, 9), (8193, 9), (16390, 9), (32767, 9), (40001, 5)])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_statistics_of_a_long_chain(spec, V, N, dt):
    """All nodes accepted, then the last token drawn: the path shows the statistics only through the draw, whose token must
    lie where the float64 distribution has it (within 1e-5 of the uniform: float32 sums of V terms)."""
    rng = np.random.default_rng(V)
    x = torch.from_numpy(rng.standard_normal((1, N, V)).astype(np.float32) * 3).to(torch.bfloat16 if dt == "bf16" else torch.float32)
    par = torch.arange(-1, N - 1, dtype=torch.int32, device=DEV).view(1, N)
    tok = torch.from_numpy(rng.integers(0, V, size=(1, N)).astype(np.int32)).to(DEV)
    probs = torch.full((1, V), 1.0 / V, device=DEV)
    zero = torch.zeros((1, N), device=DEV)
    for u in (0.0, 0.123, 0.5, 0.999, 1.0 - 2.0 ** -24):
        path, ln, out = spec.spec_verify_stochastic(x.to(DEV), probs, torch.zeros((1, N), dtype=torch.int32, device=DEV), tok, par, zero, zero,
                                                    torch.tensor([u], device=DEV))
        assert ln.item() == N and path.cpu().tolist() == [list(range(N))]
        assert out[0, :N - 1].cpu().tolist() == tok[0, 1:].cpu().tolist()
        z = x[0, -1].double().numpy()
        cdf = np.cumsum(np.exp(z - z.max()))
        cdf /= cdf[-1]
        t = out[0, N - 1].item()
        assert 0 <= t < V and cdf[t] > u - 1e-5 and (t == 0 or cdf[t - 1] <= u + 1e-5)
