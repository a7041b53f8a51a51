"""float32 attention kernel at the edges of its tiles: queries per K/V head around one and two 16-query tiles and past
one workgroup, keys around a wavefront tile, a round of the four wavefronts and a chunk, the key range cut by default.

Bar: max abs error 1e-5 against the float64 oracle. Inputs are N(0, 1), so scores are O(1) after the scale, a float32
sum of 128 products is good to about 128 * 2^-24 = 8e-6 of its largest partial sum at worst and 1e-6 typically, and the
outputs are averages of N(0, 1) values."""
import numpy as np
import pytest
import torch

from paper_2305_09781_amd import workloads as wl
from test_gpu_parity import _check_attention, _oracle_append_attention, _run_append_attention

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    # B, H, H_kv, D, (P lo, hi), N
    (2, 4, 4, 64, (0, 1), 1),          # nothing but the tree
    (2, 4, 4, 64, (15, 17), 16),       # one full query tile, keys around one tile
    (2, 3, 3, 128, (47, 49), 17),      # two query tiles, the tree crosses a wavefront round
    (2, 2, 2, 128, (61, 67), 33),      # a second workgroup for the last query
    (1, 2, 2, 64, (127, 127), 128),    # widest tree
    (3, 8, 2, 128, (30, 90), 5),       # grouped heads: 20 queries of four heads in two tiles
    (2, 6, 1, 64, (100, 130), 16),     # one K/V head for six: three workgroups of two heads
    (2, 4, 4, 128, (300, 447), 9),     # around the length from which the key range is cut
    (2, 4, 4, 128, (440, 700), 24),    # cut by default, chunks past the shorter request's end
    (40, 7, 7, 128, (180, 400), 11),   # uncut: one query tile, up to seven tiles a wavefront
    (40, 7, 7, 64, (180, 400), 11),
    (33, 8, 8, 64, (180, 400), 19),    # two query tiles
], ids=lambda c: f"B{c[0]}H{c[1]}kv{c[2]}D{c[3]}P{c[4][0]}-{c[4][1]}N{c[5]}")
def test_float32_attention_tile_edges(spec, case):
    B, H, H_kv, D, P, N = case
    cfg = wl.Config(90, "f32", "f32", B=B, H=H, D=D, P=P if P[0] != P[1] else P[0], N=N, tree="random_branching", H_kv=H_kv)
    inp = wl.make_attention_inputs(cfg, seed=3000 + N + D + H, S_cap=P[1] + N + 3)
    ref, kco, vco = _oracle_append_attention(inp)
    for fused in (False, True):
        status = torch.zeros(B, dtype=torch.int32, device="cuda:0")
        if fused or H == H_kv:      # the append-only call takes its layout from k_new alone
            out, kc, vc = _run_append_attention(spec, inp, status=status, fused=fused)
            _check_attention(out, ref, torch.float32)
            assert (status.cpu().numpy() == 0).all()
            assert np.array_equal(kc.double().cpu().numpy(), kco) and np.array_equal(vc.double().cpu().numpy(), vco), fused


def test_float32_fused_append_of_a_malformed_tree(spec):
    """The append does not depend on the tree: its rows are written, the outputs are zeros and the request is flagged."""
    cfg = wl.Config(90, "f32", "f32", B=2, H=2, D=64, P=50, N=8, tree="random_parent")
    inp = wl.make_attention_inputs(cfg, seed=3)
    ref, kco, vco = _oracle_append_attention(inp)
    inp["tree_parent"][1, 3] = 5
    status = torch.zeros(2, dtype=torch.int32, device="cuda:0")
    out, kc, vc = _run_append_attention(spec, inp, status=status, fused=True)
    assert status.tolist() == [0, spec.ST_BAD_TREE]
    _check_attention(out[:1], ref[:1], torch.float32)
    assert (out[1] == 0).all()
    assert np.array_equal(kc.double().cpu().numpy(), kco) and np.array_equal(vc.double().cpu().numpy(), vco)


def _float32_loop(q, k, v, mask, scale):
    """One query at a time in float32: scores as four sums of fused products, added in pairs, softmax and output one key after
    the other. (A fused multiply-add is a float64 one, rounded: the product of two float32 is exact there.)"""
    f32 = np.float32
    fma = lambda a, b, c: (a.astype(np.float64) * b + c).astype(f32)  # noqa: E731
    s4 = [np.zeros((q.shape[0], k.shape[0]), f32) for _ in range(4)]
    for d in range(0, q.shape[1], 4):
        for e in range(4):
            s4[e] = fma(q[:, None, d + e], k[None, :, d + e], s4[e])
    s = ((s4[0] + s4[1]) + (s4[2] + s4[3])) * f32(scale * 1.4426950408889634)
    s[~mask] = -np.inf
    p = np.exp2(s - s.max(1, keepdims=True))
    l, o = np.zeros(q.shape[0], f32), np.zeros((q.shape[0], v.shape[1]), f32)
    for j in range(k.shape[0]):
        l = l + p[:, j]
        o = fma(p[:, j:j + 1], v[j][None], o)
    return o * (f32(1) / l)[:, None]


@pytest.mark.parametrize("H,H_kv,D,P,N", [(4, 4, 128, 40, 19), (8, 8, 64, 16, 4), (6, 3, 128, 60, 40), (4, 4, 128, 30, 1), (4, 4, 64, 128, 8)])
def test_float32_attention_is_no_further_off_than_a_float32_loop(spec, H, H_kv, D, P, N):
    """Relative error against float64 over short key ranges, where it is that of the scores, averaged over four inputs."""
    err = np.zeros((4, 2))
    for seed in range(4):
        cfg = wl.Config(90, "f32", "f32", B=2, H=H, D=D, P=P, N=N, tree="random_branching", H_kv=H_kv)
        inp = wl.make_attention_inputs(cfg, seed=6000 + seed, S_cap=P + N + 3)
        ref, kco, vco = _oracle_append_attention(inp)
        out, _, _ = _run_append_attention(spec, inp, fused=True)
        loop = np.empty_like(ref)
        for b in range(2):
            par = inp["tree_parent"][b].numpy()
            mask = np.ones((N, P + N), bool)
            mask[:, P:] = False
            for n in range(N):
                u = n
                while u >= 0:
                    mask[n, P + u] = True
                    u = int(par[u])
            for h in range(H):
                kv = h // (H // H_kv)
                loop[b, :, h] = _float32_loop(inp["q"][0][b, :, h].numpy(), kco[b, kv, :P + N].astype(np.float32),
                                              vco[b, kv, :P + N].astype(np.float32), mask, 1 / np.sqrt(D))
        err[seed] = [np.linalg.norm(x - ref) / np.linalg.norm(ref) for x in (out.double().cpu().numpy(), loop)]
    kernel, plain = err.mean(0)
    print("relative error: kernel %.3e, float32 loop %.3e" % (kernel, plain))
    assert kernel <= plain
