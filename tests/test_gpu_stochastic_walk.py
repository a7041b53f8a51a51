"""The stochastic walk over the vocabulary sizes where its form changes (rows of whole 16-byte groups or not, one to
eight groups per thread, the buffer form), with the nodes' statistics taken by the walk or before it, against the oracle on vetted
uniforms: bit-exact paths, lengths, tokens and status."""
import numpy as np
import pytest
import torch

from oracle import spec_oracle as orc
from oracle import vetting
from paper_2305_09781_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _dev(x):
    return (torch.from_numpy(np.ascontiguousarray(x)) if isinstance(x, np.ndarray) else x).to(DEV)


def _case(V, B, N, dt, seed, tau=1.2, n_ssm=3, parent=None):
    cfg = wl.Config(96, "walk", "f32", B=B, H=1, D=64, P=1, N=N, tree="random_branching", V=V, n_ssm=n_ssm)
    i = wl.make_verify_inputs(cfg, seed=seed, mode="stochastic", parent=parent, logits_dtype=torch.bfloat16 if dt == "bf16" else torch.float32, tau=tau)
    args = (i["logits"].float().numpy(), i["probs_ssm"].numpy(), i["ssm_row"].numpy(), i["tree_token"].numpy(), i["tree_parent"].numpy())
    ua, uf, _ = vetting.vet_uniforms(*args, i["u_accept"].numpy(), i["u_order"].numpy(), i["u_final"].numpy(), i["rng"])
    ref = orc.verify_stochastic(*args, ua, i["u_order"].numpy(), uf)
    dev = [_dev(x) for x in (i["probs_ssm"], i["ssm_row"], i["tree_token"], i["tree_parent"], ua, i["u_order"], uf)]
    return _dev(i["logits"]), dev, ref


@pytest.mark.parametrize("V,B,N,dt,tau", [(4, 3, 12, "f32", None), (1023, 3, 24, "f32", None), (4096, 3, 24, "bf16", 1.2), (4100, 3, 24, "f32", 2.0),
                                          (8191, 3, 20, "f32", 2.0), (8193, 3, 20, "bf16", 2.0),
                                          (12001, 3, 20, "f32", 2.0), (16383, 3, 20, "bf16", 2.0), (16385, 3, 20, "f32", 2.0),
                                          (16384, 3, 20, "bf16", 2.0), (16388, 3, 20, "f32", 2.0), (32768, 2, 16, "f32", 2.0),
                                          (32767, 2, 16, "bf16", 2.0), (32769, 2, 12, "f32", 1.2), (32772, 2, 16, "f32", 2.0)])
def test_walk_from_given_statistics_and_from_its_own(spec, V, B, N, dt, tau):
    logits, dev, ref = _case(V, B, N, dt, seed=V + N, tau=tau)
    status = torch.zeros(B, dtype=torch.int32, device=DEV)
    got = spec.spec_verify_stochastic(logits, *dev, status=status)      # few rows: statistics before the walk
    for g, r in zip(list(got) + [status], ref):
        assert np.array_equal(g.cpu().numpy(), r)


def _us(call):
    times = []
    for _ in range(5):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        for _ in range(10):
            call()
        end.record()
        torch.cuda.synchronize()
        times.append(start.elapsed_time(end) * 100)
    return sorted(times)[2]


def _own_levels(V, B, N, dt, Lmax):
    """Levels up to which the walk takes a tree's statistics itself (the rule of spec_verify_stochastic)."""
    pass_us = B * N * V * (2 if dt == "bf16" else 4) / 5.5e6
    levels = int(min(pass_us / (V * 0.9e-4), 128))
    return levels if levels >= 8 or levels >= min(Lmax, N) else 0


@pytest.mark.parametrize("V,B,N,dt", [(32000, 16, 72, "f32"), (32003, 16, 80, "f32"), (16384, 16, 100, "f32"), (32768, 16, 128, "bf16"),
                                      (32001, 16, 128, "bf16")])
def test_walk_that_takes_its_own_statistics(spec, V, B, N, dt):
    """Enough rows that the statistics of shallow trees' nodes are left to the walk and those of deeper ones are not; trees of
    both kinds, exactly at the line and one level past it, malformed and padding nodes among them."""
    levels = _own_levels(V, B, N, dt, N)
    assert 8 <= levels < N - 1
    def spine(n):      # a chain of n levels whose other nodes hang on the root
        return np.concatenate([np.arange(-1, n - 1), np.zeros(N - n)]).astype(np.int32)
    rng = np.random.default_rng(V)
    par = np.stack([wl.tree_random_branching(rng, N) for _ in range(B)])
    par[3], par[4], par[5], par[6] = spine(levels), spine(levels + 1), spine(N), spine(2)
    depth = [int(wl.depth_of(p).max()) + 1 for p in par]
    assert min(depth) <= levels < max(depth)
    logits, dev, ref = _case(V, B, N, dt, seed=V, n_ssm=1, tau=2.0, parent=par)
    got = spec.spec_verify_stochastic(logits, *dev)
    for g, r in zip(got, ref):
        assert np.array_equal(g.cpu().numpy(), r)
    # a stated longest path within the levels: no tree needs the pass. (Paths as long as that would be cut: there are none.)
    assert ref[1].max() < levels
    got = spec.spec_verify_stochastic(logits, *dev, Lmax=levels)
    for g, r in zip(got, ref):
        assert np.array_equal(g.cpu().numpy(), r[:, :levels] if r.ndim == 2 else r)
    status = torch.zeros(B, dtype=torch.int32, device=DEV)
    bad = [d.clone() for d in dev]
    bad[3][1, 2] = 5                    # a parent after its child
    bad[2][0, 1:] = -1                  # only padding nodes: the root's own token is drawn
    path, ln, tok = spec.spec_verify_stochastic(logits, *bad, status=status)
    st = status.cpu().numpy()
    assert st[1] == orc.ST_BAD_TREE and ln[1].item() == 0 and (path[1] == -1).all() and (tok[1] == -1).all()
    assert ln[0].item() == 1 and path[0, 0].item() == 0
    for g, r in zip((path, ln, tok), ref):
        assert np.array_equal(g[2:].cpu().numpy(), r[2:])


def test_long_accepted_paths_do_not_wait_for_their_rows(spec):
    """Chains of 128 nodes that are accepted to the end: the call takes no longer than the walk over given statistics and one
    read of all logits at 2.5 TB/s (it reads them once, at twice that), where a walk that takes the statistics of every node
    itself takes three times as long."""
    B, N, V = 16, 128, 32000
    g = torch.Generator(device=DEV).manual_seed(1)
    logits = torch.randn((B, N, V), generator=g, device=DEV)
    tok = torch.randint(0, V, (B, N), generator=g, device=DEV, dtype=torch.int32)
    par = torch.arange(-1, N - 1, dtype=torch.int32, device=DEV).repeat(B, 1).contiguous()
    probs = torch.full((1, V), 1.0 / V, device=DEV)
    row = torch.zeros((B, N), dtype=torch.int32, device=DEV)
    u = torch.zeros((B, N), device=DEV)
    uf = torch.full((B,), 0.5, device=DEV)
    mx = logits.max(-1).values.contiguous()
    se = torch.exp(logits - mx[..., None]).sum(-1).contiguous()
    given = lambda: spec.spec_verify_stochastic_stats(logits, mx, se, probs, row, tok, par, u, u, uf)  # noqa: E731
    whole = lambda: spec.spec_verify_stochastic(logits, probs, row, tok, par, u, u, uf)  # noqa: E731
    for a, b in zip(given(), whole()):
        assert torch.equal(a, b)
    assert (whole()[1] == N).all()

    t_given, t_whole = _us(given), _us(whole)
    assert t_whole < t_given + logits.numel() * 4 / 2.5e6, (t_given, t_whole)


def test_odd_vocabularies_have_registers_of_their_size(spec):
    """Eight rejections over 9001 elements, read one by one, take about as long as over 16384, read in groups of four (1.2 times;
    a form with registers for 32768 elements takes twice as long)."""
    t = []
    for V in (9001, 16384):
        B, N = 4, 9
        logits = torch.randn((B, N, V), generator=torch.Generator(device=DEV).manual_seed(V), device=DEV)
        logits[:, :, :N] = -30.0
        tok = torch.arange(N, dtype=torch.int32, device=DEV).repeat(B, 1).contiguous()
        par = torch.tensor([-1] + [0] * (N - 1), dtype=torch.int32, device=DEV).repeat(B, 1).contiguous()
        probs = torch.full((1, V), 1.0 / V, device=DEV)
        row = torch.zeros((B, N), dtype=torch.int32, device=DEV)
        u = torch.full((B, N), 0.75, device=DEV)
        mx = logits.max(-1).values.contiguous()
        se = torch.exp(logits - mx[..., None]).sum(-1).contiguous()
        out = tuple(torch.empty(s, dtype=torch.int32, device=DEV) for s in ((B, N), (B,), (B, N)))
        ws = torch.empty(8 * B * V + 256, dtype=torch.uint8, device=DEV)
        call = lambda: spec.spec_verify_stochastic_stats(logits, mx, se, probs, row, tok, par, u, u, u[:, 0].contiguous(),  # noqa: E731
                                                         workspace=ws, out=out)
        call()
        assert out[1].tolist() == [1] * B       # every child rejected
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(10):
                call()
        t.append(_us(graph.replay))
    assert t[0] < 1.6 * t[1], t


@pytest.mark.parametrize("V", [1000, 32767, 40001])      # in registers, in a buffer
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_weights_below_the_smallest_normal_number_count(spec, V, dt):
    """exp(-95) is a float32, if not a normal one: a draw at 0 takes the first token that has any weight, by either sampler, and a
    ratio test compares such a probability with a draft's."""
    logits = torch.zeros((1, 2, V), dtype=dt, device=DEV)
    logits[:, :, :3] = float("-inf")
    logits[:, :, 3] = -95.0
    logits[:, :, 4:] = -30.0
    logits[:, :, V // 2] = 0.0
    tok = torch.tensor([[0, 3]], dtype=torch.int32, device=DEV)
    par = torch.tensor([[-1, 0]], dtype=torch.int32, device=DEV)
    row = torch.zeros((1, 2), dtype=torch.int32, device=DEV)
    probs = torch.full((1, V), 1e-42, device=DEV)
    for u, path_want, tok_want in ((0.5, [0, 1], [3, 3]), (1e9, [0, -1], [3, -1])):     # accepted: 0.5e-42 of 5.5e-42; rejected
        path, ln, out = spec.spec_verify_stochastic(logits, probs, row, tok, par, torch.full((1, 2), u, device=DEV),
                                                    torch.zeros((1, 2), device=DEV), torch.zeros(1, device=DEV))
        assert path[0].tolist() == path_want and out[0].tolist() == tok_want
    zero = torch.zeros((1, 2), device=DEV)
    path, ln, out, sample = spec.spec_verify_naive(logits, tok, par, zero)
    assert sample[0].tolist() == [3, 3]


@pytest.mark.parametrize("V", [1000, 40001])
def test_every_step_of_a_long_path_is_in_the_outputs(spec, V):
    """A chain of 128 accepted from given statistics, with nothing to wait for between its steps: the accepted nodes and tokens
    stand over the filling of both outputs, from the first to the last, and the filling stands behind them."""
    B, N, Lmax = 8, 128, 200
    g = torch.Generator(device=DEV).manual_seed(V)
    logits = torch.randn((B, N, V), generator=g, device=DEV)
    tok = torch.randint(0, V, (B, N), generator=g, device=DEV, dtype=torch.int32)
    par = torch.arange(-1, N - 1, dtype=torch.int32, device=DEV).repeat(B, 1).contiguous()
    mx = logits.max(-1).values.contiguous()
    se = torch.exp(logits - mx[..., None]).sum(-1).contiguous()
    zero = torch.zeros((B, N), device=DEV)
    path, ln, out = spec.spec_verify_stochastic_stats(logits, mx, se, torch.full((1, V), 1.0 / V, device=DEV), torch.zeros_like(tok), tok, par,
                                                      zero, zero, torch.full((B,), 0.5, device=DEV), Lmax=Lmax)
    want = torch.full((B, Lmax), -1, dtype=torch.int32, device=DEV)
    want[:, :N] = torch.arange(N, dtype=torch.int32, device=DEV)
    assert (ln == N).all() and torch.equal(path, want)
    assert torch.equal(out[:, :N - 1], tok[:, 1:]) and (out[:, N - 1] >= 0).all() and (out[:, N:] == -1).all()


def _rejections(parent, tok, order, path, ln):
    """Rejections in a row at each node that an accepted path visits: its children tested before the accepted one, or all."""
    out = []
    for k in range(ln):
        kids = sorted((v for v in range(1, len(parent)) if parent[v] == path[k] and tok[v] >= 0), key=lambda v: (order[v], v))
        out.append(kids.index(path[k + 1]) if k + 1 < ln else len(kids))
    return out


@pytest.mark.parametrize("V,B,N,dt,tau,seed", [(50257, 3, 16, "bf16", 2.0, 3), (65539, 3, 16, "f32", 1.2, 2), (128256, 2, 12, "bf16", 2.0, 2),
                                               (65536, 3, 16, "f32", 2.0, 0)])
def test_rejections_of_large_vocabularies(spec, V, B, N, dt, tau, seed):
    """The buffer form with two rejections and more at one node (both residual buffers), over several sweeps of a row."""
    logits, dev, ref = _case(V, B, N, dt, seed=V + seed, tau=tau)
    tok, par, order = (dev[i].cpu().numpy() for i in (2, 3, 5))
    assert max(max(_rejections(par[b], tok[b], order[b], ref[0][b], ref[1][b])) for b in range(B)) >= 2
    status = torch.zeros(B, dtype=torch.int32, device=DEV)
    got = spec.spec_verify_stochastic(logits, *dev, status=status)
    for g, r in zip(list(got) + [status], ref):
        assert np.array_equal(g.cpu().numpy(), r)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("V,rows", [(2048, 60), (2049, 60), (4096, 60), (4097, 60), (8192, 60), (8193, 60), (16384, 60), (16387, 60),
                                    (2047, 1024), (2049, 1024), (4100, 1024), (8193, 1024)])
def test_statistics_at_the_ends_of_sweeps(spec, V, rows, dt):
    """Sweeps of two, four and eight groups a thread, in workgroups of 256 and 1024: walks whose statistics come from the pass
    end in the same tokens as over those that torch takes, the last element the likeliest of a third of the rows."""
    B = rows // 20
    N = rows // B
    g = torch.Generator(device=DEV).manual_seed(V + rows)
    logits = torch.randn((B, N, V), generator=g, device=DEV)
    logits[:, ::3, V - 1] = 9.0
    logits[0, N - 1, : V - 1] = float("-inf")
    logits = logits.to(torch.bfloat16 if dt == "bf16" else torch.float32)
    par = torch.arange(-1, N - 1, dtype=torch.int32, device=DEV).repeat(B, 1).contiguous()
    tok = torch.randint(0, V, (B, N), generator=g, device=DEV, dtype=torch.int32)
    probs = torch.full((1, V), 1.0 / V, device=DEV)
    zero, row = torch.zeros((B, N), device=DEV), torch.zeros((B, N), dtype=torch.int32, device=DEV)
    tok[0, N - 1] = V - 1
    x = logits.double()
    mx = x.max(-1).values
    se = torch.exp(x - mx[..., None]).sum(-1)
    for u in (0.05, 0.5, 0.97):
        # an acceptance test at half and at twice the ratio: decided by the statistics, far from rounding
        q = torch.exp(torch.gather(x[:, :-1], 2, tok[:, 1:, None].long())[..., 0] - mx[:, :-1]) / se[:, :-1] * V
        ua = torch.cat([zero[:, :1], torch.where(torch.rand((B, N - 1), generator=g, device=DEV) < 0.05, 2.0, 0.5) * q.float()], 1)
        args = (probs, row, tok, par, ua.contiguous(), zero, torch.full((B,), u, device=DEV))
        got = spec.spec_verify_stochastic(logits, *args)
        want = spec.spec_verify_stochastic_stats(logits, mx.float().contiguous(), se.float().contiguous(), *args)
        for a, b in zip(got[:2], want[:2]):
            assert torch.equal(a, b)
        assert (got[2] == want[2]).float().mean() > 0.999       # (a draw within rounding of a border)
