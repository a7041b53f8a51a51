"""The stochastic walk over the vocabulary sizes where its form changes (rows of whole 16-byte groups or not, one to
eight groups per thread, the buffer form), with the nodes' statistics taken by the walk or before it, against the oracle on vetted
uniforms: bit-exact paths, lengths, tokens and status."""
import ctypes

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


def _case(V, B, N, dt, seed, tau=1.2, n_ssm=3):
    cfg = wl.Config(96, "walk", "f32", B=B, H=1, D=64, P=1, N=N, tree="random_branching", V=V, n_ssm=n_ssm)
    i = wl.make_verify_inputs(cfg, seed=seed, mode="stochastic", logits_dtype=torch.bfloat16 if dt == "bf16" else torch.float32, tau=tau)
    args = (i["logits"].float().numpy(), i["probs_ssm"].numpy(), i["ssm_row"].numpy(), i["tree_token"].numpy(), i["tree_parent"].numpy())
    ua, uf, _ = vetting.vet_uniforms(*args, i["u_accept"].numpy(), i["u_order"].numpy(), i["u_final"].numpy(), i["rng"])
    ref = orc.verify_stochastic(*args, ua, i["u_order"].numpy(), uf)
    dev = [_dev(x) for x in (i["probs_ssm"], i["ssm_row"], i["tree_token"], i["tree_parent"], ua, i["u_order"], uf)]
    return _dev(i["logits"]), dev, ref


@pytest.mark.parametrize("V,B,N,dt,tau", [(4, 3, 12, "f32", None), (1023, 3, 24, "f32", None), (4096, 3, 24, "bf16", 1.2), (4100, 3, 24, "f32", 2.0),
                                          (8191, 3, 20, "f32", 2.0), (8193, 3, 20, "bf16", 2.0),
                                          (16384, 3, 20, "bf16", 2.0), (16388, 3, 20, "f32", 2.0), (32768, 2, 16, "f32", 2.0),
                                          (32767, 2, 16, "bf16", 2.0), (32769, 2, 12, "f32", 1.2), (32772, 2, 16, "f32", 2.0)])
def test_walk_from_given_statistics_and_from_its_own(spec, V, B, N, dt, tau):
    logits, dev, ref = _case(V, B, N, dt, seed=V + N, tau=tau)
    status = torch.zeros(B, dtype=torch.int32, device=DEV)
    got = spec.spec_verify_stochastic(logits, *dev, status=status)      # few rows: statistics before the walk
    for g, r in zip(list(got) + [status], ref):
        assert np.array_equal(g.cpu().numpy(), r)


@pytest.mark.parametrize("V,B,N,dt", [(32000, 16, 50, "f32"), (32003, 16, 52, "f32"), (16384, 16, 100, "f32"), (32768, 16, 96, "bf16")])
def test_walk_that_takes_its_own_statistics(spec, V, B, N, dt):
    """Enough rows that the nodes' statistics are left to the walk; malformed and padding nodes among them."""
    logits, dev, ref = _case(V, B, N, dt, seed=V, n_ssm=1, tau=2.0)
    got = spec.spec_verify_stochastic(logits, *dev)
    for g, r in zip(got, ref):
        assert np.array_equal(g.cpu().numpy(), r)
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
