"""The binding's native marshalling on CPU tensors: descriptors field by field, and what is refused before anything is
launched (no call here reaches a kernel)."""
import ctypes
import types

import numpy as np
import pytest
import torch

from paper_2305_09781_amd import binding as spec

STREAM = types.SimpleNamespace(cuda_stream=0)


def _fields(d):
    return {n: getattr(d, n) for n, *_ in d._fields_}


def test_descriptors_field_by_field():
    q = torch.zeros(2, 5, 8, 128, dtype=torch.bfloat16).transpose(1, 2).contiguous().transpose(1, 2)   # head-major
    kc = torch.zeros(2, 4, 100, 64 + 64, dtype=torch.bfloat16)[:, 1:3]
    kn = torch.zeros(2, 5, 2, 128, dtype=torch.bfloat16)
    d = _fields(spec.make_desc(q, kc, np.int64(90), 0.5, k_new=kn, plan=[64, np.int32(-1), 2]))
    assert d == {"B": 2, "H": 8, "H_kv": 2, "D": 128, "N": 5, "S_cap": 100, "dtype": spec.SPEC_BF16, "max_prefix_len": 90,
                 "q_stride_b": 5120, "q_stride_n": 128, "q_stride_h": 640, "kv_stride_b": 51200, "kv_stride_h": 12800,
                 "kv_stride_s": 128, "new_stride_b": 1280, "new_stride_n": 256, "new_stride_h": 128, "softmax_scale": 0.5,
                 "plan_chunk_keys": 64, "plan_balanced_wgs": -1, "plan_heads_per_wg": 2}
    for plan in (torch.tensor([64, -1, 2]), {0: 64, 1: -1, 2: 2}, np.array([64, -1, 2]), (64.0, -1.0, 2.5)):   # whatever plan[0..2] gives
        p = _fields(spec.make_desc(q, kc, plan=plan))
        assert (p["plan_chunk_keys"], p["plan_balanced_wgs"], p["plan_heads_per_wg"]) == (64, -1, 2)
    pool, table = torch.zeros(7, 2, 64, 128), torch.zeros(3, 4, dtype=torch.int32)
    d, p = spec.make_paged_desc(torch.zeros(3, 5, 2, 128), pool, table)
    assert (d.S_cap, d.dtype, d.new_stride_b, d.max_prefix_len) == (256, spec.SPEC_F32, 0, 0)
    assert (p.block_table, p.max_blocks, p.block_tokens, p.n_blocks) == (table.data_ptr(), 4, 64, 7)


def _attention(**kw):
    B, N, H, D, S = 1, 4, 2, 64, 32
    i32 = lambda *s: torch.zeros(s, dtype=torch.int32)  # noqa: E731
    a = dict(q=torch.zeros(B, N, H, D), k_new=torch.zeros(B, N, H, D), v_new=torch.zeros(B, N, H, D), k_cache=torch.zeros(B, H, S, D),
             v_cache=torch.zeros(B, H, S, D), tree_parent=i32(B, N), tree_depth=i32(B, N), prefix_len=i32(B), stream=STREAM)
    a.update(kw)
    return a


def _rope(**kw):
    return _attention(rope_cos=torch.zeros(32, 32), rope_sin=torch.zeros(32, 32), **kw)


@pytest.mark.parametrize("call,error", [
    (lambda: spec.spec_tree_attention_append(**_attention(k_new=None)), TypeError),
    (lambda: spec.spec_tree_attention_append(**_attention(v_cache=torch.zeros(1, 2, 16, 64))), ValueError),
    (lambda: spec.spec_tree_attention_append(**_attention(v_new=torch.zeros(1, 2, 4, 64).transpose(1, 2))), ValueError),
    (lambda: spec.spec_tree_attention_append(**_attention(out=torch.zeros(1, 4, 2, 64, dtype=torch.float16))), ValueError),
    (lambda: spec.spec_tree_attention_append(**_attention(q=np.zeros(3))), TypeError),
    (lambda: spec.spec_tree_attention_append(**_attention(desc=3)), TypeError),
    (lambda: spec.spec_tree_attention_append(**_attention(desc=spec.KvPages())), ctypes.ArgumentError),
    (lambda: spec.spec_tree_attention_append(**_attention(desc=ctypes.pointer(spec.AttnDesc()))), ctypes.ArgumentError),
    (lambda: spec.spec_tree_attention_append_static(**_attention(desc=ctypes.c_int(3), out=torch.zeros(1, 4, 2, 64))), ctypes.ArgumentError),
    (lambda: spec.spec_tree_attention(**{k: v for k, v in _attention(desc=spec.KvPages()).items() if "new" not in k}), ctypes.ArgumentError),
    (lambda: spec.spec_tree_attention_append(**_attention(max_prefix_len=29)), spec.SpecError),
    (lambda: spec.spec_tree_attention_append_static(**_attention(out=None)), TypeError),
    (lambda: spec.spec_tree_attention_append_rope(**{**_rope(), "rope_cos": None}), TypeError),
    (lambda: spec.spec_tree_attention_append_rope(**{**_rope(), "rope_sin": torch.zeros(32, 33)}), ValueError),
    (lambda: spec.spec_tree_attention_append_rope(**_rope()), spec.SpecError),                       # float32: unsupported
    (lambda: spec.spec_tree_attention_append_rope(**_rope(block_table=torch.zeros(1, 4))), ValueError),
    (lambda: spec.spec_tree_attention_paged(*[_attention()[k] for k in ("q", "k_cache", "v_cache")], None, *[None] * 3), TypeError),
    (lambda: spec.make_desc(torch.zeros(1, 4, 2, 64, dtype=torch.float16), torch.zeros(1, 2, 8, 64)), TypeError),
    (lambda: spec.make_desc(torch.zeros(4, 2, 64), torch.zeros(1, 2, 8, 64)), ValueError),
    (lambda: spec.spec_verify_greedy(torch.zeros(1, 200, 8), torch.zeros(1, 200), torch.zeros(1, 200), stream=STREAM), spec.SpecError),
    (lambda: spec.spec_verify_greedy(torch.zeros(1, 2, 8), torch.zeros(1, 2), torch.zeros(1, 2), Lmax=2.0), ctypes.ArgumentError),
    (lambda: spec.spec_verify_greedy(torch.zeros(1, 2, 8), torch.zeros(1, 2), torch.zeros(1, 2), out=(1, 2)), ValueError),
    (lambda: spec.spec_verify_greedy(torch.zeros(1, 2, 8), torch.zeros(1, 2), torch.zeros(1, 2), out=(None,) * 4, stream=STREAM),
     spec.SpecError),
    (lambda: spec.spec_verify_stochastic(torch.zeros(1, 2, 8), torch.zeros(3, 7), *[torch.zeros(2)] * 6), ValueError),
    (lambda: spec.spec_verify_stochastic_stats(torch.zeros(1, 2, 8), None, None, torch.zeros(3, 8), *[torch.zeros(2)] * 6), ValueError),
    (lambda: spec.spec_verify_stochastic(torch.zeros(1, 2, 8), torch.zeros(3, 8), *[torch.zeros(2)] * 6, temperature=-1.0, stream=STREAM),
     spec.SpecError),
    (lambda: spec.spec_tree_expand_topk(torch.zeros(1, 2, 8), 2, torch.zeros(2, 3, dtype=torch.int32), torch.zeros(1, 4, dtype=torch.int32)),
     ValueError),
    (lambda: spec.spec_tree_expand_topk(torch.zeros(1, 2, 8), 9, torch.zeros(2, 9, dtype=torch.int32), torch.zeros(1, 4, dtype=torch.int32),
                                        stream=STREAM), spec.SpecError),
    (lambda: spec.spec_tree_merge(torch.zeros(1, 2, 3), torch.zeros(1, 2, 3), torch.zeros(1, 2), 4), ValueError),
    (lambda: spec.spec_lm_head_argmax(torch.zeros(2, 256), torch.zeros(8, 256)), ValueError),
    (lambda: spec.spec_lm_head_logits_stats(torch.zeros(2, 128, dtype=torch.bfloat16), torch.zeros(8, 128, dtype=torch.bfloat16),
                                            stream=STREAM), spec.SpecError),
    (lambda: spec.spec_verify_greedy_lm_head(torch.zeros(2, 256, dtype=torch.bfloat16), torch.zeros(8, 256, dtype=torch.bfloat16),
                                             torch.zeros(1, 3), torch.zeros(1, 3)), ValueError),
    (lambda: spec.spec_kv_commit([], [], torch.zeros(1, 2), torch.zeros(1), torch.zeros(1), 2), IndexError),
    (lambda: spec.spec_kv_commit([torch.zeros(1, 2, 8, 64)], [torch.zeros(1, 2, 9, 64)], torch.zeros(1, 2), torch.zeros(1), torch.zeros(1), 2),
     ValueError),
    (lambda: spec.spec_kv_commit([torch.zeros(1, 2, 8, 64)] * 2, [torch.zeros(1, 2, 8, 64)], torch.zeros(1, 2), torch.zeros(1), torch.zeros(1),
                                 2, stream=STREAM), spec.SpecError),
    (lambda: spec.spec_kv_commit_paged([torch.zeros(1, 2, 64, 64)], [torch.zeros(1, 2, 64, 64)], None, torch.zeros(1, 2), torch.zeros(1),
                                       torch.zeros(1), 2), TypeError),
])
def test_what_is_refused_before_a_launch(call, error):
    with pytest.raises(error):
        call()


def test_another_torch_is_a_message(monkeypatch):
    """The module is bound to one Python and one torch, its name says which, and their absence is an error that says so."""
    monkeypatch.setattr(spec, "_marshal", None)
    monkeypatch.setattr(torch, "__version__", "1.0")
    with pytest.raises(RuntimeError, match="torch-1.0.so not found.*one Python and one torch"):
        spec.make_desc(torch.zeros(1, 4, 2, 64), torch.zeros(1, 2, 8, 64))
