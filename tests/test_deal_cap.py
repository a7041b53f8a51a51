"""The deal's number of workgroups, from the size of the partials it asks for: partials up to three fifths of the K/V stream as long
as they fit the library's own scratch array, a quarter of the stream where that is more."""
import pytest

from paper_2305_09781_amd import binding as b
from test_balanced_deal import query_groups

SCRATCH = 64 << 20


def _need(B, H, H_kv, D, N, P, wgs=0):
    d = b.AttnDesc(B, H, H_kv, D, N, P + N + 8, 1, P, N * H * D, H * D, D, H_kv * (P + N + 8) * D, (P + N + 8) * D, D,
                   N * H_kv * D, H_kv * D, D, 0.0, 0, wgs, 0)
    return b.spec_tree_attention_workspace_bytes(d)


@pytest.mark.parametrize("B,H,H_kv,N,P,cut_more", [
    (2, 64, 8, 128, 16000, True),     # a quarter of the stream: fewer than two chunks per pair
    (2, 64, 8, 120, 16000, True),
    (3, 64, 8, 100, 16000, False),    # the quarter itself exceeds the scratch array
    (3, 64, 8, 128, 16000, False),
    (2, 64, 8, 64, 16000, False),     # the device's 512 workgroups are fewer than a quarter allows
])
def test_partials_and_the_scratch_array(B, H, H_kv, N, P, cut_more):
    D, n_qg = 128, query_groups(H, H_kv, N)
    heads_per_wg = -(-(H // H_kv) // n_qg)      # a group's partials are those of its own heads only
    quarter = int(0.25 * (B * H_kv * (P + N) * D * 4) / (2.0 * heads_per_wg * N * (D + 2) * 4))
    need, at_quarter = _need(B, H, H_kv, D, N, P), _need(B, H, H_kv, D, N, P, min(quarter, 512))
    assert need <= max(SCRATCH, at_quarter)
    assert (need > at_quarter) == cut_more, (need, at_quarter)
