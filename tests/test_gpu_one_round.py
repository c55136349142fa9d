"""Attention over as many splits as are resident at once, against the CPU oracle: numbers of (sequence, KV head) pairs
that fill the compute units unevenly, with the retrieval alone (svf_score_select, which keeps its own number of
workgroups) and all step modes on one workspace: full_parity() asks for the same blocks and the same bits."""
import pytest

from svf_harness import full_parity
from test_gpu_parity import small

pytestmark = pytest.mark.gpu

CASES = {
    # splits for 256 compute units over the groups, rounded up -> as many as an XCD holds at once
    "pairs_24_11_to_10": small(B=3, Hq=8, Hkv=8, gamma=3, T=3000, k_blocks=44, min_len=900),
    "pairs_20_two_row_groups_7_to_5": small(B=5, Hq=16, Hkv=4, gamma=10, T=1800, k_blocks=27),
    "pairs_28_grows_a_tile_5_to_4": small(B=7, Hq=28, Hkv=4, gamma=6, T=1500, k_blocks=17, page_size=0),
    "pairs_80_two_to_one": small(B=5, Hq=64, Hkv=16, gamma=9, T=600, k_blocks=8),
    "pairs_9_just_past_one_per_xcd": small(B=9, Hq=2, Hkv=1, gamma=2, T=8000, k_blocks=120),
    "pairs_48_least_splits_do_not_fit": small(B=6, Hq=32, Hkv=8, gamma=10, T=2200, k_blocks=33, min_len=300),
    "rows_48_6_to_5": small(B=6, Hq=32, Hkv=8, gamma=20, tree_depth=5, T=600, k_blocks=8, min_len=100),
    "rows_1_pair_66_to_32": small(B=1, Hq=8, Hkv=1, gamma=12, T=2200, k_blocks=33),
    "rows_3_pairs_d64_86_to_32": small(B=3, Hq=8, Hkv=1, d=64, gamma=12, T=4200, k_blocks=64),
    "pairs_24_d64_11_to_10": small(B=3, Hq=8, Hkv=8, d=64, gamma=3, T=3000, k_blocks=44, min_len=900),
    "pairs_20_d64_two_row_groups_7_to_5": small(B=5, Hq=16, Hkv=4, d=64, gamma=10, T=1800, k_blocks=27),
    "pairs_80_d64_two_to_one": small(B=5, Hq=64, Hkv=16, d=64, gamma=9, T=600, k_blocks=8),
    "rows_48_d64_6_to_5": small(B=6, Hq=32, Hkv=8, d=64, gamma=20, tree_depth=5, T=600, k_blocks=8, min_len=100),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_one_round(name):
    r = full_parity(CASES[name])
    print(f"[one round] {name}: max_abs_err={r['max_abs_err']:.3e} near_ties={r['near_ties']}", flush=True)
