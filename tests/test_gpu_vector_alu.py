"""The fp32 attention kernel (which took over from one on the vector ALU) and its merge against the CPU oracle: both types
and head dimensions, a single split, one and two trips of eight splits, several tiles per wavefront, two draft
tiles, blocks that are no multiple of four tokens."""
import pytest

from svf_harness import full_parity
from test_gpu_parity import small

pytestmark = pytest.mark.gpu

CASES = {
    "one_row_one_block": small(dtype="f32", d=64, B=1, Hq=1, Hkv=1, gamma=1, T=50, block_size=16, k_blocks=1),
    "one_split_several_tiles": small(dtype="f32", B=32, Hq=32, Hkv=16, T=256, gamma=3, min_len=30),
    "splits_8": small(dtype="f32", d=64, B=1, Hq=4, Hkv=1, T=2048, block_size=32, k_blocks=15),
    "splits_8_contiguous": small(dtype="f32", B=1, Hq=4, Hkv=1, T=2000, block_size=32, k_blocks=16, page_size=0),
    "splits_16": small(dtype="f32", B=1, Hq=4, Hkv=1, T=8000, k_blocks=50),
    "two_draft_tiles": small(dtype="f32", d=64, B=1, gamma=40, tree_depth=5),
    "bf16_block_6": small(B=2, T=600, block_size=6, page_size=6, k_blocks=20, min_len=200),
    "bf16_block_130_d64": small(d=64, T=1300, block_size=130, page_size=26, k_blocks=4, min_len=700),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_vector_alu(name):
    r = full_parity(CASES[name])
    print(f"[vector ALU] {name}: max_abs_err={r['max_abs_err']:.3e} near_ties={r['near_ties']}", flush=True)
