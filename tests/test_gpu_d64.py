"""The matrix-core kernels at head dimension 64 (K and V row of a token side by side in LDS, fp32
partials), against the CPU oracle, at the sizes where their tiles, splits and row groups have edges,
and bit for bit whatever the workgroups' waits for each other do."""
import pytest
import torch

import paper_2512_21911_amd as S
import workloads as W
from svf_harness import DeviceRun, full_parity, to_gpu
from test_gpu_parity import same_bits_whatever_the_wait, small

pytestmark = pytest.mark.gpu

D64 = {
    "one_tile": small(d=64, B=1, gamma=1, k_blocks=1, T=70, block_size=32),
    "ragged_tail_contiguous": small(d=64, T=999, min_len=37, page_size=0, k_blocks=7),
    "two_row_groups": small(d=64, Hq=16, gamma=7, n_sink=1, n_local=1),
    "two_draft_tiles": small(d=64, Hq=2, gamma=40),
    "several_tiles_per_wavefront": small(d=64, B=4, Hq=32, Hkv=16, gamma=7, T=8192, k_blocks=60, min_len=3000),
    "one_split": small(d=64, B=16, Hq=32, Hkv=16, gamma=3, T=1024, k_blocks=4),
    "more_than_16_splits": small(d=64, B=1, Hq=4, Hkv=1, T=20000, k_blocks=150, min_len=15000),
    "blocks_768": small(d=64, B=1, Hq=4, Hkv=1, T=49152, k_blocks=24, planted=5, min_len=40000),
    "two_retrieval_kernels": small(d=64, B=1, Hq=4, Hkv=1, T=32768, block_size=16, k_blocks=40, planted=6),
    "rows_tree24": small(d=64, gamma=24, tree_depth=5),
    "rows_ring_of_stages": small(d=64, B=8, Hq=32, Hkv=8, gamma=24, T=4096, k_blocks=32, tree_depth=4, min_len=3000),
    "rows_single_split": small(d=64, B=32, Hq=32, Hkv=8, gamma=20, T=1024, k_blocks=4),
    "rows_two_sets_of_eight": small(d=64, B=1, Hq=16, Hkv=2, gamma=64, T=2048, k_blocks=8),
    "rows_merged_behind": small(d=64, B=1, Hq=24, Hkv=1, gamma=4, T=8192, k_blocks=100),
}


@pytest.mark.parametrize("name", sorted(D64))
def test_d64(name):
    r = full_parity(D64[name])
    print(f"[d64] {name}: max_abs_err={r['max_abs_err']:.3e} near_ties={r['near_ties']}", flush=True)


@pytest.mark.parametrize("name", ["ragged_tail_contiguous", "several_tiles_per_wavefront", "rows_tree24"])
def test_d64_same_bits_whatever_the_workgroups_wait_for_each_other(name):
    same_bits_whatever_the_wait(D64[name])


@pytest.mark.parametrize("name", ["ragged_tail_contiguous", "several_tiles_per_wavefront", "rows_tree24"])
def test_d64_gather_mode_relies_on_its_arguments_alone(name):
    """A selection that no anchor call made, a workspace that no call has used: SVF_STEP_REUSE_GATHER of a
    shape without a gather list is SVF_STEP_REUSE, bit for bit."""
    cfg = D64[name]
    run = DeviceRun(cfg, to_gpu(W.make_layer(cfg)))
    run.block_reps().score_select().verify_step(S.SVF_STEP_REUSE).sync()
    out, lse = run.out.clone(), run.lse.clone()
    run.ws = S.new_workspace(run.shape)
    run.out.fill_(float("nan"))
    run.lse.fill_(float("nan"))
    run.verify_step(S.SVF_STEP_REUSE_GATHER).sync()
    assert torch.equal(run.out.view(torch.int16), out.view(torch.int16))
    assert torch.equal(run.lse.view(torch.int32), lse.view(torch.int32))
