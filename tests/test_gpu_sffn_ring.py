"""The joint gate / up walks over their rings of stages, against the fp64 oracle, the same bits call after call.

Which walk a size takes: up to 2048 hidden channels the split kernel with 8 channels per workgroup; up to 4096
(more than 32 tokens: 8192) with 16; beyond that the fused walk, with one tile per workgroup (up to 32 tokens
and 8192 channels as a rule) or two.  Its stages: split 8 / 8 / 6 / 3 (8 channels) and 7 / 6 / 4 / 3 (16) for up
to 8 / 16 / 32 / 64 tokens, a chunk of 64 dimensions of every fourth chunk each; fused 7 (6 for more
than 32 tokens) chunks, or 6 pairs of chunks with one tile."""
import numpy as np
import pytest

import workloads.ffn as WF
from test_gpu_sffn import WALKS, check, run_gpu

pytestmark = pytest.mark.gpu


def same_bits_each_time(M, d_model, d_ff):
    cfg = WF.FFN_CONFIGS[1].scaled(M=M, d_model=d_model, d_ff=d_ff)
    w = WF.make_ffn(cfg)
    y, act = check(cfg, w, walk=WALKS["together"])
    for _ in range(2):
        y1, act1 = run_gpu(cfg, w, walk=WALKS["together"])
        assert np.array_equal(y, y1) and np.array_equal(act, act1)


@pytest.mark.parametrize("M", [1, 32, 33, 64])
@pytest.mark.parametrize("d_model,d_ff", [(128, 32), (384, 64), (512, 544), (896, 8224), (256, 14368)])
def test_ring(d_model, d_ff, M):
    """Few chunks and few channels (split kernel), then hidden sizes whose tile is cut below 32 channels, with a last
    tile moved back and an odd number of tiles: every channel is written once."""
    same_bits_each_time(M, d_model, d_ff)


@pytest.mark.parametrize("M,stages", [(8, 8), (9, 8), (16, 8), (17, 6), (32, 6), (33, 3), (64, 3)])
@pytest.mark.parametrize("turns", ["one_less", "full", "one_more", "twice"])
def test_split_ring_of_eight_channels(M, stages, turns):
    """Chunks per wavefront around the number of its stages (the last wavefronts have one less where the
    dimension is no multiple of four chunks)."""
    per_wave = {"one_less": stages - 1, "full": stages, "one_more": stages + 1, "twice": 2 * stages + 1}[turns]
    same_bits_each_time(M, 256 * per_wave - 128, 96)


@pytest.mark.parametrize("M,stages", [(8, 7), (16, 6), (32, 4), (33, 3), (64, 3)])
@pytest.mark.parametrize("extra", [-1, 0, 1])
def test_split_ring_of_sixteen_channels(M, stages, extra):
    same_bits_each_time(M, 256 * (stages + extra), 2080)


@pytest.mark.parametrize("M,d_ff", [(17, 4096), (60, 8192), (9, 2048)])
def test_split_at_its_largest(M, d_ff):
    same_bits_each_time(M, 1152, d_ff)


@pytest.mark.parametrize("M", [3, 32])
@pytest.mark.parametrize("d_model,d_ff", [(d, f) for f in (4128, 7200, 8192) for d in (128, 640, 768, 896, 1664)] + [(768, 16896)])
def test_fused_ring_of_one_tile(d_model, d_ff, M):
    """1, 5 .. 7 and 13 pairs of chunks through 6 stages; tiles of 20, 32 (a last one moved back; none) and, where
    it fills its rounds better than two, 24 channels."""
    same_bits_each_time(M, d_model, d_ff)


@pytest.mark.parametrize("M", [5, 40])
@pytest.mark.parametrize("d_model", [256, 384, 512, 1024])
def test_fused_ring_of_two_tiles(d_model, M):
    """4, 6, 8 and 16 chunks through 7 stages (6 for 40 tokens)."""
    same_bits_each_time(M, d_model, 9248)
