"""How many splits a plan has, and whether they are spread thinly (fp32 partials at d = 128), as the size of its
workspace tells: that the shapes of test_gpu_thin_splits.py are what their names say, and what a plan does where the thin one
would outgrow the static array."""
import pytest

import paper_2512_21911_amd as S
from test_gpu_thin_splits import AT_THE_LIMIT, CASES, THIN, limit_shape

TILE, WAVES = 32, 8


def aligned(n):
    return -(-n // 256) * 256


def planned(shape):
    """(splits, thin) of a bf16 plan of one or two row groups whose pairs share nothing out."""
    pairs, m = shape.B * shape.Hkv, shape.gamma * (shape.Hq // shape.Hkv)
    rows = -(-m // 32) * 32
    groups, nb = pairs * rows // 32, -(-shape.max_seq_len // shape.block_size)
    tokens = shape.k_blocks * shape.block_size
    tiles = -(-tokens // TILE) + -(-shape.gamma // TILE)
    rest = S.svf_workspace_bytes(shape) - aligned(pairs * nb * 4)                    # the scores
    rest -= aligned(groups * 64) + aligned(groups * 8)                               # arrival words, call counters
    if shape.k_blocks <= 1024:
        rest -= aligned(pairs * -(-tokens // TILE) * 8 * 8) if shape.d == 128 else 0  # gather list
        rest -= aligned(groups * nb * 8) if nb <= 1024 else 0                        # exchanged keys
    found = set()
    for row in (256, 512):                               # a partial's bytes, and sixteen for its record
        n, left = divmod(rest, pairs * rows * (row + 16))
        thin = tiles - 1 <= WAVES * (n - 1)
        if left == 0 and row == (512 if thin and shape.d == 128 else 256):
            found.add((n, thin))
    assert len(found) == 1, (rest, found)
    return found.pop()


def shape_of(cfg):
    pages = -(-cfg.T // cfg.page_size) if cfg.page_size else 0
    return S.make_shape(B=cfg.B, gamma=cfg.gamma, Hq=cfg.Hq, Hkv=cfg.Hkv, d=cfg.d, dtype="bf16", block_size=cfg.block_size,
                        max_seq_len=cfg.T, k_blocks=cfg.k_blocks, page_size=cfg.page_size, max_pages_per_seq=pages,
                        kv_strides=((cfg.page_size or cfg.T) * cfg.Hkv * cfg.d, cfg.Hkv * cfg.d, cfg.d))


PLANS = {
    "one_tile_and_the_draft": (1, False),
    "draft_only_splits_empty": (1, False),
    "nine_tiles_one_split": (1, False),
    "seventeen_tiles_eight_splits": (8, True),
    "eighteen_tiles_eight_splits": (8, True),
    "33_tiles_ten_splits_cut_to_eight": (8, True),
    "33_tiles_sixteen_splits": (16, True),
    "34_tiles_seventeenth_split_not_taken": (16, True),
    "129_tiles_full_wavefronts": (16, False),
    "131_tiles_seventeen_splits": (17, False),
    "two_row_groups_sixteen_splits": (16, True),
    "two_draft_tiles": (8, True),
    "ragged_lists_shorter_than_the_plan": (16, True),
    "d64_one_tile_and_the_draft": (1, False),
    "d64_draft_only_splits_empty": (8, True),
    "d64_nine_tiles_eight_splits": (8, True),
    "d64_33_tiles": (8, True),
    "d64_seventeen_tiles_two_row_groups": (8, True),
    "sixteen_splits": (16, True),
    "sixteen_splits_two_row_groups": (16, True),
    "eight_splits": (8, True),
    "four_splits": (4, True),
    "three_splits": (3, True),
    "d64_sixteen_splits": (16, True),
}


@pytest.mark.parametrize("name", sorted({**CASES, **THIN}))
def test_plan_of(name):
    assert planned(shape_of({**CASES, **THIN}[name])) == PLANS[name]


@pytest.mark.parametrize("d,pairs,tokens,plan", [
    (64, 2, 64, (1, False)), (64, 16, 96, (1, False)), (64, 112, 192, (1, False)), (64, 32, 224, (1, False)), (64, 8, 256, (8, True)),
    (64, 48, 256, (5, True)), (64, 64, 256, (4, True)), (64, 80, 256, (1, False)), (64, 112, 256, (1, False)), (64, 80, 288, (3, True)),
    (128, 8, 256, (1, False)), (128, 112, 256, (1, False)), (128, 80, 288, (3, True)),
])
def test_lists_that_one_workgroup_can_take(d, pairs, tokens, plan):
    """Up to eight tiles and the drafts': one split, but for nine tiles at d = 64 that four or more workgroups share."""
    shape = S.make_shape(B=pairs // 2, gamma=4, Hq=8, Hkv=2, d=d, dtype="bf16", block_size=32, max_seq_len=4096, k_blocks=tokens // 32,
                         kv_strides=(4096 * 2 * d, 2 * d, d))
    assert planned(shape) == plan


@pytest.mark.parametrize("d", [64, 128])
def test_plans_at_the_size_of_the_static_array(d):
    """33 tiles of eight pairs: sixteen splits where they fit the array, the four of a tile per wavefront where only
    those do, sixteen where neither does."""
    limit = S.svf_static_workspace_bytes()
    last_thin, last_full = AT_THE_LIMIT[d]
    for nb, plan, fits in ((last_thin, (16, True), True), (last_thin + 8, (4, False), True),
                           (last_full, (4, False), True), (last_full + 8, (16, True), False)):
        shape = limit_shape(d, nb)
        assert planned(shape) == plan and (S.svf_workspace_bytes(shape) <= limit) == fits, nb
