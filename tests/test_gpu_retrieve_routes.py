"""The routes of a retrieval at their edges: the selection behind the scores in a launch of its own, up to 32 keys per thread in
registers (a KV head, or all of a sequence), one more, short sequences under a long limit, and the gather list
of a step.  Exact scores, as in test_gpu_retrieve."""
import pytest

from svf_harness import full_parity
from test_gpu_parity import small
from test_gpu_retrieve import BLOCK, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [8193, 9216, 9217, 32768, 32769])
@pytest.mark.parametrize("levels", [2, 100000])
def test_per_head(nb, levels):
    run([nb * BLOCK, 0, 5 * BLOCK, 1025 * BLOCK - 3], 1, nb, min(nb, 1500), 0, levels, seed=nb, n_sink=1, n_local=2)


@pytest.mark.parametrize("Hkv,nb", [(2, 4097), (3, 2731), (9, 1024), (256, 33), (256, 128), (32, 1024), (7, 4681), (1, 32768)])
@pytest.mark.parametrize("levels", [1, 100000])
def test_all_heads(Hkv, nb, levels):
    for total in (1, 3000, Hkv * nb):
        run([nb * BLOCK, 0, max(1, nb * BLOCK // 9)], Hkv, nb, 0, total, levels, G=1, seed=nb + total)


@pytest.mark.parametrize("B,Hkv,nb", [(128, 2, 129), (128, 2, 256), (129, 2, 130), (257, 2, 100), (256, 2, 128), (33, 8, 2048), (33, 8, 2049), (4, 2, 8192)])
def test_many_workgroups(B, Hkv, nb):
    """One launch up to 256 workgroups (512 of one chunk of 128 blocks), the scores and a selection from there, by
    small workgroups for more than 256 heads of up to 2048 blocks."""
    lens = [max(0, nb * BLOCK - 37 * b) for b in range(B)]
    run(lens, Hkv, nb, min(nb, 40), 0, 50, n_sink=1, n_local=1, seed=nb)


@pytest.mark.parametrize("B,Hkv,nb", [(32, 8, 128), (33, 8, 128), (16, 4, 2048), (300, 2, 30)])
def test_many_workgroups_all_heads(B, Hkv, nb):
    run([max(0, nb * BLOCK - 11 * b) for b in range(B)], Hkv, nb, 0, 200, 50, G=1, seed=nb)


def test_step_with_gather_list():
    full_parity(small(T=8200 * 4, block_size=4, page_size=4, k_blocks=40, planted=5, n_sink=1, n_local=1))
