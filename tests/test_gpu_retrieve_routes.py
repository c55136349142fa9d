"""The selection behind the scores in a launch of its own, at the edges of its routes: up to 32 keys per thread in
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


def test_step_with_gather_list():
    full_parity(small(T=8200 * 4, block_size=4, page_size=4, k_blocks=40, planted=5, n_sink=1, n_local=1))
