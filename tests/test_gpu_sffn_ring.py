"""The joint gate / up walk over its ring of stages: fewer chunks than stages, as many, one more; hidden
sizes whose tile is cut below 32 channels, with a last tile moved back and an odd number of tiles: every
channel is written once, the same bits call after call."""
import numpy as np
import pytest

import workloads.ffn as WF
from test_gpu_sffn import WALKS, check, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 32, 33, 64])
@pytest.mark.parametrize("d_model,d_ff", [(128, 32), (384, 64), (512, 544), (896, 8224), (256, 14368)])
def test_ring(d_model, d_ff, M):
    cfg = WF.FFN_CONFIGS[1].scaled(M=M, d_model=d_model, d_ff=d_ff)
    w = WF.make_ffn(cfg)
    y, act = check(cfg, w, walk=WALKS["together"])
    for _ in range(2):
        y1, act1 = run_gpu(cfg, w, walk=WALKS["together"])
        assert np.array_equal(y, y1) and np.array_equal(act, act1)
