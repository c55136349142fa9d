"""Argument forms of the native calls: a mode is whatever int() takes, a workspace counts in elements."""
import pytest
import torch

import paper_2512_21911_amd as S
import workloads as W
from svf_harness import DeviceRun, to_gpu
from test_gpu_parity import small

pytestmark = pytest.mark.gpu


def test_modes_and_workspaces_of_other_types():
    cfg = small(T=256)
    run = DeviceRun(cfg, to_gpu(W.make_layer(cfg)))
    run.block_reps().verify_step(S.SVF_STEP_ANCHOR).sync()
    out = run.out.clone()
    for mode in (float(S.SVF_STEP_ANCHOR), str(S.SVF_STEP_ANCHOR)):
        run.out.fill_(float("nan"))
        run.verify_step(mode).sync()
        assert torch.equal(run.out, out)
    with pytest.raises(ValueError):
        run.verify_step("anchor")
    with pytest.raises(OverflowError):
        run.verify_step(1 << 40)
    run.ws = run.ws.view(torch.float32)                   # a quarter of the elements: refused, nothing is launched
    with pytest.raises(S.SvfError):
        run.verify_step(S.SVF_STEP_ANCHOR)
