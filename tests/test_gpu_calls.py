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


class Holder:
    """Memory of a tensor behind the three things a call asks of one."""

    def __init__(self, t):
        self.t, self.shape = t, t.shape

    def data_ptr(self):
        return self.t.data_ptr()

    def numel(self):
        return self.t.numel()


def test_objects_with_a_data_pointer():
    class MyShape(S.SvfShape):
        pass

    cfg = small(T=256)
    run = DeviceRun(cfg, to_gpu(W.make_layer(cfg)))
    run.block_reps().score_select().sync()
    reps, idx = run.reps.clone(), run.sel_idx.clone()
    run.reps.fill_(float("nan"))
    run.sel_idx.fill_(-7)
    x = run.x
    shape = MyShape.from_buffer_copy(run.shape)
    S.svf_block_reps(shape, Holder(x["k_pool"]), Holder(x["block_table"]), x["seq_lens"], Holder(run.reps))
    S.svf_score_select(shape, Holder(x["q"]), run.reps, x["seq_lens"], Holder(run.sel_idx), run.sel_cnt, Holder(run.ws))
    w = torch.rand(5, 4, device="cuda") + 0.1
    beta = torch.tensor([0.2, 0.4, 0.6], device="cuda")
    n, keep, n1, keep1 = (torch.full((5,), -1, dtype=torch.int32, device="cuda") for _ in range(4))
    S.svf_moe_skip(w, 2, beta, n, keep)
    S.svf_moe_skip(Holder(w), 2, Holder(beta), Holder(n1), Holder(keep1))
    torch.cuda.synchronize()
    assert torch.equal(torch.nan_to_num(run.reps), torch.nan_to_num(reps)) and torch.equal(run.sel_idx, idx)
    assert torch.equal(n, n1) and torch.equal(keep, keep1)
