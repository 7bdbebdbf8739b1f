"""dX with its two products in tiles of their own, which meet where the second of them is done: short batches.  Both tiles, cut
rows and columns, ragged K, both scaling recipes and output types; every element against binary64 on the device (the bar of
every contraction: 2e-3 of the largest element), and the same bits whichever product comes first."""
import os
import subprocess
import sys

import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

import paper_2409_12517_amd as ssg  # noqa: E402
import gpu_util as gu  # noqa: E402
import test_gpu_grouping as tgr  # noqa: E402
import test_gpu_mlp as tm  # noqa: E402
import test_gpu_paths as tp  # noqa: E402

# less than one small tile, small tiles with every edge cut, and 65 large ones with a ragged last K step
SHAPES = [(16, 80, 784, 128), (272, 304, 1040, 128), (384, 512, 1408, 128), (1168, 3088, 2064, 256)]


@pytest.mark.parametrize("T,d,f,tile", SHAPES)
@pytest.mark.parametrize("mode", [ssg.SSG_SCALE_CURRENT, ssg.SSG_SCALE_DELAYED])
def test_dx_in_halves(T, d, f, tile, mode):
    state = torch.empty(ssg.ssg_mlp_scaling_state_bytes(), dtype=torch.uint8, device=gu.DEV)
    ssg.ssg_mlp_scaling_init(state)
    kw = dict(scaling_state=state, keep_bf16_grads=int(mode == ssg.SSG_SCALE_DELAYED))
    blk = tp._training(T, d, f, **kw)
    blk.fwd()
    blk.bwd()                                             # current scaling: fills the history
    blk.desc = ssg.make_desc(T, d, f, y_dtype=ssg.SSG_F32, scale_mode=mode, **kw)
    p = ssg.ssg_mlp_gemm_plan(blk.desc, ssg.SSG_PLAN_BWD_SECOND)
    assert (p.tile, p.launches) == (tile, 1)
    assert ssg.ssg_mlp_gemm_route(blk.desc, ssg.SSG_PLAN_BWD_SECOND).dx_form == ssg.SSG_DX_HALVES
    blk.fwd()
    first = None
    for _ in range(4):
        for t in (blk.dx, blk.dW1, blk.dW2, blk.dW3):
            t.fill_(float("nan"))
        blk.work.fill_(0x7F)                              # nothing of an earlier call is counted on
        saved_state = state.clone()
        blk.bwd()
        state.copy_(saved_state)                          # the same scales again
        if first is None:
            first = blk.dx.clone()
            tp._check_backward(blk, mode == ssg.SSG_SCALE_DELAYED)
        assert torch.equal(first.view(torch.int32), blk.dx.view(torch.int32))


# more halves than an XCD has compute units for, so that some share one and leave their results while it stores others
@pytest.mark.parametrize("T,d,f", [(2688, 608, 2272), (640, 3456, 12800), (896, 3072, 10240)])
def test_dx_in_halves_with_compute_units_shared(T, d, f):
    blk = tp._training(T, d, f)
    blk.desc = ssg.make_desc(T, d, f, y_dtype=ssg.SSG_F32)
    assert ssg.ssg_mlp_gemm_plan(blk.desc, ssg.SSG_PLAN_BWD_SECOND).tile == 128
    assert ssg.ssg_mlp_gemm_route(blk.desc, ssg.SSG_PLAN_BWD_SECOND).dx_form == ssg.SSG_DX_HALVES
    blk.fwd()
    blk.bwd()
    tp._check_backward(blk, False)
    first = blk.dx.clone()
    for _ in range(40):
        blk.dx.fill_(float("nan"))
        blk.bwd()
        assert torch.equal(first.view(torch.int32), blk.dx.view(torch.int32))


def test_dx_in_halves_in_bf16_and_on_its_own(tmp_path):
    """bf16 dX from the same sum; and launched without the weight gradients (the switch that takes the groups apart), the
    same bits."""
    for shape in ((272, 304, 1040), (1168, 3088, 2064)):
        desc = ssg.make_desc(*shape)
        assert ssg.ssg_mlp_gemm_route(desc, ssg.SSG_PLAN_BWD_SECOND).dx_form == ssg.SSG_DX_HALVES
        blk = tm.Block(synth.make_inputs(*shape, seed=tgr.SEED), y_dtype=ssg.SSG_F32)
        blk.fwd()
        blk.bwd()
        old, tgr.SHAPE = tgr.SHAPE, shape
        try:
            grouped = tgr.run_block()
        finally:
            tgr.SHAPE = old
        assert torch.equal(grouped["dx"], blk.dx.to(torch.bfloat16))
        path = str(tmp_path / "single.pt")
        code = tgr.CHILD.format(root=tgr.ROOT, tests=os.path.join(tgr.ROOT, "tests"), path=path).replace(
            "out = tg.run_block()", f"tg.SHAPE = {shape}; out = tg.run_block()")
        r = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, SSG_GEMM_GROUPING="0"), capture_output=True, text=True, timeout=300)
        assert r.returncode == 0 and "child done" in r.stdout, r.stderr[-2000:]
        single = torch.load(path, weights_only=True)
        assert torch.equal(grouped["dx"].cpu().view(torch.int16), single["dx"].view(torch.int16))
