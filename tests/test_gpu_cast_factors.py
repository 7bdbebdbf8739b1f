"""GPU parity of the forward's casts of h and w3 with the channel factors formed in the same launch (workgroups exchange the ranges) with
the separate launches that a captured call takes: every stored tensor and scale, in each of the three tile heights, Smooth-SwiGLU and
plain block, with counters, a given scale of h and the history of delayed scaling."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

import paper_2409_12517_amd as ssg  # noqa: E402
import gpu_util as gu  # noqa: E402
import test_gpu_mlp as tm  # noqa: E402

# one group of 128 channels, cut; nine with 16 channels left over (few tiles: 16 rows each); 600 tiles (64 rows); 4128 tiles (128 rows),
# 129 groups, so that the plain block's two ranges have no room; the most channels that Smooth-SwiGLU's have, and one group more
SHAPES = [(16, 16, 16), (144, 528, 1040), (2560, 256, 1936), (2048, 64, 16512), (16, 16, 32768), (32, 16, 32784)]


def _outputs(blk, state):
    out = [blk.y, blk.sv("scales", (16,), torch.float32), blk.sv("s", (blk.f,), torch.float32), blk.sv("sinv", (blk.f,), torch.float32),
           blk.sv("h_q", (blk.T, blk.f), torch.uint8), blk.sv("w3_q", (blk.d, blk.f), torch.uint8), state[: 6 * 32 * 4]]
    if blk.h_counters is not None:
        out.append(blk.h_counters)
    return [t.clone().view(torch.uint8) for t in out]


@pytest.mark.parametrize("T,d,f", SHAPES)
@pytest.mark.parametrize("variant", ["smooth", "plain", "given"])
@pytest.mark.parametrize("delayed", [False, True])
def test_factors_in_the_launch_equal_a_launch_of_their_own(T, d, f, variant, delayed):
    inp = synth.make_inputs(T, d, f, seed=T + f)
    inp["W1"][f // 2] = 0                              # a channel without range
    results = []
    for captured in (False, True):
        blk = tm.Block(inp, smooth=int(variant == "smooth"), h_scale=300.0 if variant == "given" else None, count=True)
        state = torch.empty(ssg.ssg_mlp_scaling_state_bytes(), dtype=torch.uint8, device=gu.DEV)
        ssg.ssg_mlp_scaling_init(state)
        blk.desc.scaling_state = state.data_ptr()
        blk.fwd()                                      # fills the history
        if delayed:
            blk.desc.scale_mode = ssg.SSG_SCALE_DELAYED
        blk.saved.fill_(0x7B)
        if captured:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                ssg.ssg_mlp_fwd(blk.desc, blk.x, blk.W1, blk.W2, blk.W3, blk.y, blk.saved)
            graph.replay()
            torch.cuda.synchronize()
        else:
            blk.fwd()
        results.append(_outputs(blk, state))
    for k, (a, b) in enumerate(zip(*results)):
        assert torch.equal(a, b), k
