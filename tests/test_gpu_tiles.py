"""GPU parity at the edges of the two GEMM tiles (128 x 128 and 256 x 256), at sizes that select either."""
import numpy as np
import pytest
import torch

import synth
from oracle import fp8, gemm

pytestmark = pytest.mark.gpu

import paper_2409_12517_amd as ssg  # noqa: E402
import gpu_util as gu  # noqa: E402
import test_gpu_gemm as tg  # noqa: E402
import test_gpu_mlp as tm  # noqa: E402

SMALL = [(128, 128, 128), (16, 144, 272), (144, 112, 16), (272, 128, 400), (112, 400, 256)]
# 256 tiles of 256 x 256, one for every compute unit: the large tile, with a ragged last K step (1168 = 9 * 128 + 16),
# a short last row and column of tiles
LARGE = [(4048, 4080, 1168)]


@pytest.mark.parametrize("M,N,K", SMALL + LARGE)
@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 1)])
def test_contraction_at_tile_edges(M, N, K, layout):
    rng = np.random.default_rng(M + 3 * N + K)
    a, b = tg._codes(rng, ssg.SSG_E5M2, (M, K)), tg._codes(rng, ssg.SSG_E4M3, (N, K))
    ref = fp8.decode(a, fp8.E5M2).astype(np.float64) @ fp8.decode(b, fp8.E4M3).astype(np.float64).T / (2.0 * 0.5)
    A = gu.dev(torch.from_numpy(np.ascontiguousarray(a.T) if layout[0] else a))
    B = gu.dev(torch.from_numpy(np.ascontiguousarray(b.T) if layout[1] else b))
    sa, sb = torch.tensor([2.0], device=gu.DEV), torch.tensor([0.5], device=gu.DEV)
    # one row more than the result: nothing is written past its end
    C = torch.full((M + 1, N), -7.0, device=gu.DEV)
    ssg.ssg_gemm_fp8_layout(A, ssg.SSG_E5M2, layout[0], B, ssg.SSG_E4M3, layout[1], M, N, K, sa, sb, C, ssg.SSG_F32)
    torch.cuda.synchronize()
    gu.assert_close_gemm(gu.f32(C[:M]), ref, False, f"{M} {N} {K} {layout}")
    assert bool((C[M] == -7.0).all())


@pytest.mark.parametrize("T,d,f", [(144, 272, 400), (400, 144, 1168), (3856, 784, 4096)])
def test_block_at_tile_edges(T, d, f):
    """Odd extents in every direction; the last shape runs U, G in the large tile (16 x 32 tiles of 256 x 128 channels)
    over a ragged K, and everything else in the small one."""
    inp = synth.make_inputs(T, d, f, seed=T + d + f)
    npi = tm._np_inputs(inp)
    blk = tm.Block(inp)
    blk.fwd()
    ref_fw, g = tm.check_forward(blk, npi)
    blk.bwd()
    tm.check_backward(blk, npi, ref_fw, g)


@pytest.mark.parametrize("f", [688, 768])
@pytest.mark.parametrize("du_exp,dg_exp", [(0, 90), (90, 0), (-60, 60)])
def test_input_gradient_with_scales_far_apart(f, du_exp, dg_exp):
    """dX sums two products whose scales may be any two binary32 numbers (here given as delayed scales, 2^90 or 2^120
    apart): the result is the sum of both, whichever is the larger, and finite."""
    T, d = 272, 256
    inp = synth.make_inputs(T, d, f, seed=5)
    blk = tm.Block(inp, y_dtype=ssg.SSG_F32)
    state = torch.empty(ssg.ssg_mlp_scaling_state_bytes(), dtype=torch.uint8, device=gu.DEV)
    ssg.ssg_mlp_scaling_init(state)
    blk.desc.scaling_state = state.data_ptr()
    blk.fwd()
    blk.bwd()                                    # current scaling: fills the history
    blk.desc.scale_mode = ssg.SSG_SCALE_DELAYED
    words = state[: 6 * 32 * 4].view(torch.float32)
    words[4 * 32] *= 2.0 ** du_exp
    words[5 * 32] *= 2.0 ** dg_exp
    blk.fwd()
    blk.bwd()
    sc, wsc = gu.f32(blk.sv("scales", (16,), torch.float32)).astype(np.float64), gu.f32(blk.wv("scales", (8,), torch.float32)).astype(np.float64)

    def dec(t, fmt):
        return fp8.decode(gu.u8(t), fmt).astype(np.float64)

    ref = (dec(blk.wv("du_q", (T, f), torch.uint8), fp8.E5M2) @ dec(blk.sv("w1_q", (f, d), torch.uint8), fp8.E4M3) / (wsc[1] * sc[1]) +
           dec(blk.wv("dg_q", (T, f), torch.uint8), fp8.E5M2) @ dec(blk.sv("w2_q", (f, d), torch.uint8), fp8.E4M3) / (wsc[2] * sc[2]))
    assert np.isfinite(gu.f32(blk.dx)).all() and np.abs(ref).max() > 0
    gu.assert_close_gemm(gu.f32(blk.dx), ref, False, f"dX {f} {du_exp} {dg_exp}")
