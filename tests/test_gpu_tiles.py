"""GPU parity at the edges of the two GEMM tiles (128 x 128 and 256 x 256), at sizes that select either,
and of the kernel for few rows."""
import numpy as np
import pytest
import torch

import synth
from oracle import fp8, gemm

pytestmark = pytest.mark.gpu

import paper_2409_12517_amd as ssg  # noqa: E402
import gpu_util as gu  # noqa: E402
import test_gpu_gemm as tg  # noqa: E402
import test_gpu_infer as ti  # noqa: E402
import test_gpu_mlp as tm  # noqa: E402

SMALL = [(128, 128, 128), (16, 144, 272), (144, 112, 16), (272, 128, 400), (112, 400, 256)]
# 256 tiles of 256 x 256, one for every compute unit, with a ragged last K step (1168 = 9 * 128 + 16), a short last row and
# column of tiles; and 272 of them.  (Sizes around the tiles' edges; which kernel a shape takes is asserted in
# test_gpu_paths.py, with every route.)
LARGE = [(4048, 4080, 1168), (4080, 4336, 1040)]


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
    """Odd extents in every direction; the last shape has 16 x 32 tiles of 256 x 128 channels in U, G, over a ragged K."""
    inp = synth.make_inputs(T, d, f, seed=T + d + f)
    npi = tm._np_inputs(inp)
    blk = tm.Block(inp)
    blk.fwd()
    ref_fw, g = tm.check_forward(blk, npi)
    blk.bwd()
    tm.check_backward(blk, npi, ref_fw, g)


# Either form of the sum in either tile: both products in one tile, which changes the units of its accumulators between
# them (small tiles over whole and ragged K, large ones over whole K, which is all that they take), and in halves
SUMS = [(272, 256, 688, ssg.SSG_DX_HALVES, 128), (272, 256, 768, ssg.SSG_DX_HALVES, 128), (1552, 2064, 2064, ssg.SSG_DX_HALVES, 256),
        (1040, 272, 272, ssg.SSG_DX_ONE_TILE, 128), (528, 256, 256, ssg.SSG_DX_ONE_TILE, 128), (2064, 4096, 1024, ssg.SSG_DX_ONE_TILE, 256)]


def _assert_sum_form(desc, form, tile):
    p, r = ssg.ssg_mlp_gemm_plan(desc, ssg.SSG_PLAN_BWD_SECOND), ssg.ssg_mlp_gemm_route(desc, ssg.SSG_PLAN_BWD_SECOND)
    assert (r.dx_form, p.tile, p.launches) == (form, tile, 1)


@pytest.mark.parametrize("T,d,f,form,tile", SUMS)
@pytest.mark.parametrize("du_exp,dg_exp", [(0, 90), (90, 0), (-60, 60)])
def test_input_gradient_with_scales_far_apart(T, d, f, form, tile, du_exp, dg_exp):
    """dX sums two products whose scales may be any two binary32 numbers (here given as delayed scales, 2^90 or 2^120
    apart): the result is the sum of both, whichever is the larger, and finite."""
    inp = synth.make_inputs(T, d, f, seed=5)
    blk = tm.Block(inp, y_dtype=ssg.SSG_F32)
    state = torch.empty(ssg.ssg_mlp_scaling_state_bytes(), dtype=torch.uint8, device=gu.DEV)
    ssg.ssg_mlp_scaling_init(state)
    blk.desc.scaling_state = state.data_ptr()
    blk.fwd()
    blk.bwd()                                    # current scaling: fills the history
    blk.desc.scale_mode = ssg.SSG_SCALE_DELAYED
    _assert_sum_form(blk.desc, form, tile)
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
    gu.assert_close_gemm(gu.f32(blk.dx), ref, False, f"dX {T} {d} {f} {du_exp} {dg_exp}")


@pytest.mark.parametrize("T,d,f,form,tile", SUMS)
@pytest.mark.parametrize("du_exp,dg_exp", [(115, -37), (-37, 115)])
def test_input_gradient_where_one_gradient_flushes_to_zero(T, d, f, form, tile, du_exp, dg_exp):
    """Given scales 2^152 apart: the codes of one gradient are all zero, those of the other saturate, and dX (about 2^-98)
    is the product of the latter alone.  The change of units between the two products, 2^-152 or so, is no binary32 number,
    the product of an accumulator (2^28) with it is one."""
    inp = synth.make_inputs(T, d, f, seed=5)
    blk = tm.Block(inp, y_dtype=ssg.SSG_F32)
    state = torch.empty(ssg.ssg_mlp_scaling_state_bytes(), dtype=torch.uint8, device=gu.DEV)
    ssg.ssg_mlp_scaling_init(state)
    blk.desc.scaling_state = state.data_ptr()
    blk.fwd()
    blk.bwd()                                    # current scaling: fills the history
    blk.desc.scale_mode = ssg.SSG_SCALE_DELAYED
    _assert_sum_form(blk.desc, form, tile)
    words = state[: 6 * 32 * 4].view(torch.float32)
    words[4 * 32], words[5 * 32] = 2.0 ** du_exp, 2.0 ** dg_exp
    blk.fwd()
    blk.bwd()
    sc, wsc = gu.f32(blk.sv("scales", (16,), torch.float32)).astype(np.float64), gu.f32(blk.wv("scales", (8,), torch.float32)).astype(np.float64)
    grad, weight, i, j = ("du_q", "w1_q", 1, 1) if du_exp > 0 else ("dg_q", "w2_q", 2, 2)
    other = "dg_q" if du_exp > 0 else "du_q"
    assert not (gu.u8(blk.wv(other, (T, f), torch.uint8)) & 0x7F).any()
    ref = (fp8.decode(gu.u8(blk.wv(grad, (T, f), torch.uint8)), fp8.E5M2).astype(np.float64) @
           fp8.decode(gu.u8(blk.sv(weight, (f, d), torch.uint8)), fp8.E4M3).astype(np.float64)) / (wsc[i] * sc[j])
    # binary32 sums of 256 to 2064 products: 2e-3 of the largest element, as for every contraction here
    assert 2.0 ** -126 < np.abs(ref).max() and np.abs(gu.f32(blk.dx) - ref).max() <= 2e-3 * np.abs(ref).max()


# Few rows with ragged K and a last workgroup with part of its columns, rows beyond the last one; K shorter than one step
# for each wave; and 4096 rows by 1024 columns (K ragged and whole), in small tiles
@pytest.mark.parametrize("M,N,K", [(16, 4112, 1040), (48, 2032, 1168), (64, 4080, 784), (112, 4080, 656), (176, 4080, 912),
                                   (272, 4000, 1168), (32, 48, 16), (16, 16, 272), (4096, 1040, 400), (4096, 1024, 512)])
@pytest.mark.parametrize("a_fmt,c_dtype", [(ssg.SSG_E4M3, ssg.SSG_F32), (ssg.SSG_E5M2, ssg.SSG_BF16)])
def test_few_rows(M, N, K, a_fmt, c_dtype):
    rng = np.random.default_rng(M + 3 * N + K)
    a, b = tg._codes(rng, a_fmt, (M, K)), tg._codes(rng, ssg.SSG_E4M3, (N, K))
    ref = fp8.decode(a, tg.FMT[a_fmt]).astype(np.float64) @ fp8.decode(b, fp8.E4M3).astype(np.float64).T / (2.0 * 0.5)
    sa, sb = torch.tensor([2.0], device=gu.DEV), torch.tensor([0.5], device=gu.DEV)
    C = torch.full((M + 1, N), -7.0, device=gu.DEV, dtype=torch.float32 if c_dtype == ssg.SSG_F32 else torch.bfloat16)
    ssg.ssg_gemm_fp8(gu.dev(torch.from_numpy(a)), a_fmt, gu.dev(torch.from_numpy(b)), ssg.SSG_E4M3, M, N, K, sa, sb, C, c_dtype)
    torch.cuda.synchronize()
    gu.assert_close_gemm(gu.f32(C[:M]), ref, c_dtype == ssg.SSG_BF16, f"{M} {N} {K}")
    assert bool((C[M] == -7.0).all())


def test_few_rows_with_nan_and_extreme_scales():
    """A NaN code reaches its own row or column only; scales whose product leaves the binary32 range."""
    rng = np.random.default_rng(3)
    M, N, K = 48, 96, 272
    a, b = tg._codes(rng, ssg.SSG_E4M3, (M, K)), tg._codes(rng, ssg.SSG_E4M3, (N, K))
    ref = fp8.decode(a, fp8.E4M3).astype(np.float64) @ fp8.decode(b, fp8.E4M3).astype(np.float64).T
    a[5, 3], b[70, 271] = 0x7F, 0xFF
    got = tg._run(a, ssg.SSG_E4M3, b, 1e30, 1e-30, ssg.SSG_F32)
    assert np.isnan(got[5]).all() and np.isnan(got[:, 70]).all()
    keep = np.ix_([i for i in range(M) if i != 5], [j for j in range(N) if j != 70])
    assert np.abs(got[keep] - ref[keep]).max() <= 2e-3 * np.abs(ref).max()
    got = tg._run(a, ssg.SSG_E4M3, b, 1e30, 1e6, ssg.SSG_F32)
    assert np.abs(got[keep] * 1e36 - ref[keep]).max() <= 2e-3 * np.abs(ref).max()


@pytest.mark.parametrize("T_inf", [16, 48, 128, 144])
def test_few_rows_of_the_inference_form(T_inf):
    """16 rows, 17 to 128 rows and the first batch beyond them; d and f that are no multiples of the tiles.  (f is wide
    enough that the check's bar on codes more than a step apart, a share of 1e-4, means 4 of at least 40192 elements: a
    product next to zero, 2^-9 apart in code, now and then crosses more than one step when its sum rounds otherwise.)"""
    inp = synth.make_inputs(64, 272, 2512, seed=59)
    ti.check(ti.Infer(inp, T_inf=T_inf, seed_inf=8), tm._np_inputs(inp))


@pytest.mark.parametrize("T_inf,d,f,rows", [(2064, 272, 1040, 0), (1040, 400, 4096, 16), (528, 528, 4112, 16), (544, 1040, 4112, 32),
                                            (1584, 400, 2576, 48), (1088, 400, 4096, 64)])
def test_inference_form_with_its_last_rows_in_the_few_rows_form(T_inf, d, f, rows):
    """16 to 64 rows beyond whole large tiles, 260 to 512 small tiles for the others; one and two row blocks of 16 and of 32 rows,
    the last one half full; K with a last step of 16 bytes, a last column of tiles and a last set of few-rows workgroups that
    are cut.  And a batch of such a remainder that stays in tiles."""
    desc = ssg.make_desc(T_inf, d, f)
    p, r = ssg.ssg_mlp_gemm_plan(desc, ssg.SSG_PLAN_INFER_GATE_UP), ssg.ssg_mlp_gemm_route(desc, ssg.SSG_PLAN_INFER_GATE_UP)
    assert (p.tile, p.ring, p.whole_sets, p.launches) == (128, 5, 0, 1)
    assert (r.few_rows, r.few_rows_block) == (rows, 0 if rows == 0 else 16 if rows == 16 else 32)
    inp = synth.make_inputs(64, d, f, seed=67)
    ti.check(ti.Infer(inp, T_inf=T_inf, seed_inf=10), tm._np_inputs(inp))


def test_inference_form_in_whole_rounds_and_a_rest():
    """9 x 33 tiles of 256 rows by 128 channels, 41 more than one round of large ones."""
    inp = synth.make_inputs(64, 272, 4112, seed=61)
    ti.check(ti.Infer(inp, T_inf=2064, seed_inf=9), tm._np_inputs(inp))


def test_large_tile_sum_of_two_products_over_a_ragged_last_column():
    """dX in one launch of large tiles (16 x 16 of them, K = 8192 twice) whose last row and column of tiles are cut, with
    dW1, dW2 beside it: every element against the contraction of the stored codes in binary64 on the device."""
    T, d, f = 4080, 3984, 8192
    blk = tm.Block(synth.make_inputs(T, d, f, seed=17), y_dtype=ssg.SSG_F32)
    blk.fwd()
    blk.bwd()
    sc, wsc = blk.sv("scales", (16,), torch.float32).double(), blk.wv("scales", (8,), torch.float32).double()

    def dec(t, dtype):
        return t.view(dtype).double()

    duq, dgq = (dec(blk.wv(n, (T, f), torch.uint8), torch.float8_e5m2) for n in ("du_q", "dg_q"))
    w1, w2 = (dec(blk.sv(n, (f, d), torch.uint8), torch.float8_e4m3fn) for n in ("w1_q", "w2_q"))
    xq = dec(blk.sv("x_q", (T, d), torch.uint8), torch.float8_e4m3fn)
    for name, got, ref in (("dX", blk.dx, duq @ w1 / (wsc[1] * sc[1]) + dgq @ w2 / (wsc[2] * sc[2])),
                           ("dW1", blk.dW1, duq.t() @ xq / (wsc[1] * sc[0])), ("dW2", blk.dW2, dgq.t() @ xq / (wsc[2] * sc[0]))):
        assert float((got.double() - ref).abs().max()) <= 2e-3 * float(ref.abs().max()), name
