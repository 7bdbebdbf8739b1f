"""GPU parity of the eight-value encode where a group holds what takes its rare branch (NaN of either sign, infinities, overflow at
each place of eight), in the launches that cast a whole tensor (ssg_quantize in one and in separate launches and each tile height,
the block's own recording cast and its one-launch form of small tensors) and in the epilogues that cast; and of the SwiGLU product
with 64 bits."""
import numpy as np
import pytest
import torch

import synth
from oracle import fp8

pytestmark = pytest.mark.gpu

import paper_2409_12517_amd as ssg  # noqa: E402
import gpu_util as gu  # noqa: E402
import test_gpu_infer as ti  # noqa: E402
import test_gpu_mlp as tm  # noqa: E402

FMT = {ssg.SSG_E4M3: fp8.E4M3, ssg.SSG_E5M2: fp8.E5M2}


def _specials(src, special, seed):
    """Sets each of `special` at every place of eight, in one of the first rows and in the last, groups 5 apart; the rows touched."""
    rows, cols = src.shape
    touched = {rows - 1, rows // 2}
    for i, v in enumerate(special):
        for k in range(8):
            for r in ((i + seed) % rows, rows - 1):
                src[r, (8 * (5 * i + k) + k) % cols] = v
                touched.add(r)
    return sorted(touched)


# Current scaling: all in one launch but the last, too large for it.  A given scale: casts alone, with the transposed copy and in
# fp32 always in tiles of 128 rows, else of 16, 64 and 128 (up to 512, up to 4096, more tiles of 128 x 128)
@pytest.mark.parametrize("fmt", [ssg.SSG_E4M3, ssg.SSG_E5M2])
@pytest.mark.parametrize("rows,cols,dtype", [(16, 64, torch.bfloat16), (272, 1040, torch.float32), (2064, 4096, torch.bfloat16),
                                             (8208, 8192, torch.bfloat16)])
@pytest.mark.parametrize("mode", [ssg.SSG_SCALE_GIVEN, ssg.SSG_SCALE_CURRENT])
@pytest.mark.parametrize("transposed", [True, False])
def test_specials_at_each_place_of_eight(rows, cols, dtype, fmt, mode, transposed):
    gen = torch.Generator(device=gu.DEV).manual_seed(rows + fmt)
    src = torch.randn(rows, cols, generator=gen, device=gu.DEV)
    given = mode == ssg.SSG_SCALE_GIVEN
    pick = _specials(src, [float("nan"), -float("nan")] + ([float("inf"), -float("inf"), 3e38, -6e4, 449.0, -1e-30] if given else [-0.0, 1e-30]), 0)
    src = src.to(dtype)
    q, qt = gu.empty_u8(rows, cols), gu.empty_u8(cols, rows) if transposed else None
    sc, am = torch.ones(1, device=gu.DEV), gu.empty_f32(1)
    ssg.ssg_quantize(src, ssg.SSG_F32 if dtype == torch.float32 else ssg.SSG_BF16, rows, cols, fmt, mode, ssg.SSG_ROUND_EXACT_DIV, q, qt, sc, am)
    assert not transposed or torch.equal(qt.T, q)
    ref = fp8.satcast(src[pick].float().cpu().numpy() * gu.scalar(sc), FMT[fmt])
    assert np.array_equal(gu.u8(q)[pick], ref)


# The block's own casts of x, W1, W2 (E4M3) and dY (E5M2).  Current scaling: up to 2^18 elements in one launch without an exchange;
# delayed: with the recording cast, tiles of 16, 64 and 128 rows by the tiles of all items of a launch
@pytest.mark.parametrize("T,d,f,delayed", [(48, 64, 96, 0), (48, 64, 96, 1), (1040, 1024, 6896, 1), (2064, 2048, 11008, 1), (8208, 8192, 48, 1)])
def test_specials_in_the_casts_of_the_block(T, d, f, delayed):
    gen = torch.Generator(device=gu.DEV).manual_seed(T + f)
    blk = tm.Block({"x": torch.zeros(T, d, dtype=torch.bfloat16), "W1": torch.zeros(f, d, dtype=torch.bfloat16),
                    "W2": torch.zeros(f, d, dtype=torch.bfloat16), "W3": torch.ones(d, f, dtype=torch.bfloat16),
                    "dY": torch.zeros(T, d, dtype=torch.bfloat16)})
    state = torch.empty(ssg.ssg_mlp_scaling_state_bytes(), dtype=torch.uint8, device=gu.DEV)
    ssg.ssg_mlp_scaling_init(state)                       # scales 1
    if delayed:
        blk.desc = ssg.make_desc(T, d, f, scale_mode=ssg.SSG_SCALE_DELAYED, scaling_state=state)
    special = [float("nan"), -float("nan")] + ([float("inf"), -float("inf"), 3e38, -6e4, 449.0, -1e-30] if delayed else [-0.0, 1e-30])
    picks = []
    for k, t in enumerate((blk.x, blk.W1, blk.W2, blk.dY)):
        v = torch.randn(t.shape, generator=gen, device=gu.DEV)
        picks.append(_specials(v, special, k))
        t.copy_(v.to(torch.bfloat16))
    blk.fwd()
    blk.bwd()
    sc, wsc = gu.f32(blk.sv("scales", (16,), torch.float32)), gu.f32(blk.wv("scales", (8,), torch.float32))
    got = (("x_q", blk.x, sc[0], fp8.E4M3), ("w1_q", blk.W1, sc[1], fp8.E4M3), ("w2_q", blk.W2, sc[2], fp8.E4M3), ("dy_q", blk.dY, wsc[0], fp8.E5M2))
    for (name, t, scale, fmt), pick in zip(got, picks):
        assert scale == 1.0 or not delayed
        q = (blk.wv if name == "dy_q" else blk.sv)(name, tuple(t.shape), torch.uint8)
        assert np.array_equal(gu.u8(q[pick]), fp8.satcast(t[pick].float().cpu().numpy() * scale, fmt)), name


@pytest.mark.parametrize("T,f", [(272, 144), (528, 2064)])
def test_epilogue_that_casts_keeps_overflow_of_bf16(T, f):
    """dU, dG that leave the dH epilogue as E5M2 codes, kept in bf16 too: what overflows bf16 in rounding is an infinity there, as in
    the stored-tensor path, in every group after a conversion that saturates; NaN stays in its row.  All operands are powers of
    two and a few bits, so every number is exact: dU = 1.96875 2^119 x 260 = 3.4019e38, a float that rounds to no bf16."""
    d = 16
    inp = {k: torch.zeros(s, dtype=torch.bfloat16) for k, s in (("x", (T, d)), ("W1", (f, d)), ("W2", (f, d)), ("W3", (d, f)), ("dY", (T, d)))}
    inp["x"][:, 0] = inp["x"][:, 1] = 1.0
    inp["W1"][:, 0] = 1.0                                  # U = 1
    inp["W2"][:, 0], inp["W2"][:, 1] = 256.0, 4.0          # G = 260, Swish(G) = 260, its derivative 1
    inp["W3"][:] = 288.0                                   # 1.125 2^8; the range is 448: scale 1
    inp["W3"][d - 1] = 448.0
    big = 57344.0 * 2.0 ** 96
    row = torch.arange(T)
    inp["dY"][row, row % 8] = torch.where(row % 3 == 0, big, torch.where(row % 3 == 1, -big, big / 8)).to(torch.bfloat16)
    nan_row = T - 9
    inp["dY"][nan_row, 3] = float("nan")
    state = torch.empty(ssg.ssg_mlp_scaling_state_bytes(), dtype=torch.uint8, device=gu.DEV)
    ssg.ssg_mlp_scaling_init(state)
    words = state[: 6 * 32 * 4].view(torch.float32).view(6, 32)
    words[3, 0] = 2.0 ** -96                               # the scale of dY
    blk = tm.Block(inp, smooth=0)
    blk.desc = ssg.make_desc(T, d, f, smooth=0, scale_mode=ssg.SSG_SCALE_DELAYED, scaling_state=state, keep_bf16_grads=1)
    blk.fwd()
    blk.bwd()
    assert bool((blk.sv("U", (T, f), torch.bfloat16) == 1).all()) and bool((blk.sv("G", (T, f), torch.bfloat16) == 260).all())
    dH = inp["dY"].double().sum(1) * 288.0                 # one element a row
    dU, dG = blk.wv("dU", (T, f), torch.bfloat16).cpu(), blk.wv("dG", (T, f), torch.bfloat16).cpu()
    want_u, want_g = (dH * 260.0).float().to(torch.bfloat16), dH.float().to(torch.bfloat16)
    assert bool(torch.isinf(want_u[row % 3 != 2].float()).sum() > 0) and bool(torch.isfinite((dH * 260.0).float()[row != nan_row]).all())
    keep = row != nan_row
    assert torch.equal(dU[keep], want_u[keep, None].expand(-1, f)) and torch.equal(dG[keep], want_g[keep, None].expand(-1, f))
    assert bool(torch.isnan(dU[nan_row].float()).all())
    for name, v in (("du_q", dU), ("dg_q", dG)):           # their scales are 1
        assert np.array_equal(gu.u8(blk.wv(name, (T, f), torch.uint8)), fp8.satcast(gu.f32(v), fp8.E5M2)), name
    after = words.cpu()
    assert after[4, 2] == float("inf") and after[5, 2] == dH[keep].abs().max().float().to(torch.bfloat16).float()


@pytest.mark.parametrize("T,d,f,tile", [(16, 256, 688, 0), (272, 256, 688, 128), (4096, 4096, 4096, 256)])
def test_epilogue_of_the_inference_form_with_nan_and_overflow(T, d, f, tile):
    ok = ti.Infer(synth.make_inputs(256, d, f, seed=5), T_inf=T, seed_inf=3)
    assert ssg.ssg_mlp_gemm_plan(ok.desc, ssg.SSG_PLAN_INFER_GATE_UP).tile == tile
    x = ok.x.clone()
    bad = sorted({1, T // 2, T - 1})
    x[bad[0], 7], x[bad[1], 0], x[bad[2], d - 1] = float("nan"), -float("nan"), float("nan")
    first = ok.wv("h_q", (T, f), torch.uint8).clone()
    for factor in (1.0, 64.0):                             # 64 times the calibrated range: most of h saturates
        y = torch.empty_like(ok.y)
        ssg.ssg_infer_fwd(ok.desc, x * factor, ok.prep, y, ok.work)
        torch.cuda.synchronize()
        h = ok.wv("h_q", (T, f), torch.uint8)
        assert bool(((h[bad] & 0x7F) == 0x7F).all())
        good = [r for r in range(T) if r not in bad]
        assert not bool(((h[good] & 0x7F) == 0x7F).any())
        if factor == 1.0 and float(x[good].float().abs().max()) == float(ok.x.float().abs().max()):
            assert torch.equal(h[good], first[good])       # the same scale of x: the same codes
        if factor > 1.0:
            assert float(((h[good] & 0x7F) == 0x7E).float().mean()) > 0.2


@pytest.mark.parametrize("spread", [1.0, 8.0, 100.0])
def test_swiglu_against_64_bits(spread):
    gen = torch.Generator(device=gu.DEV).manual_seed(int(spread))
    T, f = 512, 1024
    u, g = (torch.randn(T, f, generator=gen, device=gu.DEV) + 1.5).to(torch.bfloat16), (spread * torch.randn(T, f, generator=gen, device=gu.DEV)).to(torch.bfloat16)
    g[0, :8] = torch.tensor([0.0, -0.0, 88.0, -88.0, 3e38, -3e38, -1e7, 1e-30])
    u[0, :8] = 1.0                               # (3e38 times more is no float)
    h = gu.empty_f32(T, f)
    ssg.ssg_swiglu(u, g, T, f, h)
    ref = (u.double() * g.double() * torch.sigmoid(g.double())).cpu().numpy()
    # exp2 and the reciprocal to an ulp (2^-23), four roundings (2^-24): 6 ulp with room; below e^-87 the sigmoid is flushed to zero
    assert np.all(np.abs(gu.f32(h) - ref) <= 6 * 2.0 ** -23 * np.abs(ref) + 1e-34)
