"""GPU parity of Q(x), Q(W1), Q(W2), Q(dY) on both sides of the size (2^18 elements) up to which range and cast share a
launch, with NaN and infinities, and of the state that the call's first kernel zeroes for the later ones."""
import numpy as np
import pytest
import torch

import synth
from oracle import fp8, quant

pytestmark = pytest.mark.gpu

import paper_2409_12517_amd as ssg  # noqa: E402
import gpu_util as gu  # noqa: E402
import test_gpu_mlp as tm  # noqa: E402

SHAPES = [(16, 16, 16), (256, 1024, 256), (272, 1024, 256), (16, 1040, 272)]


@pytest.mark.parametrize("T,d,f", SHAPES)
def test_quantized_operands_bit_for_bit(T, d, f):
    inp = synth.make_inputs(T, d, f, seed=T + d)
    inp["x"][3, 5], inp["x"][T - 1, d - 1] = float("nan"), -float("nan")
    inp["dY"][0, 0] = float("inf")
    blk = tm.Block(inp)
    # garbage in the state a call may find there
    blk.saved.fill_(0x7B)
    blk.work.fill_(0x7B)
    blk.fwd()
    blk.bwd()
    sc, wsc = gu.f32(blk.sv("scales", (16,), torch.float32)), gu.f32(blk.wv("scales", (8,), torch.float32))
    npi = tm._np_inputs(inp)
    for name, key, shape, fmt, scale, amax in (("x_q", "x", (T, d), fp8.E4M3, sc[0], sc[4]), ("w1_q", "W1", (f, d), fp8.E4M3, sc[1], sc[5]),
                                               ("w2_q", "W2", (f, d), fp8.E4M3, sc[2], sc[6]), ("dy_q", "dY", (T, d), fp8.E5M2, wsc[0], wsc[3])):
        q, s, a = quant.quantize_per_tensor(npi[key], fmt)
        got = gu.u8((blk.sv if name != "dy_q" else blk.wv)(name, shape, torch.uint8))
        assert scale == s and amax == a, name
        assert np.array_equal(got, q), name


@pytest.mark.parametrize("T,d,f", SHAPES)
@pytest.mark.parametrize("delayed", [False, True])
def test_garbage_in_the_buffers_changes_nothing(T, d, f, delayed):
    inp = synth.make_inputs(T, d, f, seed=T + f)
    out = []
    for fill in (0, 0xFF):
        blk = tm.Block(inp)
        state = torch.empty(ssg.ssg_mlp_scaling_state_bytes(), dtype=torch.uint8, device=gu.DEV)
        ssg.ssg_mlp_scaling_init(state)
        blk.desc.scaling_state = state.data_ptr()
        blk.fwd()
        blk.bwd()                                 # current scaling: fills the history
        if delayed:
            blk.desc.scale_mode = ssg.SSG_SCALE_DELAYED
        blk.saved.fill_(fill)
        blk.work.fill_(fill)
        blk.fwd()
        blk.bwd()
        out.append([t.view(torch.uint8).cpu() for t in (blk.y, blk.dx, blk.dW1, blk.dW2, blk.dW3, state[: 6 * 32 * 4])])
    for a, b in zip(*out):
        assert torch.equal(a, b)


@pytest.mark.parametrize("rows,cols", [(16, 16), (16, 1040), (1024, 1040), (4096, 2064)])
@pytest.mark.parametrize("src_dtype", [ssg.SSG_BF16, ssg.SSG_F32])
def test_quantize_with_its_range_words_in_the_result_buffer(rows, cols, src_dtype):
    """One to 1024 range words, which the range pass leaves in dst; the largest element first, last and in between, and
    scales rounded to powers of two; GIVEN with a range asked for."""
    gen = torch.Generator().manual_seed(rows + cols)
    base = torch.randn(rows, cols, generator=gen).to(torch.bfloat16 if src_dtype == ssg.SSG_BF16 else torch.float32)
    for at in ((0, 0), (rows - 1, cols - 1), (rows // 2, 7)):
        v = base.clone()
        v[at] = -37.5
        x = gu.dev(v)
        q, qt = gu.empty_u8(rows, cols), gu.empty_u8(cols, rows)
        scale, amax = gu.empty_f32(1), gu.empty_f32(1)
        for rnd, pow2 in ((ssg.SSG_ROUND_EXACT_DIV, False), (ssg.SSG_ROUND_POW2, True)):
            ssg.ssg_quantize(x, src_dtype, rows, cols, ssg.SSG_E4M3, ssg.SSG_SCALE_CURRENT, rnd, q, qt, scale, amax)
            ref_q, ref_s, ref_a = quant.quantize_per_tensor(v.float().numpy(), fp8.E4M3, pow2=pow2)
            assert gu.scalar(amax) == ref_a == np.float32(37.5) and gu.scalar(scale) == ref_s
            assert np.array_equal(gu.u8(q), ref_q) and np.array_equal(gu.u8(qt), ref_q.T)
        amax.zero_()
        ssg.ssg_quantize(x, src_dtype, rows, cols, ssg.SSG_E4M3, ssg.SSG_SCALE_GIVEN, ssg.SSG_ROUND_EXACT_DIV, q, None, scale, amax)
        assert gu.scalar(amax) == np.float32(37.5) and gu.scalar(scale) == ref_s
        assert np.array_equal(gu.u8(q), ref_q)


@pytest.mark.parametrize("n,src_dtype", [(16, ssg.SSG_BF16), (1 << 25, ssg.SSG_BF16), ((1 << 25) + 16, ssg.SSG_BF16),
                                         (16, ssg.SSG_F32), (1 << 23, ssg.SSG_F32), ((1 << 23) + 16, ssg.SSG_F32)])
def test_range_on_both_sides_of_looking_before_the_atomic(n, src_dtype):
    """Up to 2^25 bf16 elements (four runs for each of 1024 workgroups), 2^23 fp32 ones (one unit for each of 512): every
    workgroup's maximum goes to the word; above, only those that can raise it.  The largest element first, last, in the
    middle; NaN beside it; all zeros."""
    dt = torch.bfloat16 if src_dtype == ssg.SSG_BF16 else torch.float32
    x = torch.randn(n, device=gu.DEV).to(dt)
    amax = gu.empty_f32(1)
    for at in (0, n - 1, n // 2):
        v = x.clone()
        v[at] = -37.5
        v[(at + 5) % n] = float("nan")
        ssg.ssg_amax(v, src_dtype, n, amax)
        assert gu.scalar(amax) == np.float32(37.5), at
    ssg.ssg_amax(torch.zeros(n, device=gu.DEV, dtype=dt), src_dtype, n, amax)
    assert gu.scalar(amax) == 0.0
