"""GPU parity of every route a GEMM can take, each at shapes for which the library's own plan names that route (asserted
before the run, so that a change of an estimate cannot move a test off its path unseen).  Rows and columns of tiles are
cut; every element is compared with the contraction of the stored codes in binary64 on the device, to the stated bar
(2e-3 of the largest element, and one unit of bf16 where the output is bf16)."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

import paper_2409_12517_amd as ssg  # noqa: E402
import gpu_util as gu  # noqa: E402
import test_gpu_infer as ti  # noqa: E402
import test_gpu_mlp as tm  # noqa: E402

F8 = {ssg.SSG_E4M3: torch.float8_e4m3fn, ssg.SSG_E5M2: torch.float8_e5m2}


def _dec(codes, fmt=ssg.SSG_E4M3):
    return codes.view(F8[fmt]).double()


def _close(got, ref, what):
    bound = 2e-3 * ref.abs().max()
    err = (got.double() - ref).abs() - bound
    if got.dtype == torch.bfloat16:
        err -= torch.exp2(torch.floor(torch.log2(ref.abs().clamp_min(2.0 ** -126))) - 7)
    assert bool(torch.isfinite(got).all()) and float(err.max()) <= 0, (what, float((got.double() - ref).abs().max()), float(bound))


def _codes(gen, fmt, *shape):
    return (torch.randn(*shape, device=gu.DEV, generator=gen) * 8).to(F8[fmt]).view(torch.uint8)


def _contract(M, N, K, layout, a_fmt, c_dtype):
    """Runs one public contraction with a guard row after the result; compares every element."""
    gen = torch.Generator(device=gu.DEV).manual_seed(M + 3 * N + 7 * K + layout)
    a, b = _codes(gen, a_fmt, *((K, M) if layout == 2 else (M, K))), _codes(gen, ssg.SSG_E4M3, *((K, N) if layout else (N, K)))
    sa, sb = torch.tensor([2.0], device=gu.DEV), torch.tensor([0.25], device=gu.DEV)
    C = torch.full((M + 1, N), -7.0, device=gu.DEV, dtype=torch.float32 if c_dtype == ssg.SSG_F32 else torch.bfloat16)
    ssg.ssg_gemm_fp8_layout(a, a_fmt, int(layout == 2), b, ssg.SSG_E4M3, int(layout >= 1), M, N, K, sa, sb, C, c_dtype)
    torch.cuda.synchronize()
    ad, bd = _dec(a, a_fmt), _dec(b)
    _close(C[:M], (ad.t() if layout == 2 else ad) @ (bd if layout else bd.t()) / 0.5, "C")
    assert bool((C[M] == -7.0).all())


def _plan(M, N, K, layout, a_fmt, c_dtype):
    p = ssg.ssg_gemm_fp8_plan(a_fmt, int(layout == 2), int(layout >= 1), M, N, K, c_dtype)
    return p.tile, p.ring, p.whole_sets, p.launches


# Tile, ring, sets of large tiles run first, launches.  Large tiles in one round and more, K ragged and whole; small tiles two
# to a compute unit; the long ring with more K steps than it holds; whole rounds of large tiles and the rest in small ones,
# with either ring
@pytest.mark.parametrize("M,N,K,route", [
    (4048, 4080, 1552, (256, 5, 0, 1)), (2064, 6160, 4112, (256, 5, 0, 1)), (4096, 4096, 4096, (256, 5, 0, 1)),
    (1040, 4336, 656, (128, 5, 0, 1)), (2048, 3072, 640, (128, 5, 0, 1)),
    (2032, 1040, 2064, (128, 9, 0, 1)), (2048, 1024, 2048, (128, 9, 0, 1)),
    (6544, 6032, 784, (128, 5, 64, 2)), (2736, 6464, 2064, (128, 9, 32, 2))])
@pytest.mark.parametrize("layout,c_dtype", [(0, ssg.SSG_F32), (1, ssg.SSG_F32), (2, ssg.SSG_F32), (0, ssg.SSG_BF16)])
def test_contraction_on_each_tile_route(M, N, K, route, layout, c_dtype):
    if (M, c_dtype) == (6544, ssg.SSG_BF16):
        route = (256, 5, 0, 1)                          # the shorter epilogue keeps that shape whole
    a_fmt = ssg.SSG_E5M2 if layout else ssg.SSG_E4M3
    assert _plan(M, N, K, layout, a_fmt, c_dtype) == route
    _contract(M, N, K, layout, a_fmt, c_dtype)


# Every form of the few-rows kernel with more K steps for each wave than its ring holds (41 steps for four waves, the last
# one ragged; 40 whole), in both formats; rows and columns cut.  And with fewer steps than waves
@pytest.mark.parametrize("M,N,rows,cols,ring", [(16, 4080, 16, 16, 5), (32, 4080, 16, 32, 3), (64, 4080, 32, 32, 2), (112, 4080, 64, 32, 3),
                                                (176, 4080, 64, 64, 2), (272, 4000, 96, 64, 2)])
@pytest.mark.parametrize("K,a_fmt,c_dtype", [(5136, ssg.SSG_E4M3, ssg.SSG_F32), (5120, ssg.SSG_E5M2, ssg.SSG_BF16)])
def test_contraction_in_each_form_of_the_few_rows_kernel(M, N, rows, cols, ring, K, a_fmt, c_dtype):
    p = ssg.ssg_gemm_fp8_plan(a_fmt, 0, 0, M, N, K, c_dtype)
    assert (p.tile, p.rows, p.cols, p.ring) == (0, rows, cols, ring)
    assert (-(-K // 128) + 3) // 4 >= 2 * ring          # every slot is used again
    _contract(M, N, K, 0, a_fmt, c_dtype)


@pytest.mark.parametrize("T,rows,ring,waves", [(16, 16, 3, 4), (48, 64, 2, 2), (112, 64, 2, 2)])
def test_inference_gate_up_in_each_form_of_the_few_rows_kernel(T, rows, ring, waves):
    d, f = 3600, 2512                                   # 29 K steps, the last one ragged
    p = ssg.ssg_mlp_gemm_plan(ssg.make_desc(T, d, f), ssg.SSG_PLAN_INFER_GATE_UP)
    assert (p.tile, p.rows, p.ring) == (0, rows, ring) and 29 // waves >= 2 * ring
    inp = synth.make_inputs(64, d, f, seed=63)
    ti.check(ti.Infer(inp, T_inf=T, seed_inf=T), tm._np_inputs(inp))


@pytest.mark.parametrize("T,d,f,route", [(1952, 1168, 5744, (128, 5, 32)), (2960, 1040, 5856, (128, 9, 64)), (400, 784, 5744, (128, 5, 0)),
                                         (272, 2064, 1552, (128, 9, 0)), (1040, 2064, 5744, (256, 5, 0))])
def test_inference_gate_up_on_each_tile_route(T, d, f, route):
    """h^ of the inference form, whole rounds and a rest among them, on every element and to the bars of
    test_gpu_infer.check: the code is a rounding of some product within the propagated tolerance of the contractions (1e-4
    of the largest u and g, to first order through u * Swish(g)), and less than 5e-3 of the codes differ from the rounding
    of the exact product."""
    p = ssg.ssg_mlp_gemm_plan(ssg.make_desc(T, d, f), ssg.SSG_PLAN_INFER_GATE_UP)
    assert (p.tile, p.ring, p.whole_sets) == route
    inf = ti.Infer(synth.make_inputs(64, d, f, seed=65), T_inf=T, seed_inf=T)
    sw, sx = inf.pv("weight_scales", (8,), torch.float32).double(), inf.wv("x_scale", (2,), torch.float32).double()[0]
    xq = _dec(inf.wv("x_q", (T, d), torch.uint8))
    u, g = (xq @ _dec(inf.pv(n, (f, d), torch.uint8)).t() / (sx * sw[i]) for i, n in ((0, "w1_q"), (1, "w2_q")))
    sg = torch.sigmoid(g)
    tol = (g * sg).abs() * (1e-4 * u.abs().max()) + (u * sg * (1 + g * (1 - sg))).abs() * (1e-4 * g.abs().max())
    h = (u * g * sg).clamp(-448, 448)                     # the cast saturates
    got = _dec(inf.wv("h_q", (T, f), torch.uint8))
    half = torch.exp2(torch.floor(torch.log2(got.abs().clamp_min(2.0 ** -6))) - 4)
    assert float(((got - h).abs() - half * (1 + 1e-6) - tol).max()) <= 0
    assert float((got != h.float().to(torch.float8_e4m3fn).double()).double().mean()) < 5e-3


def _training(T, d, f, **kw):
    blk = tm.Block(synth.make_inputs(T, d, f, seed=T + d), y_dtype=ssg.SSG_F32)
    if kw:
        blk.desc = ssg.make_desc(T, d, f, y_dtype=ssg.SSG_F32, **kw)
    return blk


def _check_forward(blk):
    T, d, f = blk.T, blk.d, blk.f
    sc = blk.sv("scales", (16,), torch.float32).double()
    xq = _dec(blk.sv("x_q", (T, d), torch.uint8))
    U, G = blk.sv("U", (T, f), torch.bfloat16), blk.sv("G", (T, f), torch.bfloat16)
    _close(U, xq @ _dec(blk.sv("w1_q", (f, d), torch.uint8)).t() / (sc[0] * sc[1]), "U")
    _close(G, xq @ _dec(blk.sv("w2_q", (f, d), torch.uint8)).t() / (sc[0] * sc[2]), "G")
    h = gu.empty_f32(T, f)
    ssg.ssg_swiglu(U, G, T, f, h)
    assert torch.equal(blk.sv("h_camax", (f,), torch.float32), h.abs().amax(dim=0))
    assert torch.equal(blk.sv("w3_camax", (f,), torch.float32), blk.W3.float().abs().amax(dim=0))
    _close(blk.y, _dec(blk.sv("h_q", (T, f), torch.uint8)) @ _dec(blk.sv("w3_q", (d, f), torch.uint8)).t() / sc[3], "y")


@pytest.mark.parametrize("T,d,f,cached,route", [(1728, 784, 5856, 0, (128, 5, 32)), (1952, 1040, 4624, 0, (128, 9, 32)),
                                                (1728, 784, 5968, 1, (128, 5, 32)), (2288, 1040, 3952, 1, (128, 9, 32)),
                                                (1040, 784, 2736, 0, (128, 5, 0)), (4096, 784, 2064, 0, (256, 5, 0))])
def test_training_gate_up_on_each_route(T, d, f, cached, route):
    """U, G, the channel maxima and, where W3 is not cached, the range pass over it that rides in the last launch."""
    p = ssg.ssg_mlp_gemm_plan(ssg.make_desc(T, d, f, weights_cached=cached), ssg.SSG_PLAN_GATE_UP)
    assert (p.tile, p.ring, p.whole_sets) == route
    blk = _training(T, d, f)
    blk.fwd()
    if cached:
        for name in ("U", "G"):
            blk.sv(name, (T, f), torch.bfloat16).fill_(float("nan"))
        blk.desc = ssg.make_desc(T, d, f, y_dtype=ssg.SSG_F32, weights_cached=1)
        blk.fwd()
    _check_forward(blk)


def _check_backward(blk, delayed):
    T, d, f = blk.T, blk.d, blk.f
    sc, wsc = blk.sv("scales", (16,), torch.float32).double(), blk.wv("scales", (8,), torch.float32).double()
    U, G = blk.sv("U", (T, f), torch.bfloat16).double(), blk.sv("G", (T, f), torch.bfloat16).double()
    s, sinv = blk.sv("s", (f,), torch.float32).double(), blk.sv("sinv", (f,), torch.float32).double()
    dyq, hq, xq = _dec(blk.wv("dy_q", (T, d), torch.uint8), ssg.SSG_E5M2), _dec(blk.sv("h_q", (T, f), torch.uint8)), _dec(blk.sv("x_q", (T, d), torch.uint8))
    w1, w2, w3 = _dec(blk.sv("w1_q", (f, d), torch.uint8)), _dec(blk.sv("w2_q", (f, d), torch.uint8)), _dec(blk.sv("w3_q", (d, f), torch.uint8))
    dH = dyq @ w3 / (wsc[0] * sc[3]) * s
    sg = torch.sigmoid(G)
    dU, dG = blk.wv("dU", (T, f), torch.bfloat16), blk.wv("dG", (T, f), torch.bfloat16)
    _close(dU, dH * G * sg, "dU")
    _close(dG, dH * U * sg * (1 + G * (1 - sg)), "dG")
    duq, dgq = blk.wv("du_q", (T, f), torch.uint8), blk.wv("dg_q", (T, f), torch.uint8)
    for q, v, k in ((duq, dU, 1), (dgq, dG, 2)):          # E5M2 has an infinity: the cast saturates to 57344 first
        ref = (v.float() * wsc[k].float()).clamp(-57344, 57344).to(torch.float8_e5m2).view(torch.uint8)
        assert torch.equal(q, ref), k
        if not delayed:
            assert float(wsc[3 + k]) == float(v.float().abs().max())
    du, dg = _dec(duq, ssg.SSG_E5M2), _dec(dgq, ssg.SSG_E5M2)
    _close(blk.dx, du @ w1 / (wsc[1] * sc[1]) + dg @ w2 / (wsc[2] * sc[2]), "dX")
    _close(blk.dW1, du.t() @ xq / (wsc[1] * sc[0]), "dW1")
    _close(blk.dW2, dg.t() @ xq / (wsc[2] * sc[0]), "dW2")
    _close(blk.dW3, dyq.t() @ hq * sinv / wsc[0], "dW3")


# Tiles of the first and second backward launch, launches of the second, and dX's form: both groups in either tile, a different
# one each; both products of dX in one tile over whole and ragged K, and in halves; dX in two launches through its scratch,
# with dH and dW3 launched singly
ONE, HALVES, TWO = ssg.SSG_DX_ONE_TILE, ssg.SSG_DX_HALVES, ssg.SSG_DX_TWO_LAUNCHES
BACKWARD = [(3296, 2064, 3584, 0, 256, 256, 1, ONE), (1952, 4096, 1024, 0, 128, 256, 1, ONE), (2960, 2064, 3840, 0, 256, 128, 1, ONE),
            (1040, 784, 2736, 0, 128, 128, 1, HALVES), (5280, 3072, 2272, 0, 128, 256, 4, TWO), (3584, 640, 1680, 0, 128, 128, 1, ONE),
            (1952, 3088, 5376, 2, 256, 256, 1, ONE), (2960, 2064, 5632, 2, 256, 128, 1, ONE), (1952, 4096, 1024, 2, 128, 256, 1, ONE),
            (1040, 784, 2736, 2, 128, 128, 1, HALVES), (3584, 640, 1680, 2, 128, 128, 1, ONE)]


@pytest.mark.parametrize("T,d,f,mode,first,second,launches,form", BACKWARD)
def test_backward_on_each_route(T, d, f, mode, first, second, launches, form):
    state = torch.empty(ssg.ssg_mlp_scaling_state_bytes(), dtype=torch.uint8, device=gu.DEV)
    ssg.ssg_mlp_scaling_init(state)
    kw = dict(scaling_state=state, keep_bf16_grads=int(mode == ssg.SSG_SCALE_DELAYED))
    blk = _training(T, d, f, **kw)
    blk.fwd()
    blk.bwd()                                             # current scaling: fills the history
    if mode == ssg.SSG_SCALE_DELAYED:
        blk.desc = ssg.make_desc(T, d, f, y_dtype=ssg.SSG_F32, scale_mode=mode, **kw)
    p, q = (ssg.ssg_mlp_gemm_plan(blk.desc, w) for w in (ssg.SSG_PLAN_BWD_FIRST, ssg.SSG_PLAN_BWD_SECOND))
    assert (p.tile, q.tile, q.launches) == (first, second, launches)
    assert ssg.ssg_mlp_gemm_route(blk.desc, ssg.SSG_PLAN_BWD_SECOND).dx_form == form
    for t in (blk.dx, blk.dW1, blk.dW2, blk.dW3):
        t.fill_(float("nan"))
    blk.work.fill_(0x7F)
    blk.fwd()
    blk.bwd()
    _check_backward(blk, mode == ssg.SSG_SCALE_DELAYED)
    # the ranges of dY, dU, dG of this call, in the history
    words = state[: 6 * 32 * 4].view(torch.float32).view(6, 32)
    for k, v in ((3, blk.dY), (4, blk.wv("dU", (T, f), torch.bfloat16)), (5, blk.wv("dG", (T, f), torch.bfloat16))):
        assert float(words[k, 2]) == float(v.float().abs().max()), k


def test_the_recorded_launches_are_those_of_the_plan():
    """One event pair per launch: the split of the gate/up GEMM is two, the groups one each."""
    T, d, f = 1728, 784, 5856
    blk = _training(T, d, f)
    plan = [ssg.ssg_mlp_gemm_plan(blk.desc, w).launches for w in range(4)]
    assert plan[0] == 2 and plan[2:] == [1, 1]
    ssg.ssg_profile_select(-1)
    ssg.ssg_profile_enable(64)
    try:
        blk.fwd()
        blk.bwd()
        _, tags = ssg.ssg_profile_read(64)
    finally:
        ssg.ssg_profile_enable(0)
    assert [tags.count(t) for t in (18, 0, 16, 17)] == plan
