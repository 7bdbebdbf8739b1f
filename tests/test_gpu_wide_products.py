"""GPU parity of contractions with one small tile to a compute unit, on either form of the matrix instruction: a K step in two products of
half its length, or in one.  One tile, cut tiles, K of one piece and ragged, both sides of the lines between the forms (160
tiles, whole cache lines, 16 K steps), operands of every layout and format; every element against binary64."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2409_12517_amd as ssg  # noqa: E402
import gpu_util as gu  # noqa: E402

F8 = {ssg.SSG_E4M3: torch.float8_e4m3fn, ssg.SSG_E5M2: torch.float8_e5m2}
SHAPES = [(128, 128, 128), (144, 1040, 16), (272, 400, 656), (1040, 2064, 1040), (1280, 2048, 2048), (1664, 1664, 1920), (1664, 1664, 2048),
          (1664, 1664, 2064), (1664, 1648, 2048)]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("layout", [(0, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("a_fmt,c_dtype", [(ssg.SSG_E4M3, ssg.SSG_BF16), (ssg.SSG_E5M2, ssg.SSG_F32)])
def test_contraction(M, N, K, layout, a_fmt, c_dtype):
    plan = ssg.ssg_gemm_fp8_plan(a_fmt, *layout, M, N, K, c_dtype)
    if layout != (0, 0) or M >= 1040:                         # (the smallest ones with rows along K: few-rows kernel)
        assert (plan.tile, plan.ring) == (128, 9)
    gen = torch.Generator(device=gu.DEV).manual_seed(M + N + K)
    a = torch.randn(M, K, generator=gen, device=gu.DEV).to(F8[a_fmt])
    b = torch.randn(N, K, generator=gen, device=gu.DEV).to(F8[ssg.SSG_E4M3])
    ref = (a.double() @ b.double().t()) / (2.0 * 0.5)
    A = (a.view(torch.uint8).t() if layout[0] else a.view(torch.uint8)).contiguous()
    B = (b.view(torch.uint8).t() if layout[1] else b.view(torch.uint8)).contiguous()
    sa, sb = torch.tensor([2.0], device=gu.DEV), torch.tensor([0.5], device=gu.DEV)
    dt = torch.float32 if c_dtype == ssg.SSG_F32 else torch.bfloat16
    C = torch.full((M + 1, N), -7.0, device=gu.DEV, dtype=dt)          # a row more: nothing is written past the end
    ssg.ssg_gemm_fp8_layout(A, a_fmt, layout[0], B, ssg.SSG_E4M3, layout[1], M, N, K, sa, sb, C, c_dtype)
    torch.cuda.synchronize()
    gu.assert_close_gemm(gu.f32(C[:M]), ref.cpu().numpy(), c_dtype == ssg.SSG_BF16, f"{M} {N} {K}")
    assert bool((C[M] == -7.0).all())
