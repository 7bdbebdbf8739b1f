"""GPU parity of the eight-value encode where a group holds what takes its rare branch (NaN of either sign, infinities, overflow at
each place of eight), in every launch that casts a whole tensor, and of the SwiGLU product with 64 bits."""
import numpy as np
import pytest
import torch

from oracle import fp8

pytestmark = pytest.mark.gpu

import paper_2409_12517_amd as ssg  # noqa: E402
import gpu_util as gu  # noqa: E402

FMT = {ssg.SSG_E4M3: fp8.E4M3, ssg.SSG_E5M2: fp8.E5M2}


# one small launch, tiles of 16, 64 and 128 rows (up to 512, up to 4096, more tiles), and a range in the same launch
@pytest.mark.parametrize("fmt", [ssg.SSG_E4M3, ssg.SSG_E5M2])
@pytest.mark.parametrize("rows,cols,dtype", [(16, 64, torch.bfloat16), (272, 1040, torch.float32), (2064, 4096, torch.bfloat16),
                                             (8208, 8192, torch.bfloat16)])
@pytest.mark.parametrize("mode", [ssg.SSG_SCALE_GIVEN, ssg.SSG_SCALE_CURRENT])
def test_specials_at_each_place_of_eight(rows, cols, dtype, fmt, mode):
    gen = torch.Generator(device=gu.DEV).manual_seed(rows + fmt)
    src = torch.randn(rows, cols, generator=gen, device=gu.DEV)
    given = mode == ssg.SSG_SCALE_GIVEN
    special = [float("nan"), -float("nan")] + ([float("inf"), -float("inf"), 3e38, -6e4, 449.0, -1e-30] if given else [-0.0, 1e-30])
    at = []
    for i, v in enumerate(special):
        for k in range(8):                       # groups 5 apart; the first rows and the last one
            for r in (i % rows, rows - 1):
                c = (8 * (5 * i + k) + k) % cols
                src[r, c] = v
                at.append((r, c))
    src = src.to(dtype)
    q, qt = gu.empty_u8(rows, cols), gu.empty_u8(cols, rows)
    sc, am = torch.ones(1, device=gu.DEV), gu.empty_f32(1)
    ssg.ssg_quantize(src, ssg.SSG_F32 if dtype == torch.float32 else ssg.SSG_BF16, rows, cols, fmt, mode, ssg.SSG_ROUND_EXACT_DIV, q, qt, sc, am)
    assert torch.equal(qt.T, q)
    pick = sorted({r for r, _ in at} | {rows // 2})
    ref = fp8.satcast(src[pick].float().cpu().numpy() * gu.scalar(sc), FMT[fmt])
    assert np.array_equal(gu.u8(q)[pick], ref)


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
