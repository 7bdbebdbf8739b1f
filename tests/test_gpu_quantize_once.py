"""GPU parity of ssg_quantize in one launch (workgroups keep their tiles and exchange their ranges) with the separate range and cast
launches, at the edges of what a workgroup and the chip hold, with any number of looks at the others' ranges, under capture
(which takes the separate launches) and on two streams at once."""
import time

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2409_12517_amd as ssg  # noqa: E402
import gpu_util as gu  # noqa: E402

FMAX = {ssg.SSG_E4M3: 448.0, ssg.SSG_E5M2: 57344.0}
# tiles of 128 x 128: one, a cut one, rows and columns left over; 256 and 257 workgroups' worth (1 and 2 tiles each); 3 and 4 tiles
# each; the most that bf16 (12 each) and fp32 (6) hold, and one row of tiles more, which takes two launches
SHAPES = [(16, 16, 0), (128, 128, 0), (144, 1040, 0), (2048, 2048, 0), (2064, 2048, 0), (6144, 2048, 0), (6160, 2032, 0),
          (4096, 12288, 0), (4112, 12288, 0), (16, 16, 1), (144, 1040, 1), (2064, 2048, 1), (4096, 6144, 1), (4112, 6144, 1)]


def _source(rows, cols, f32, seed):
    gen = torch.Generator(device=gu.DEV).manual_seed(seed)
    src = torch.randn(rows, cols, generator=gen, device=gu.DEV) * 0.02
    src = src if f32 else src.to(torch.bfloat16)
    src[rows - 1, cols - 3], src[rows // 2, 5], src[0, 0] = 0.75, float("nan"), -0.0
    return src


def _run(src, fmt, transposed, mode, polls, scale=None):
    rows, cols = src.shape
    q, qt = gu.empty_u8(rows, cols), gu.empty_u8(cols, rows) if transposed else None
    sc, am = torch.full((1,), scale or 0.0, device=gu.DEV), gu.empty_f32(1)
    dt = ssg.SSG_F32 if src.dtype == torch.float32 else ssg.SSG_BF16
    ssg.ssg_quantize_wait(src, dt, rows, cols, fmt, mode, ssg.SSG_ROUND_EXACT_DIV, q, qt, sc, am, polls)
    return q, qt, sc, am


@pytest.mark.parametrize("rows,cols,f32", SHAPES)
@pytest.mark.parametrize("fmt,transposed", [(ssg.SSG_E4M3, True), (ssg.SSG_E5M2, False)])
def test_one_launch_equals_range_and_cast(rows, cols, f32, fmt, transposed):
    src = _source(rows, cols, f32, rows + cols)
    amax = np.float32(torch.nan_to_num(src.float(), nan=0.0).abs().max().item())
    scale = np.float32(FMAX[fmt]) / amax
    # a given scale: the cast alone
    ref_q, ref_qt, _, _ = _run(src, fmt, transposed, ssg.SSG_SCALE_GIVEN, -1, float(scale))
    for polls in (-1, 0, 1):
        q, qt, sc, am = _run(src, fmt, transposed, ssg.SSG_SCALE_CURRENT, polls)
        assert gu.scalar(sc) == scale and gu.scalar(am) == amax, polls
        assert torch.equal(q, ref_q) and (not transposed or torch.equal(qt, ref_qt)), polls


def test_a_captured_call_follows_its_input():
    rows, cols = 272, 1040
    src, q, qt = _source(rows, cols, 0, 1), gu.empty_u8(rows, cols), gu.empty_u8(cols, rows)
    sc, am = gu.empty_f32(1), gu.empty_f32(1)

    def call(stream=None):
        ssg.ssg_quantize(src, ssg.SSG_BF16, rows, cols, ssg.SSG_E4M3, ssg.SSG_SCALE_CURRENT, ssg.SSG_ROUND_EXACT_DIV, q, qt, sc, am)

    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for k in range(4):
        src.copy_(_source(rows, cols, 0, 10 + k) * (k + 1))
        q.zero_()
        graph.replay()
        torch.cuda.synchronize()
        got = q.clone(), qt.clone(), gu.scalar(sc), gu.scalar(am)
        call()
        torch.cuda.synchronize()
        assert torch.equal(got[0], q) and torch.equal(got[1], qt) and got[2:] == (gu.scalar(sc), gu.scalar(am)), k


def test_four_streams_at_once():
    """Launches that hold the whole chip each, enqueued by turns and 64 in a row (rows of words shared): the results of one alone, and
    no call waits long for workgroups that cannot come onto the chip (11 times as long as alone once, less than 2 now)."""
    rows, cols = 4096, 11008
    srcs = [_source(rows, cols, 0, 40 + k) for k in range(4)]
    refs = [_run(s, ssg.SSG_E4M3, True, ssg.SSG_SCALE_CURRENT, -1) for s in srcs]
    outs = [[torch.empty_like(t) for t in r] for r in refs]
    streams = [torch.cuda.Stream() for _ in range(4)]

    def call(k):
        q, qt, sc, am = outs[k]
        with torch.cuda.stream(streams[k]):
            ssg.ssg_quantize(srcs[k], ssg.SSG_BF16, rows, cols, ssg.SSG_E4M3, ssg.SSG_SCALE_CURRENT, ssg.SSG_ROUND_EXACT_DIV, q, qt, sc, am)

    def seconds(order):
        torch.cuda.synchronize()
        begun = time.perf_counter()
        for k in order:
            call(k)
        torch.cuda.synchronize()
        return (time.perf_counter() - begun) / len(order)

    seconds([0] * 20)
    alone = min(seconds([0] * 64) for _ in range(3))
    for order in ([0, 1, 2, 3] * 16, [0] * 64 + [1] * 64):
        assert min(seconds(order) for _ in range(3)) < 5 * alone
        for k in set(order):
            assert all(torch.equal(a, b) for a, b in zip(outs[k], refs[k]))
            for t in outs[k]:
                t.zero_()


def test_two_streams_at_once():
    rows, cols = 2048, 4096
    srcs = [_source(rows, cols, 0, 20 + k) for k in range(2)]
    refs = [_run(s, ssg.SSG_E4M3, True, ssg.SSG_SCALE_CURRENT, -1) for s in srcs]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    outs = []
    for _ in range(20):
        for k in range(2):
            with torch.cuda.stream(streams[k]):
                outs.append((k, _run(srcs[k], ssg.SSG_E4M3, True, ssg.SSG_SCALE_CURRENT, -1)))
    torch.cuda.synchronize()
    for k, out in outs:
        assert all(torch.equal(a, b) for a, b in zip(out, refs[k]))
