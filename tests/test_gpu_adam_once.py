"""GPU parity of the Adam step in one launch (workgroups keep their share and exchange the moments' ranges) with the two launches that a
captured call takes, over several steps, at the edges of what a workgroup and the chip hold, with any number of looks at the others'
ranges, and on two streams at once."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2409_12517_amd as ssg  # noqa: E402
import gpu_util as gu  # noqa: E402

ADAM = dict(lr=3e-4, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1)
CHUNK = 256 * 2048            # one group of four per lane of the whole chip
# one element group, a cut chunk, 256 chunks and one more, more than one batch of groups, the most that the lanes hold and a chunk more
CASES = [(16, 0), (2064, 1), (CHUNK, 0), (CHUNK + 16, 1), (5 * CHUNK - 1008, 0), (8 * CHUNK, 0), (8 * CHUNK, 1), (8 * CHUNK + 16, 0)]


class Tensor:
    def __init__(self, n, bf16, seed):
        gen = torch.Generator(device=gu.DEV).manual_seed(seed)
        self.n, self.gdt = n, ssg.SSG_BF16 if bf16 else ssg.SSG_F32
        self.w = torch.randn(n, generator=gen, device=gu.DEV) * 0.02
        self.wb = torch.zeros(n, dtype=torch.bfloat16, device=gu.DEV)
        self.g = (torch.randn(n, generator=gen, device=gu.DEV) * 1e-3).to(torch.bfloat16 if bf16 else torch.float32)
        self.g[n - 1], self.g[n // 2] = 0.25, float("nan") if seed % 2 else 0.0
        self.state = torch.empty(ssg.ssg_adam_state_bytes(n), dtype=torch.uint8, device=gu.DEV)
        ssg.ssg_adam_init(n, self.state)

    def step(self, k, polls=-1):
        ssg.ssg_adam_step_wait(ssg.make_adam_desc(self.n, k, grad_dtype=self.gdt, **ADAM), self.g, self.w, self.wb, self.state, polls)

    def same(self, other):
        return all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in ((self.w, other.w), (self.wb, other.wb), (self.state, other.state)))


@pytest.mark.parametrize("n,bf16", CASES)
def test_one_launch_equals_two(n, bf16):
    """Weights, their copy and the state (codes, scales; not the slots and words in which the ranges were formed) after each of three steps."""
    ref, once = Tensor(n, bf16, n), [Tensor(n, bf16, n) for _ in range(3)]
    torch.cuda.synchronize()
    for k in (1, 2, 3):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            ref.step(k)
        graph.replay()
        for t, polls in zip(once, (-1, 0, 1)):
            t.step(k, polls)
        torch.cuda.synchronize()
        # the slots of the step's own parity hold ranges where the step was two launches; the next step clears them
        codes = ref.state.numel() - 2 * ((n + 255) // 256 * 256)
        for t in once:
            assert torch.equal(t.state[:256], ref.state[:256]) and torch.equal(t.state[codes:], ref.state[codes:]), k
            assert torch.equal(t.w.view(torch.int32), ref.w.view(torch.int32)) and torch.equal(t.wb.view(torch.int16), ref.wb.view(torch.int16)), k


def test_steps_of_both_kinds_alternate():
    """The range slots that a step in two launches leaves are cleared by the next one, of either kind."""
    n = 3 * CHUNK + 16
    a, b = Tensor(n, 0, 5), Tensor(n, 0, 5)
    torch.cuda.synchronize()
    for k in range(1, 6):
        b.g.mul_(0.5)
        a.g.mul_(0.5)
        torch.cuda.synchronize()
        a.step(k)
        if k % 2:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                b.step(k)
            graph.replay()
        else:
            b.step(k)
        torch.cuda.synchronize()
        assert torch.equal(a.w.view(torch.int32), b.w.view(torch.int32)), k


def test_many_tensors_on_one_stream_then_on_another():
    """As a program does that enqueues the steps of a group of tensors on one stream and those of another group on another: every
    exchange has words of its own.  Cut last chunks, so that workgroups have lanes without elements."""
    sizes = [16 * (1 + 37 * i) for i in range(32)] + [CHUNK // 2 + 1040 * i for i in range(32)]
    groups = [[Tensor(n, i % 3 == 0, 2 * i + s) for i, n in enumerate(sizes)] for s in range(2)]
    want = [[Tensor(n, i % 3 == 0, 2 * i + s) for i, n in enumerate(sizes)] for s in range(2)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for k in (1, 2, 3):
        for s in range(2):
            with torch.cuda.stream(streams[s]):
                for t in groups[s]:
                    t.step(k)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()                       # two launches each
        with torch.cuda.graph(graph):
            for s in range(2):
                for t in want[s]:
                    t.step(k)
        graph.replay()
        torch.cuda.synchronize()
        for s in range(2):
            for a, b in zip(groups[s], want[s]):
                codes = a.state.numel() - 2 * ((a.n + 255) // 256 * 256)
                assert torch.equal(a.state[:256], b.state[:256]) and torch.equal(a.state[codes:], b.state[codes:]), (k, s, a.n)
                assert torch.equal(a.w.view(torch.int32), b.w.view(torch.int32)) and torch.equal(a.wb.view(torch.int16), b.wb.view(torch.int16)), (k, s, a.n)


def test_two_streams_at_once():
    n = 6 * CHUNK
    pairs = [(Tensor(n, 0, 7 + s), Tensor(n, 0, 7 + s)) for s in range(2)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for k in range(1, 9):
        for s in range(2):
            with torch.cuda.stream(streams[s]):
                pairs[s][0].step(k)
    torch.cuda.synchronize()
    for s in range(2):
        for k in range(1, 9):
            pairs[s][1].step(k)
        torch.cuda.synchronize()
        assert pairs[s][0].same(pairs[s][1])
