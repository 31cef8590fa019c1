"""A GBS step is one launch whose last workgroup waits for the partial sums of the others: sizes around one, a full
and more than a full workgroup grid, scratch memory that holds garbage or the partials of an earlier step with the
same sums, and the two-launch form that is captured into graphs."""
import pytest
import torch

import paper_2505_18663_amd as dvdq

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _l1(cur, prev):
    c, p = cur.double(), prev.double()
    return float((c - p).abs().sum() / p.abs().sum())


@pytest.mark.parametrize("n", [1, 4095, 4096, 4097, 8 * 512 * 511 + 3, 8 * 512 * 512, 8 * 512 * 512 * 2 + 9])
def test_steps_on_garbage_scratch(n):
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    f = [torch.randn((n,), generator=g, device=DEV).to(torch.bfloat16) for _ in range(3)]
    ctl = dvdq.GbsController(delta=1e9)
    ctl.workspace.copy_(torch.randint(0, 256, ctl.workspace.shape, generator=g, device=DEV, dtype=torch.uint8))
    total = 0.0
    for i in range(12):
        # (the same pairs again and again: what lies in the scratch is a partial with the same sums)
        cur, prev = f[(i // 4 + 1) % 3], f[i // 4 % 3]
        ctl.step(cur, prev)
        total += _l1(cur, prev)
        acc, l1, bits = ctl.read()
        # fp32 sums of up to 64 bf16 terms a lane, then of 64 lanes: 70 roundings of 2^-24 at most, mostly cancelling
        assert abs(l1 - _l1(cur, prev)) <= 4e-6 * l1 and abs(acc - total) <= 4e-6 * total and bits == 4


def test_zero_difference_after_zero_output():
    """num == den == 0, then num == den: the words of the partials differ from the old ones by the same bits"""
    z, o = torch.zeros(100000, dtype=torch.bfloat16, device=DEV), torch.ones(100000, dtype=torch.bfloat16, device=DEV)
    ctl = dvdq.GbsController(delta=1e9)
    for _ in range(5):
        ctl.step(z, z)
        assert ctl.read()[1] == 0.0
        ctl.step(z, o)
        assert ctl.read()[1] == 1.0


def test_captured_steps_replay():
    n = 300001
    cur, prev = (torch.randn(n, device=DEV).to(torch.bfloat16) for _ in range(2))
    ctl, ref = dvdq.GbsController(delta=1e9), dvdq.GbsController(delta=1e9)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        ctl.step(cur, prev)
    for i in range(4):
        cur.copy_(torch.randn(n, device=DEV))
        graph.replay()
        ref.step(cur, prev)
        torch.cuda.synchronize()
        assert ctl.read() == ref.read()


@pytest.mark.parametrize("n", [1, 8 * 512 * 512 + 3])
def test_a_step_without_its_partial_sums_says_so(n):
    """what happens when another step overwrites the scratch: no number, the higher bit-width, the sum kept; later steps
    are not affected"""
    cur, prev = (torch.randn(n, device=DEV).to(torch.bfloat16) for _ in range(2))
    ctl = dvdq.GbsController(delta=1e9, b_low=4, b_high=6)
    ctl.step(cur, prev)
    acc, l1, bits = ctl.read()
    assert bits == 4 and acc > 0
    try:
        dvdq.bench_set_gbs_wait(100000)   # one millisecond
        ctl.step(cur, prev)
        lost = ctl.read()
    finally:
        dvdq.bench_set_gbs_wait(-1)
    assert lost[0] == acc and lost[1] != lost[1] and lost[2] == 6
    ctl.step(cur, prev)
    assert ctl.read() == (acc + acc, l1, 4)
