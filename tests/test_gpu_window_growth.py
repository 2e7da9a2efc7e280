"""A step that needs many more cycles than the ones before it gets them in few reads of
the control block: increments double, so a shortfall of d cycles takes at most
ceil(log2(d + 1)) reads (up to 64 cycles each)."""
from dataclasses import replace
from math import ceil, log2

import torch
import pytest

from paper_0710_0736_amd import acseg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lam,amp", [(1e4, 1e-7), (1e3, 1e-6)])
def test_reads_grow_with_the_logarithm_of_the_shortfall(lam, amp):
    W, H, N, C, steps = 61, 47, 3, 3, 3
    g = torch.Generator().manual_seed(0)
    image = torch.rand((C, H, W), generator=g).cuda()
    # phases almost alike: the first step hardly moves, a later one separates them
    u0 = (torch.full((N, H, W), 1 / N) + amp * torch.randn((N, H, W), generator=g)).cuda()
    p = acseg.Problem(H=H, W=W, C=C, N=N, h=1.0, eps=2.0, tau=4.0, lam=lam, steps=steps, levels=1, max_cycles=400)
    q = replace(p, flags=acseg.FLAG_NO_HOST_WAIT)
    runs = [acseg.solve(replace(q, steps=k), image, u0.clone()) for k in range(1, steps + 1)]
    total = [0] + [r[2]["cycles_total"] for r in runs]
    need = [b - a for a, b in zip(total, total[1:])]
    assert max(need) >= 8 * need[0], need  # the jump this test is about
    # the last guess of a call is the next one's first: one cycle after a step that has nothing to do
    acseg.step(replace(p, lam=0.0), image, torch.full((N, H, W), 1 / N).cuda())
    acseg.timing_enable(True)
    acseg.timing_read()
    u, c, st, _ = acseg.solve(p, image, u0.clone())
    ends = acseg.timing_read()["other"][0]
    acseg.timing_enable(False)
    assert torch.equal(u, runs[-1][0]) and torch.equal(c, runs[-1][1]) and st == runs[-1][2]
    bound, last = 0, [1, 1]
    for n in need:
        bound += 1 + ceil(log2(max(0, n - max(last)) + 1))
        last = [last[1], n]
    assert ends <= bound + 1, (ends, bound, need)  # and one end enqueued behind a blocked step
