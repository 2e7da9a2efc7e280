"""A node rounds alike wherever it lies in a tile, and lambda's gradient is as close
as its terms allow.

Turning a lattice by 180 degrees keeps every node's class and, for even W + H, its colour, and
swaps its neighbours in pairs, whose sums commute; the tiles do not turn with it.  So with
fixed colour means (their sums depend on the order) the turned problem has the turned
result bit for bit, and the sums of the gradients differ by the order of float64 additions.
"""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_0710_0736_amd import acseg
from test_gpu_parity import cuda, host

pytestmark = pytest.mark.gpu


def made(N, C, W, H, seed, pixel):
    r = np.random.Generator(np.random.PCG64(seed))
    e = r.exponential(size=(N, H, W)) + 1e-9
    h = 1.0 if pixel else 1.0 / (max(W, H) - 1)
    P = dict(H=H, W=W, C=C, N=N, h=h, eps=2 * h, tau=4 * h * h, lam=1.0 if pixel else 100.0)
    return P, cuda(r.random((C, H, W))), cuda(e / e.sum(0)), cuda(r.random((N, C))), cuda(r.standard_normal((N, H, W)))


def turned(t):
    return t.flip(-1, -2).contiguous()


@pytest.mark.parametrize("pixel", [False, True], ids=["unit", "pixel"])
@pytest.mark.parametrize("N,C", [(2, 1), (3, 3), (4, 3), (5, 4), (6, 2), (7, 3), (8, 4)])
def test_turned_lattice_has_the_turned_result(N, C, pixel):
    for W, H in ((131, 77), (60, 28), (2, 58)):
        P, image, u0, c, gT = made(N, C, W, H, N, pixel)
        for flags in (0, acseg.FLAG_SOR):
            p = acseg.Problem(**P, steps=3, levels=1, max_cycles=2, flags=flags | acseg.FLAG_FIXED_CYCLES)
            u, _, st, ck = acseg.solve(p, image, u0.clone(), checkpoints=True, c_fixed=c)
            v, _, sv, kv = acseg.solve(p, turned(image), turned(u0), checkpoints=True, c_fixed=c)
            assert torch.equal(kv, turned(ck)), (W, H, flags)
            assert sv["final_residual"] == st["final_residual"]
        p = acseg.Problem(**P, steps=3, levels=1, max_cycles=200)
        gI, gu0, gp, _, bst = acseg.backward(p, image, ck, gT, c_fixed=c)
        hI, hu0, hp, _, bsv = acseg.backward(p, turned(image), kv, turned(gT), c_fixed=c)
        assert bst["cycles_total"] == bsv["cycles_total"]
        assert torch.equal(hI, turned(gI)) and torch.equal(hu0, turned(gu0)), (W, H)
        assert float((hp - gp).abs().max()) <= 1e-9 * float(gp.abs().max())


@pytest.mark.parametrize("seed", range(8))
def test_lambda_gradient_in_units_of_its_terms(seed):
    """One step back: z is within rtol = 1e-6 of its largest value (the stopping rule) plus
    rounding, so the sum of z M F is within that of the sums of its terms."""
    P, image, u0, _, gT = made(4, 3, 131, 77, 100 + seed, False)
    p = acseg.Problem(**P, steps=1, levels=1, max_cycles=100)
    u, _, _, ck = acseg.solve(p, image, u0.clone(), checkpoints=True)
    _, _, gp, _, _ = acseg.backward(p, image, ck, gT)
    Q = orc.Params(**P, tol=1e-12)
    I = host(image)
    c, _ = orc.colour_means(Q, I, host(ck[0]))
    z = orc.adjoint_solve(Q, host(ck[1]), host(gT))
    w = np.ones((Q.H, Q.W))
    w[[0, -1]] *= 0.5
    w[:, [0, -1]] *= 0.5
    w[0, 0] = w[-1, -1] = 1 / 3
    w[0, -1] = w[-1, 0] = 1 / 6
    MF = Q.h ** 2 * w * ((I[None] - c[:, :, None, None]) ** 2).sum(1)
    bound = 1e-6 * np.abs(z).max() * MF.sum() + 1e-6 * np.abs(z * MF).sum()
    assert abs(float(gp[0]) + (z * MF).sum()) <= bound
