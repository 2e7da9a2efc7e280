"""Every update leaves its node on the Gibbs simplex, whatever it started from.

u^0 need not lie on the simplex (an unnormalised field, a half-precision softmax,
zeros), and the coupling may be close to one.  Sums are compared with one within
N 2^-23: the threshold's partial sums and the N differences each round at 2^-24.
A fixed schedule is compared with the same sweeps in float64: each of its half-sweeps
rounds N + 8 operations of order-one values at 2^-24, 2e-5 for up to 12 of them.
"""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_0710_0736_amd import acseg
from test_gpu_parity import cuda, host

pytestmark = pytest.mark.gpu

W, H, C = 121, 57, 3  # tiles at the border and one inside
STARTS = {"half": 0.5, "almost": 0.996, "more": 1.2, "zero": 0.0}


def field(N, seed, scale=1.0):
    r = np.random.Generator(np.random.PCG64(seed))
    e = r.exponential(size=(N, H, W)) + 1e-9
    return (scale * e / e.sum(0)).astype(np.float32), r.random((C, H, W)).astype(np.float32)


def problem(N, **kw):
    kw = {"h": 1.0, "eps": 2.0, "tau": 4.0, "lam": 1.0, "steps": 1, "levels": 1, "tol": 1e-6, **kw}
    return acseg.Problem(H=H, W=W, C=C, N=N, **kw)


def project(v):
    s = -np.sort(-v, axis=0)
    t = (np.cumsum(s, 0) - 1.0) / np.arange(1, v.shape[0] + 1)[:, None, None]
    return np.maximum(v - t.max(0), 0.0)


def diagonal(P):
    d = np.empty((H, W))
    for y in range(2):
        for x in range(2):  # nodes of one class of (x mod 2, y mod 2) are no neighbours of each other
            e = np.zeros((P.N, H, W))
            e[0, y::2, x::2] = 1.0
            d[y::2, x::2] = orc.apply_H(P, e)[0, y::2, x::2]
    return d


def sweeps(P, image, u0, cycles, sor):
    """`cycles` cycles of two red-black sweeps; the last black half-sweep of a cycle is plain."""
    c, _ = orc.colour_means(P, image, u0)
    b = orc.rhs(P, image, u0, c)
    d = diagonal(P)
    e2 = P.eps / P.h ** 2
    q = min(max(4 * e2 / (1 / P.tau + 4 * e2), 2 * e2 / (0.5 / P.tau + 2 * e2), e2 / (1 / 3 / P.tau + e2),
                e2 / (1 / 6 / P.tau + e2)), 0.999)
    om = min(1.95, 2.0 / (1.0 + np.sqrt(1.0 - q * q))) if sor else 1.0
    red = (np.arange(H)[:, None] + np.arange(W)[None, :]) % 2 == 0
    u = u0.astype(np.float64)
    for s in range(2 * cycles):
        for mask in (red, ~red):
            w = 1.0 if s % 2 == 1 and mask is not red else om
            y = u + (b - orc.apply_H(P, u)) / d
            u = np.where(mask, project(u + w * (y - u)), u)
    return u, b


@pytest.mark.parametrize("sor", [False, True], ids=["gs", "sor"])
@pytest.mark.parametrize("N", [2, 3, 4, 5, 8])
def test_fixed_sweeps_from_any_start(N, sor):
    P = orc.Params(H=H, W=W, C=C, N=N, h=1.0, eps=2.0, lam=1.0, tau=4.0)
    flags = acseg.FLAG_FIXED_CYCLES | (acseg.FLAG_SOR if sor else 0)
    for cycles in (1, 3):
        p = problem(N, max_cycles=cycles, flags=flags)
        for name, scale in STARTS.items():
            u0, image = field(N, N + cycles, scale)
            ref, b = sweeps(P, image, u0, cycles, sor)
            u, _, st, _ = acseg.solve(p, cuda(image), cuda(u0))
            ug = host(u)
            assert np.abs(ug.sum(0) - 1.0).max() <= N * 2.0 ** -23, (name, cycles)
            assert np.abs(ug - ref).max() <= 2e-5, (name, cycles)
            assert abs(st["final_residual"] - orc.residual(P, b, ug)) <= 2e-5, (name, cycles, st)


@pytest.mark.parametrize("levels", [1, 0], ids=["gs", "mg"])
@pytest.mark.parametrize("N", [4, 7])
def test_batch_from_any_start(N, levels):
    """Single and batched solves: on the simplex and the same bits."""
    for cycles in (1, 2):
        p = problem(N, steps=2, levels=levels, max_cycles=cycles, flags=acseg.FLAG_FIXED_CYCLES)
        made = [field(N, k, s) for k, s in enumerate(STARTS.values())]
        us, _, _ = acseg.solve_batched([p] * len(made), [cuda(i) for _, i in made], [cuda(u) for u, _ in made])
        for (u0, image), ub in zip(made, us):
            u, _, _, _ = acseg.solve(p, cuda(image), cuda(u0))
            assert torch.equal(u, ub)
            assert np.abs(host(u).sum(0) - 1.0).max() <= N * 2.0 ** -23


@pytest.mark.parametrize("N", [3, 4, 8])
def test_sums_with_the_coupling_close_to_one(N):
    for eps, tau in ((50.0, 1e4), (400.0, 1e6)):
        p = problem(N, eps=eps, tau=tau, lam=0.001, steps=2, max_cycles=60)
        u0, image = field(N, 3)
        u, _, _, _ = acseg.solve(p, cuda(image), cuda(u0))
        assert np.abs(host(u).sum(0) - 1.0).max() <= N * 2.0 ** -23


def test_step_from_a_half_precision_softmax():
    N = 4
    _, image = field(N, 1)
    g = torch.Generator().manual_seed(0)
    u0 = torch.softmax(3 * torch.randn((N, H, W), generator=g), 0).half().float()
    P = orc.Params(H=H, W=W, C=C, N=N, h=1.0, eps=2.0, lam=1.0, tau=4.0, tol=1e-12)
    ref, _, _ = orc.step(P, image, u0.numpy())
    u, _, st = acseg.step(problem(N, max_cycles=400), cuda(image), u0.cuda())
    assert st["status"] == acseg.OK
    assert np.abs(host(u) - ref).max() <= 1e-4  # the tolerance over one minus the contraction
    assert np.abs(host(u).sum(0) - 1.0).max() <= N * 2.0 ** -23
