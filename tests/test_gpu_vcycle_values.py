"""One V-cycle's iterate, node by node, against the same cycle in float64.

The steps of the other multigrid tests end converged, and the smoother and the line search
repair much on the way there: a value wrong at a tile's seam or in a doubled last row
would cost a few cycles and pass.  Here a step makes one cycle.  The fields stay well
inside the simplex, so no truncation depends on a rounding.

Tolerance: a nodal value is a sum of five products with values in [0, 1], 2e-7 of rounding
each half-sweep, which the next ones average: 1.5e-6 after at most eight.  The correction
solves for a defect of that rounding times D, which is independent from node to node, so the
coarse levels average it: 1e-5 covers both.  Planted mistakes are 1e-4 and more (below).
"""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_0710_0736_amd import acseg

TOL = 1e-5
EPS, TAU, LAM = 20.0, 5.0, 0.05  # kappa times the neighbours' weights: 0.9975


def classes(W, H):
    """Lumped-mass weights and stiffness diagonals of the nodes (h = 1)."""
    w, a = np.ones((H, W)), np.full((H, W), 4.0)
    for s in (np.s_[0], np.s_[-1], np.s_[:, 0], np.s_[:, -1]):
        w[s], a[s] = 0.5, 2.0
    for y, x, m in ((0, 0, 1 / 3), (-1, -1, 1 / 3), (0, -1, 1 / 6), (-1, 0, 1 / 6)):
        w[y, x], a[y, x] = m, 1.0
    return w, a


class Level:
    def __init__(self, W, H, l):
        w, a = classes(W, H)
        self.W, self.H, self.D = W, H, 4.0 ** l * w / TAU + EPS * a
        self.P = orc.Params(H=H, W=W, C=1, N=1, h=2.0 ** l, eps=EPS, lam=0.0, tau=TAU)
        self.red = np.add.outer(np.arange(H), np.arange(W)) % 2 == 0

    def apply(self, v):
        return np.stack([orc.apply_H(self.P, x[None])[0] for x in v])

    def sweeps(self, v, r, n):
        for _ in range(n):
            for m in (self.red, ~self.red):
                v = np.where(m, v + (r - self.apply(v)) / self.D, v)
        return v


def project(y):
    s = -np.sort(-y, axis=0)
    k = np.arange(1, len(y) + 1).reshape(-1, *[1] * (y.ndim - 1))
    return np.maximum(y - ((np.cumsum(s, 0) - 1) / k).max(0), 0)


def coarse_sweeps(lev):
    rho = (EPS * classes(lev.W, lev.H)[1] / lev.D).max()
    return int(min(max(np.ceil(24 * np.log(2) / -np.log(rho)), 1), 8))


def correct(lv, l, r, nu, spoil):
    """Approximate solution of H_l v = r by a V-cycle of nu sweeps from zero down and up."""
    v = np.zeros_like(r)
    if l == len(lv) - 1:
        return lv[l].sweeps(v, r, coarse_sweeps(lv[l]))
    v = lv[l].sweeps(v, r, nu)
    rc = spoil(l + 1, orc.restrict(r - lv[l].apply(v)))
    v = v + orc.prolong(correct(lv, l + 1, rc, nu, spoil), lv[l].W, lv[l].H)
    return lv[l].sweeps(v, r, nu)


def cycle(u, b, lv, nu, extra, spoil=lambda l, r: r):
    """u after one cycle: nu sweeps, the correction, nu + extra sweeps."""
    f = lv[0]

    def smooth(u, n):
        for _ in range(n):
            for m in (f.red, ~f.red):
                u = np.where(m, project(u + (b - f.apply(u)) / f.D), u)
        return u

    u = smooth(u, nu)
    assert u.min() > 0.02  # every phase free at every node
    tangent = lambda x: x - x.mean(0)
    g = tangent(b - f.apply(u))
    v = correct(lv, 1, spoil(1, orc.restrict(g)), nu, spoil)
    w = project(u + tangent(orc.prolong(v, f.W, f.H))) - u
    alpha = np.clip((g * w).sum() / (w * f.apply(w)).sum(), 0, 1)
    u = smooth(np.maximum(u + alpha * w, 0), nu + extra)
    assert u.min() > 0.02
    return u


def setup(W, H, N, levels, seed):
    rng = np.random.default_rng(seed)
    x, y = np.meshgrid(np.linspace(0, 1, W), np.linspace(0, 1, H))
    img = (0.5 + 0.5 * np.sin(3 * x + 2 * y) + 0.1 * rng.random((H, W)))[None].astype(np.float32)
    u0 = 1 + 0.3 * rng.random((N, H, W)) + 0.3 * np.stack([np.cos(2 * x + i) * np.cos(y + 2 * i) for i in range(N)])
    u0 = (u0 / u0.sum(0)).astype(np.float32)
    P = orc.Params(H=H, W=W, C=1, N=N, h=1.0, eps=EPS, lam=LAM, tau=TAU)
    b = orc.rhs(P, img, u0, orc.colour_means(P, img, u0)[0])
    lv = [Level(W, H, 0)]
    for l in range(1, levels or orc.auto_levels(W, H)):
        lv.append(Level((lv[-1].W + 1) // 2, (lv[-1].H + 1) // 2, l))
    return img, u0, b, lv, P


# level 1 at the edges of the down and up passes' tiles (see test_gpu_mg_tiles.py) and inside the tail
CASES = [(224, 48, 2, 1, 0), (225, 49, 3, 1, 0), (242, 230, 4, 1, 0), (140, 5, 4, 1, 0), (4, 180, 2, 1, 0),
         (208, 82, 2, 2, 0), (210, 170, 8, 2, 0), (150, 140, 2, 3, 0), (128, 128, 5, 1, 0), (63, 61, 7, 1, 0),
         (64, 3, 6, 2, 0), (300, 190, 3, 1, 2), (131, 130, 4, 2, 3), (34, 33, 2, 1, 2)]


def test_reference_converges_to_the_oracles_step():
    img, u0, b, lv, P = setup(70, 41, 3, 0, 1)
    u = u0.astype(np.float64)
    for _ in range(30):
        u = cycle(u, b, lv, 1, 1)
    ref, _, st = orc.step(P, img, u0)
    assert st["converged"] and np.abs(u - ref).max() < 1e-8


@pytest.mark.parametrize("level,where", [(1, np.s_[:, 8, :]), (1, np.s_[:, :, -1]), (1, np.s_[:, -1, :]), (2, np.s_[:, :, 20])],
                         ids=["seam", "last_column", "last_row", "level2"])
def test_planted_mistakes_show(level, where):
    img, u0, b, lv, _ = setup(224, 48, 2, 0, 224)

    def spoil(l, r):
        if l == level:
            r = r.copy()
            r[where] *= 0.5
        return r

    u = u0.astype(np.float64)
    assert np.abs(cycle(u, b, lv, 1, 1, spoil) - cycle(u, b, lv, 1, 1)).max() > 10 * TOL


@pytest.mark.gpu
@pytest.mark.parametrize("W,H,N,nu,levels", CASES)
def test_one_cycle_matches_float64(W, H, N, nu, levels):
    img, u0, b, lv, _ = setup(W, H, N, levels, W)
    ref = cycle(u0.astype(np.float64), b, lv, nu, 1 if nu == 1 else 0)
    p = acseg.Problem(H=H, W=W, C=1, N=N, h=1.0, eps=EPS, lam=LAM, tau=TAU, steps=1, levels=levels, nu_pre=nu,
                      nu_post=nu, max_cycles=1, flags=acseg.FLAG_FIXED_CYCLES)
    image, field = torch.from_numpy(img).cuda(), torch.from_numpy(u0).cuda()
    u, _, _, _ = acseg.solve(p, image, field.clone())
    us, _, _ = acseg.solve_batched([p] * 2, [image] * 2, [field.clone(), field.clone()])
    err = np.abs(u.cpu().numpy() - ref)
    assert err.max() <= TOL, (err.max(), np.unravel_index(err.argmax(), err.shape))
    assert torch.equal(us[0], u) and torch.equal(us[1], u)
