"""The energy at the most phases and channels, and with few, against float64 sums."""
import numpy as np
import pytest
import torch

from paper_0710_0736_amd import acseg

pytestmark = pytest.mark.gpu


def reference(p, image, u):
    """Interface, concave and fitting parts in float64 (lumped mass, edge weights 1/2 on the boundary)."""
    N, H, W = u.shape
    w = np.ones((H, W))
    w[0], w[-1] = 0.5, 0.5
    w[:, 0], w[:, -1] = 0.5, 0.5
    w[0, 0] = w[-1, -1] = 1 / 3
    w[0, -1] = w[-1, 0] = 1 / 6
    ch = np.ones((H, 1))
    ch[0] = ch[-1] = 0.5
    cv = np.ones((1, W))
    cv[:, 0] = cv[:, -1] = 0.5
    S = (w * u).sum((1, 2))
    c = np.einsum("nhw,chw->nc", w * u, image) / S[:, None]
    grad = (ch * np.diff(u, axis=2) ** 2).sum() + (cv * np.diff(u, axis=1) ** 2).sum()
    F = ((image[None] - c[:, :, None, None]) ** 2).sum(1)
    h2 = p.h * p.h
    e = np.array([0.5 * p.eps * grad, h2 / p.eps * (w * u * (1 - u)).sum(), p.lam * h2 * (w * u * F).sum()])
    return np.append(e, e.sum())


@pytest.mark.parametrize("W,H", [(2, 2), (3, 7), (257, 129), (1023, 517)])
@pytest.mark.parametrize("N,C", [(2, 1), (4, 3), (8, 3), (8, 4)])
def test_energy_matches_float64(N, C, W, H):
    rng = np.random.default_rng(31 * N + C + W)
    image = rng.random((C, H, W)).astype(np.float32)
    u = rng.random((N, H, W))
    u = (u / u.sum(0)).astype(np.float32)
    p = acseg.Problem(H=H, W=W, C=C, N=N, h=0.5, eps=1.25, tau=1.0, lam=7.0)
    e = acseg.energy(p, torch.from_numpy(image).cuda(), torch.from_numpy(u).cuda()).cpu().numpy()
    # sums of up to 16 nodes per thread and then a tree, in float64; only e[1] has terms of both signs (none here)
    assert np.allclose(e, reference(p, image.astype(np.float64), u.astype(np.float64)), rtol=1e-12, atol=0)


@pytest.mark.parametrize("x,y", [(4, 2), (0, 2), (2, 4), (3, 0), (4, 4), (0, 0)])
def test_infinite_value_at_the_boundary(x, y):
    """Its edges inside the lattice make the interface part infinite; there is none beyond."""
    u = torch.full((2, 5, 5), 0.5)
    u[0, y, x] = float("inf")
    p = acseg.Problem(H=5, W=5, C=1, N=2, h=1.0, eps=1.0, tau=1.0, lam=1.0)
    e = acseg.energy(p, torch.rand((1, 5, 5)).cuda(), u.cuda())
    assert torch.isposinf(e[0]), e
