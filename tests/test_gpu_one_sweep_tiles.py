"""A step's only launch with seven and eight phases and three or four channels takes four
rows per lane above 256 tiles also when it makes one sweep or is over-relaxed: a batch of
more tiles gives its images the bits they get alone (two rows per lane), and a single
image of more tiles the oracle's step."""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_0710_0736_amd import acseg, synth
from test_gpu_parity import GATE_U, cuda, host, orc_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nu,flags", [((1, 0), 0), ((1, 0), acseg.FLAG_SOR), ((1, 1), acseg.FLAG_SOR)],
                         ids=["one", "one_sor", "two_sor"])
@pytest.mark.parametrize("N,C", [(7, 3), (7, 4), (8, 3), (8, 4)])
def test_batch_equals_single(N, C, nu, flags):
    W, H, B = 301, 290, 4  # 6 x 13 tiles each
    g = torch.Generator().manual_seed(100 * N + C)
    p = acseg.Problem(H=H, W=W, C=C, N=N, h=1.0, eps=1.5, tau=10.0, lam=1.0, steps=3, levels=1, nu_pre=nu[0],
                      nu_post=nu[1], max_cycles=1, flags=acseg.FLAG_FIXED_CYCLES | flags)
    images = [torch.rand((C, H, W), generator=g).cuda() for _ in range(B)]
    u0 = [torch.rand((N, H, W), generator=g).cuda() for _ in range(B)]
    us, cs, _ = acseg.solve_batched([p] * B, images, [u.clone() for u in u0])
    for b in range(B):
        u, c, _, _ = acseg.solve(p, images[b], u0[b].clone())
        assert torch.equal(u, us[b]) and torch.equal(c, cs[b])


@pytest.mark.parametrize("flags", [0, acseg.FLAG_SOR], ids=["gs", "sor"])
@pytest.mark.parametrize("N", [7, 8])
def test_single_image_step(N, flags):
    w = synth.Workload("one_sweep", 898, 397, N, "voronoi", sigma=0.1, lam=100.0, steps=1, levels=0, tol=1e-6)
    img, u0, _ = w.make(N)  # 17 x 17 tiles
    P = orc_params(w, tol=1e-12, levels=0)
    u_ref, c_ref, _ = orc.step(P, img, u0.astype(np.float32), None)
    p = acseg.Problem.from_workload(w, levels=1, nu_pre=1, nu_post=0, max_cycles=50, flags=flags)
    u, c, st = acseg.step(p, cuda(img), cuda(u0))
    assert st["status"] == acseg.OK, st
    assert np.abs(host(u) - u_ref).max() <= GATE_U
    assert np.abs(host(c) - c_ref).max() < 1e-5
