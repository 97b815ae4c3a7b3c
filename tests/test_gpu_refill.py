"""A refill threshold meant for two rays per lane, given to the walks that have one."""
import numpy as np
import pytest

from workloads import meshes as M
from workloads.rays import random_rays, uniform_len

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_two_ray_threshold_in_one_ray_walks():
    from paper_2603_15780_amd import sg
    X, F = M.canonical(*M.icosphere(3))
    r = random_rays(X, F, 3001, np.random.default_rng(2), uniform_len(0.0, 2.0), K=0)
    t = [torch.from_numpy(r[k]).cuda() for k in ("f", "b", "v")]
    g = torch.from_numpy(np.random.default_rng(3).standard_normal((3001, 3)).astype(np.float32)).cuda()
    mesh, kw = sg.Mesh(X, F), dict(rays_per_lane=2, refill_min=96)
    a, b = mesh.exp(*t), mesh.exp(*t, kernel=sg.KERNEL_PARTITIONED, **kw)
    assert all(torch.equal(a[k], b[k]) for k in ("f", "b", "p", "v"))
    for x, y in zip(mesh.backward(sg.BWD_GFD, *t, g), mesh.backward(sg.BWD_GFD, *t, g, **kw)):
        assert torch.equal(x, y)
    gx = [torch.zeros(mesh.n_verts, 3, dtype=torch.float64, device="cuda") for _ in range(2)]
    for o, k in zip(gx, ({}, kw)):
        mesh.backward(sg.BWD_EP, *t, g, grad_X=o, want_vjp=False, **k)
    assert torch.allclose(*gx, rtol=1e-9, atol=1e-9 * gx[0].abs().max().item())   # (the sums' order)
