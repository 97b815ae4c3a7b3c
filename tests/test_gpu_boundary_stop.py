"""Rays that end on a boundary edge, in every kernel: where the oracle ends them, and
in the order of a step's outcomes (the cap before the boundary)."""
import numpy as np
import pytest

import oracle
from parity import assert_parity
from workloads import meshes as M
from workloads.rays import random_rays, uniform_len

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

KERNELS = [dict(kernel=1), dict(kernel=2), dict(kernel=2, rays_per_lane=2), dict(kernel=3)]


def _holed(kind):
    if kind == "mobius":
        return M.canonical(*M.mobius_strip(40, 6))
    X, F = M.icosphere(4)
    used, out = np.zeros(len(X), bool), []
    for f in np.random.default_rng(1).permutation(len(F)):   # holes of one face that share no vertex
        if not used[F[f]].any():
            used[F[f]] = True
            out.append(f)
    return M.canonical(*M.remove_faces(X, F, out[:250]))


@pytest.mark.parametrize("kind", ["holes", "mobius"])
def test_boundary_ends(kind):
    from paper_2603_15780_amd import sg
    X, F = _holed(kind)
    r = random_rays(X, F, 4099, np.random.default_rng(13), uniform_len(0.0, 2.0), K=1)
    t, mesh, om = [torch.from_numpy(r[k]).cuda() for k in ("f", "b", "v", "W")], sg.Mesh(X, F), oracle.Mesh(X, F)
    ref, runs = om.exp(r["f"], r["b"], r["v"], r["W"]), []
    for kw in KERNELS:
        g = {k: x.cpu().numpy() if x is not None else None for k, x in mesh.exp(*t, want_cross=True, want_hash=True, **kw).items()}
        g["hash"] = g["hash"].view(np.uint64)
        assert_parity(ref, g, om.mean_edge, K=1, label=str(kw))
        runs.append(g)
        assert all(np.array_equal(g[k], runs[0][k], equal_nan=k in "bpvW") for k in g)
    ends, cross = runs[0]["status"] == sg.RAY_BOUNDARY, runs[0]["n_cross"]
    assert ends.mean() > 0.3
    for cap in (1, 3, 7):
        for kw in KERNELS:
            st = mesh.exp(*t, max_steps=cap, **kw)["status"].cpu().numpy()
            assert (st[ends & (cross >= cap)] == sg.RAY_MAXSTEPS).all()
            assert (st[ends & (cross < cap)] == sg.RAY_BOUNDARY).all()
