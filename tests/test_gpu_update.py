"""sg_mesh_update_vertices packs on the device what a new handle packs on the
host: the same records, so the same rays, at mesh sizes around the kernels'
blocks of 256 faces and vertices, with boundaries, flipped faces and several
meshes in a handle."""
import numpy as np
import pytest

from workloads import meshes as M
from workloads.rays import random_rays, uniform_len

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return pytest.importorskip("torch")


def _mesh(kind):
    g = np.random.default_rng(5)
    if kind == "tetrahedron":
        return M.canonical(*M.tetrahedron())
    if kind == "icosphere2":   # 320 faces, 162 vertices
        return M.canonical(*M.icosphere(2))
    if kind == "torus256":     # 256 faces, 128 vertices: one full block
        return M.canonical(*M.torus_grid(16, 8, 0.2, g))
    if kind == "torus258":
        return M.canonical(*M.torus_grid(43, 3, 0.2, g))
    if kind == "hole":
        return M.canonical(*M.remove_faces(*M.icosphere(3), [5, 700]))
    return M.canonical(*M.mobius_strip(40, 6))


def _run(torch, mesh, r):
    t = [torch.from_numpy(r[k]).cuda() for k in ("f", "b", "v", "W")]
    out = mesh.exp(*t, want_cross=True, want_hash=True)
    return {k: x.cpu().numpy() for k, x in out.items() if x is not None}


@pytest.mark.parametrize("kind", ["tetrahedron", "icosphere2", "torus256", "torus258", "hole", "mobius", "batch"])
def test_update_equals_new_handle(torch, kind):
    from paper_2603_15780_amd import sg
    offs = {}
    if kind == "batch":
        parts = [_mesh("tetrahedron"), _mesh("torus258"), _mesh("icosphere2")]
        X, F = np.concatenate([p[0] for p in parts]), np.concatenate([p[1] for p in parts])
        offs = dict(vert_offsets=np.cumsum([0] + [p[0].shape[0] for p in parts]),
                    face_offsets=np.cumsum([0] + [p[1].shape[0] for p in parts]))
        Fg = np.concatenate([p[1] + o for p, o in zip(parts, offs["vert_offsets"])]).astype(np.int32)
    else:
        X, F = _mesh(kind)
        Fg = F
    X2 = (X * (1.0 + 0.1 * np.sin(3.0 * X[:, [1, 2, 0]] + 0.5))).astype(np.float32)
    r = random_rays(X2, Fg, 2001, np.random.default_rng(8), uniform_len(0.0, 2.0), K=1)
    mesh, new = sg.Mesh(X, F, **offs), sg.Mesh(X2, F, **offs)
    before = _run(torch, mesh, r)
    # rejected positions leave the handle as it was
    for bad, what in ((np.inf, "not finite"), (None, "zero area")):
        Xb = X2.copy()
        if bad is None:
            Xb[Fg[-1, 1]] = Xb[Fg[-1, 0]]
        else:
            Xb[-1, 2] = bad
        with pytest.raises(RuntimeError, match=what):
            mesh.update_vertices(Xb)
        again = _run(torch, mesh, r)
        assert all(np.array_equal(before[k], again[k], equal_nan=k in "bpvW") for k in before)
    mesh.update_vertices(X2)
    got, ref = _run(torch, mesh, r), _run(torch, new, r)
    for k in ref:
        assert np.array_equal(got[k], ref[k], equal_nan=k in "bpvW"), k
    # the mean edge is summed in another order
    assert abs(mesh.info()["mean_edge"] - new.info()["mean_edge"]) <= 1e-13 * new.info()["mean_edge"]
