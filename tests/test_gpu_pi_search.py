"""The PI map's grid search where its short cuts end, against the printed scan
of every face (or against itself in another order): bit for bit the same, since
both take the exact distances and the same tie rule.

  * more faces tying at a vertex than the candidate list holds (the apex of a
    cone of 24 faces, reached from outside its corner);
  * queries several cells away from the surface (steps of the length of v);
  * queries whose nearest face lies outside their cell's list (coarse steps, a
    rough surface), so that several rings of cells list the same faces;
  * faces so unequal in size that they would fill too many cells;
  * batches large enough to be reordered, on a mesh beyond one L2.
"""
import numpy as np
import pytest

from workloads import meshes as M
from workloads.rays import random_rays, uniform_len

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

KEYS = ("f", "b", "p", "v", "W", "status", "n_steps")


def _dev(r):
    return [torch.from_numpy(r[k]).cuda() for k in ("f", "b", "v", "W")]


def _same(a, b):
    for k in KEYS:
        x, y = a[k].cpu().numpy(), b[k].cpu().numpy()
        assert np.array_equal(x, y, equal_nan=x.dtype.kind == "f"), k


def _double_cone(sides=24):
    t = 2 * np.pi * np.arange(sides) / sides
    X = np.concatenate([np.stack([np.cos(t), np.sin(t), 0 * t], 1), [[0, 0, 0.7], [0, 0, -0.9]]])
    i, j = np.arange(sides), (np.arange(sides) + 1) % sides
    F = np.concatenate([np.stack([i, j, 0 * i + sides], 1), np.stack([j, i, 0 * i + sides + 1], 1)])
    return M.canonical(X, F)


def _rough():
    X, F = M.canonical(*M.icosphere(4))
    g = np.random.default_rng(41)
    return (X * (1.0 + 0.02 * g.standard_normal((X.shape[0], 1)))).astype(np.float32), F


def _unequal():   # 5,120 faces of a hundredth of the tetrahedron's size, and the tetrahedron
    (X, F), (Y, G) = M.icosphere(4), M.tetrahedron()
    return M.canonical(np.concatenate([0.01 * X + 2.0, Y]), np.concatenate([F, G + X.shape[0]]))


@pytest.mark.parametrize("kind,step,length", [
    ("rough", 0.02, 0.5), ("rough", 0.2, 2.0), ("unequal", 0.002, 0.05), ("unequal", 0.3, 2.0),
    ("cone", 0.05, 1.0), ("cone", 0.3, 2.0),
    ("tetrahedron", 1.0, 6.0), ("sphere", 1.0, 3.0),
    ("sphere", 0.1, 2.0), ("torus", 0.25, 1.5)])
def test_search_equals_scan(kind, step, length):
    from paper_2603_15780_amd import sg
    g = np.random.default_rng(17)
    X, F = {"cone": _double_cone, "tetrahedron": lambda: M.canonical(*M.tetrahedron()),
            "sphere": lambda: M.canonical(*M.icosphere(3)),
            "rough": _rough, "unequal": _unequal,
            "torus": lambda: M.canonical(*M.torus_grid(30, 10, 0.2, g))}[kind]()
    r = random_rays(X, F, 2049, g, uniform_len(0.0, length), K=1)
    if kind == "cone":   # toward the apex of the start face, so that the steps pass it
        x = X.astype(np.float64)
        p = np.einsum("nk,nkc->nc", r["b"].astype(np.float64), x[F[r["f"]]])
        d = x[F[r["f"], 2]] - p
        r["v"] = (d / np.linalg.norm(d, axis=1, keepdims=True) * r["length"][:, None]).astype(np.float32)
    mesh, t = sg.Mesh(X, F), _dev(r)
    _same(mesh.pi_exp(*t, step=step, want_steps=True),
          mesh.pi_exp(*t, step=step, want_steps=True, search=sg.PI_SCAN))


@pytest.mark.parametrize("n", [32768, 40001, 65536, 70001])
def test_ordered_batch_equals_slices(n):
    """81,920 faces: a batch from 65,536 rays on is reordered, its slices are not; the
    backward's stacked launches are (3 n rows), and their gradients do not change."""
    from paper_2603_15780_amd import sg
    X, F = M.canonical(*M.icosphere(6))
    r = random_rays(X, F, n, np.random.default_rng(3), uniform_len(0.0, 0.5), K=1)
    r["f"][::997] = -1   # (no face: the order's last bucket)
    mesh, t = sg.Mesh(X, F), _dev(r)
    got = mesh.pi_exp(*t, step=0.05, want_steps=True)
    parts = [mesh.pi_exp(*[x[i:i + 9000].contiguous() for x in t], step=0.05, want_steps=True) for i in range(0, n, 9000)]
    _same(got, {k: torch.cat([q[k] for q in parts]) for k in KEYS})
    f, b, v, _ = t
    g = torch.from_numpy(np.random.default_rng(4).normal(size=(n, 3)).astype(np.float32)).cuda()
    all_ = mesh.pi_backward(sg.BWD_GFD, f, b, v, g, step=0.05)
    cut = [mesh.pi_backward(sg.BWD_GFD, *[x[i:i + 9000].contiguous() for x in (f, b, v, g)], step=0.05)
           for i in range(0, n, 9000)]
    for k in range(2):
        x, y = all_[k].cpu().numpy(), torch.cat([c[k] for c in cut]).cpu().numpy()
        assert np.array_equal(x, y, equal_nan=True)
