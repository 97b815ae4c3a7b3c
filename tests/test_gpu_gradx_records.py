"""The vertex gradient's records, sorted by half-edge bin in the walk, against
the same sums by float64 atomics alone: batches around a wave and a buffer of
records, meshes on both sides of each bin count the kernels are made for, and
record budgets that run out."""
import numpy as np
import pytest

from workloads import meshes as M
from workloads.rays import random_rays, uniform_len

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _mesh(kind):
    g = np.random.default_rng(23)
    if kind == "tetrahedron":
        return M.canonical(*M.tetrahedron())
    if kind == "mobius":
        return M.canonical(*M.mobius_strip(40, 6))
    if kind == "holes":
        return M.canonical(*M.remove_faces(*M.icosphere(3), [5, 700]))
    return M.canonical(*M.torus_grid(*kind, 0.2, g))


def _gradx(mesh, r, g, **kw):
    t = [torch.from_numpy(r[k]).cuda() for k in ("f", "b", "v")] + [torch.from_numpy(g).cuda()]
    out = torch.zeros(mesh.n_verts, 3, dtype=torch.float64, device="cuda")
    mesh.backward(0, *t, grad_X=out, want_vjp=False, **kw)
    return out.cpu().numpy()


@pytest.mark.parametrize("kind,n,length,kw", [
    ("tetrahedron", 1, 500.0, {}),          # one ray, some hundred records: one buffer or two
    ("tetrahedron", 64, 3.0, {}),
    ("tetrahedron", 65, 40.0, {}),
    ((16, 4), 1000, 20.0, {}),              # 384 half-edges: three bins of 128, all full
    ((43, 127), 4099, 4.0, {}),             # 32,766: 256 bins of 128
    ((43, 128), 4099, 4.0, {}),             # 33,024: bins of 256
    ((418, 418), 20011, 2.0, {}),           # 1,048,344: 256 bins of 4096
    ((419, 418), 20011, 2.0, {}),           # 1,050,852: 257 bins
    ((836, 836), 20011, 1.0, {}),           # 4,193,376: 1024 bins
    ((837, 836), 20011, 1.0, {}),           # 4,198,392: 1025 bins, records as they come
    ((43, 127), 4099, 4.0, dict(gradx_records=1)),
    ((43, 127), 4099, 4.0, dict(gradx_records=20, walk_blocks=3)),
    ((419, 418), 20011, 2.0, dict(gradx_records=3)),
    ("mobius", 2049, 6.0, {}),
    ("holes", 2049, 6.0, dict(boundary_mode=1)),
])
def test_sorted_records_equal_atomics(kind, n, length, kw):
    """The terms are the same float32 numbers; the float64 sums differ by their
    order, at most 2^-53 times the terms (< 2^22) times their magnitudes' sum."""
    from paper_2603_15780_amd import sg
    X, F = _mesh(kind)
    rng = np.random.default_rng(29)
    r = random_rays(X, F, n, rng, uniform_len(0.2 * length, length), K=0)
    g = rng.standard_normal((n, 3)).astype(np.float32)
    mesh = sg.Mesh(X, F)
    atm = _gradx(mesh, r, g, **{**kw, "gradx_records": -1})
    assert np.isfinite(atm).all() and np.abs(atm).max() > 0
    got = _gradx(mesh, r, g, **kw)
    assert np.allclose(got, atm, rtol=1e-9, atol=1e-9 * np.abs(atm).max())
