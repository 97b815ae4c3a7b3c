"""The PI map's grid search on needle faces against the printed scan of every
face: bit for bit the same.  On a face w wide and 1 long the Gram determinant is
w^2 and cancels to 2^-53 / w^2 of itself, so a search that filters by a distance
formed in another way than the scan's drops the faces the scan takes."""
import numpy as np
import pytest

from workloads import meshes as M
from workloads.rays import random_rays, uniform_len

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

KEYS = ("f", "b", "p", "v", "W", "status", "n_steps")


def _strips(angles, radius, closed):
    """Strips of length 1 along y between the lines at these angles of a circle in the xz-plane."""
    n = len(angles)
    c = radius * np.stack([np.cos(angles), 0 * angles, np.sin(angles)], 1)
    X = np.concatenate([c, c + [0.0, 1.0, 0.0]])
    i = np.arange(n if closed else n - 1)
    j = (i + 1) % n
    return M.canonical(X, np.concatenate([np.stack([i, i + n, j], 1), np.stack([j, i + n, j + n], 1)]))


def _fillet(w):   # a quarter round of 24 strips
    return _strips(np.linspace(0.0, np.pi / 2, 25), 24 * w / (np.pi / 2), False)


def _tube(w):     # a closed ring of 64 strips
    return _strips(2 * np.pi * np.arange(64) / 64, 64 * w / (2 * np.pi), True)


def _mixed(w):    # the ring beside faces that are not slim
    (X, F), (Y, G) = M.icosphere(3), _tube(w)
    return M.canonical(np.concatenate([0.3 * X + [0.35, 0.5, 0.0], Y]), np.concatenate([F, G + X.shape[0]]))


@pytest.mark.parametrize("width", [1e-3, 1e-4, 3e-5, 1e-5, 3e-6, 1e-6])
@pytest.mark.parametrize("mesh", [_fillet, _tube, _mixed])
def test_search_equals_scan_on_needles(mesh, width):
    from paper_2603_15780_amd import sg
    X, F = mesh(width)
    h, g = sg.Mesh(X, F), np.random.default_rng(11)
    # steps across the strips, and steps of the strips' length
    for step, length in ((width, 40 * width), (0.01, 1.0)):
        r = random_rays(X, F, 4096, g, uniform_len(0.0, length), K=1)
        t = [torch.from_numpy(r[k]).cuda() for k in ("f", "b", "v", "W")]
        kw = dict(step=step, want_steps=True, max_steps=200)   # (a ray that leaves the fillet never gets further)
        a = h.pi_exp(*t, **kw)
        s = h.pi_exp(*t, search=sg.PI_SCAN, **kw)
        for k in KEYS:
            x, y = a[k].cpu().numpy(), s[k].cpu().numpy()
            assert np.array_equal(x, y, equal_nan=x.dtype.kind == "f"), (k, step, int((x != y).sum()))
