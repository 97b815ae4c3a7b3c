"""Record budgets too small for a chunk per wave and bin: fewer walk blocks, and streams without a chunk."""
import numpy as np
import pytest

from test_gpu_gradx_records import _gradx, _mesh
from workloads.rays import random_rays, uniform_len

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,kw", [(20011, {}), (20011, dict(gradx_records=1)), (5000, dict(gradx_records=8)),
                                  (20011, dict(gradx_records=1, walk_blocks=700))])
def test_small_budgets_equal_atomics(n, kw):
    """1,397,792 faces: 1,024 bins.  The float64 sums differ by their order, as with any other budget."""
    from paper_2603_15780_amd import sg
    X, F = _mesh((836, 836))
    rng = np.random.default_rng(31)
    r = random_rays(X, F, n, rng, uniform_len(0.2, 1.0), K=0)
    g = rng.standard_normal((n, 3)).astype(np.float32)
    mesh = sg.Mesh(X, F)
    atm = _gradx(mesh, r, g, **{**kw, "gradx_records": -1})
    got = _gradx(mesh, r, g, **kw)
    assert np.abs(atm).max() > 0 and np.allclose(got, atm, rtol=1e-9, atol=1e-9 * np.abs(atm).max())
