"""What the library's host code launches, and what it makes of failures, on a
stand-in HIP runtime (no GPU)."""
import ctypes as C
import os
import shutil

import numpy as np
import pytest

import fake_hip
from paper_2603_15780_amd import build as B
from paper_2603_15780_amd import sg
from workloads import meshes as M


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not os.path.exists(B.HIPCC) or not shutil.which("g++"):
        pytest.skip("hipcc or g++ not available")
    return fake_hip.Lib(fake_hip.build(str(tmp_path_factory.mktemp("host"))))


def _int(args, k):
    return C.cast(args[k], C.POINTER(C.c_int32)).contents.value


def _canonical(kind):
    return M.canonical(*(M.mobius_strip(40, 6) if kind == "mobius" else M.icosphere(3)))


# the refill threshold's place among the arguments, and the rays a wave holds
REFILL = {"k_walk": (6, 64), "k_walk2": (6, 128), "k_walk_bwd": (6, 64), "k_walk_gx": (6, 64),
          "k_adjoint_walk": (6, 64), "k_walk_round": (8, 64)}


@pytest.mark.parametrize("kind", ["icosphere", "mobius"])
@pytest.mark.parametrize("refill", [0, 1, 64, 65, 96, 128])
def test_refill_threshold_is_reached(lib, kind, refill):
    """A wave refills, and leaves its loop, once this many of its rays have ended:
    a threshold beyond the rays it holds would never be."""
    X, F = _canonical(kind)
    h, seen = lib.mesh(X, F), set()

    def launch(name, dev, args):
        if name in REFILL:
            seen.add((name, _int(args, REFILL[name][0])))

    gx, n, kw = fake_hip.arr(len(X), 3, dtype=np.float64), 1000, dict(rays_per_lane=2, refill_min=refill)
    with lib.on_launch(launch):
        for kernel in (sg.KERNEL_PERSISTENT, sg.KERNEL_PARTITIONED):
            assert lib.exp(h, n, kernel=kernel, **kw) == 0
            for mode in (sg.BWD_EP, sg.BWD_GFD):
                for saved in (True, False):
                    if saved or mode == sg.BWD_GFD or kind == "mobius":
                        assert lib.backward(h, mode, n, saved=saved, kernel=kernel, **kw) == 0
                assert lib.backward(h, mode, n, grad_X=gx, kernel=kernel, **kw) == 0
        assert lib.backward(h, sg.BWD_EP, n, grad_X=gx, gradx_records=-1, **kw) == 0
    assert {name for name, _ in seen} == set(REFILL) - {"k_walk"}
    assert all(1 <= at <= REFILL[name][1] for name, at in seen), seen


@pytest.fixture(scope="module")
def big(lib):   # (81,920 faces: large batches of the projection map take their rays in order)
    return lib.mesh(*M.canonical(*M.icosphere(6)))


ERROR = 719   # hipErrorLaunchFailure


@pytest.mark.parametrize("call", [
    "exp_plain", "exp", "exp_partitioned", "ep_gradx", "ep_gradx_unsorted", "ep_gradx_walked", "gfd", "gfd_walked", "gfd_gradx",
    "pi_exp", "pi_scan", "pi_ordered", "pi_backward", "pi_backward_ordered"])
def test_a_failed_launch_is_reported(lib, big, call):
    """Whichever launch of a call fails, the call returns the error, and the next one does not."""
    gx = fake_hip.arr(40962, 3, dtype=np.float64)
    run = {
        "exp_plain": lambda: lib.exp(big, 100, kernel=sg.KERNEL_PLAIN),
        "exp": lambda: lib.exp(big, 1000, kernel=sg.KERNEL_PERSISTENT),
        "exp_partitioned": lambda: lib.exp(big, 1000, kernel=sg.KERNEL_PARTITIONED),
        "ep_gradx": lambda: lib.backward(big, sg.BWD_EP, 1000, grad_X=gx),
        "ep_gradx_unsorted": lambda: lib.backward(big, sg.BWD_EP, 1000, grad_X=gx, gradx_records=-1),
        "ep_gradx_walked": lambda: lib.backward(big, sg.BWD_EP, 1000, grad_X=gx, boundary_mode=1),
        "gfd": lambda: lib.backward(big, sg.BWD_GFD, 1000),
        "gfd_walked": lambda: lib.backward(big, sg.BWD_GFD, 1000, saved=False),
        "gfd_gradx": lambda: lib.backward(big, sg.BWD_GFD, 1000, grad_X=gx),
        "pi_exp": lambda: lib.pi_exp(big, 1000),
        "pi_scan": lambda: lib.pi_exp(big, 1000, search=sg.PI_SCAN),
        "pi_ordered": lambda: lib.pi_exp(big, 70000),
        "pi_backward": lambda: lib.pi_backward(big, 1000),
        "pi_backward_ordered": lambda: lib.pi_backward(big, 30000),
    }[call]
    launched = []
    with lib.on_launch(lambda name, dev, args: launched.append(name)):
        assert run() == 0   # (the projection's first call builds its grid)
        launched.clear()
        assert run() == 0
    total, kept = len(launched), []
    for j in range(total):
        count = iter(range(10 ** 6))
        with lib.on_launch(lambda name, dev, args: ERROR if next(count) == j else 0):
            rc = run()
        if rc != sg.SG_E_HIP:
            kept.append((j, launched[j], rc))
        assert run() == 0
    assert total >= 1 and not kept, kept


def test_a_failed_grid_build_is_reported_and_tried_again(lib):
    h = lib.mesh(*_canonical("icosphere"))
    launched = []
    with lib.on_launch(lambda name, dev, args: launched.append(name)):
        assert lib.pi_exp(lib.mesh(*_canonical("icosphere")), 100) == 0
    for j in range(len(launched)):
        count = iter(range(10 ** 6))
        with lib.on_launch(lambda name, dev, args: ERROR if next(count) == j else 0):
            assert lib.pi_exp(h, 100) == sg.SG_E_HIP, launched[j]
    assert lib.pi_exp(h, 100) == 0


def test_a_mesh_is_updated_on_its_own_device(lib):
    """New positions and the projection grid are made on the mesh's device whichever is
    current, and the current one stays."""
    X, F = _canonical("icosphere")
    h, seen = lib.mesh(X, F), []
    lib.L.fake_set_device(1)
    try:
        with lib.on_launch(lambda name, dev, args: seen.append((name, dev))):
            assert lib.L.sg_mesh_update_vertices(h, fake_hip.ptr(X), len(X)) == 0
            assert lib.pi_exp(h, 100) == 0
        assert lib.L.fake_device() == 1
    finally:
        lib.L.fake_set_device(0)
    where = dict(seen)
    assert where.pop("k_pi_exp_grid") == 1   # (the call's own kernel: the caller's stream)
    assert {"k_pos_check", "k_pos_faces", "k_pos_vertices", "k_pi_faces", "k_pi_fill"} <= set(where)
    assert set(where.values()) == {0}, where


@pytest.fixture(scope="module")
def wide(lib):   # 350,284 faces: 257 bins of records, the smallest mesh of the larger kernel
    return lib.mesh(*M.canonical(*M.torus_grid(419, 418, 0.2, np.random.default_rng(1))))


@pytest.mark.parametrize("records", [1, 4, 32, 256])
@pytest.mark.parametrize("n", [100, 5000, 20011, 300000])
def test_record_budget_bounds_the_workspace(lib, wide, n, records):
    """gradx_records says how much memory the vertex gradient's records take: 48 bytes
    each, and for the partly filled chunks as much again or 192 KB for each of the
    default 768 blocks, whichever is more; with two words per 384-byte chunk and the
    block counts."""
    def need(records):
        out, o = C.c_size_t(), sg.opts(gradx_records=records)
        assert lib.L.sg_backward_workspace_size(wide, sg.BWD_EP, n, 0, 1, C.byref(o), C.byref(out)) == 0
        return out.value

    budget = 48 * n * records
    assert need(records) - need(-1) <= (1 + 8 / 384) * (budget + max(budget, 768 * 196608)) + (4 << 20)


def _extents(name, dev, args):
    """1,280 faces of edge 0.02 in a box of 1, for k_pi_extents."""
    if name == "k_pi_extents":
        out = C.cast(args[2], C.POINTER(C.POINTER(C.c_double))).contents
        for part in range(16):
            for k, x in enumerate((0.0, 0.0, 0.0, 1.0, 1.0, 1.0, 3 * 1280 * 0.02 / 16, 1.0)):
                out[8 * part + k] = x


@pytest.mark.parametrize("limit,rc", [(1 << 20, 0), (400 << 10, 0), (100 << 10, sg.SG_E_OOM)])
def test_projection_grid_without_memory_for_fine_cells(lib, limit, rc):
    """1,280 faces of edge 0.02 in a box of 1: 128 cells a face (up to 655 KB) in fine
    cells, 32 (164 KB) in wide ones, which a handle whose fine cells do not fit takes."""
    h = lib.mesh(*_canonical("icosphere"))
    with lib.on_launch(_extents):
        lib.L.fake_malloc_limit(limit)
        try:
            assert lib.pi_exp(h, 100) == rc
        finally:
            lib.L.fake_malloc_limit(2 ** 63)
        assert lib.pi_exp(h, 100) == 0


@pytest.mark.parametrize("call", ["exp", "gfd", "gradx", "pi_exp", "pi_backward", "update", "create"])
def test_a_failed_allocation_is_reported_once(lib, call):
    """The next call, with memory, does not find the error of the one before."""
    X, F = _canonical("icosphere")
    h, gx = lib.mesh(X, F), fake_hip.arr(len(X), 3, dtype=np.float64)
    run = {"exp": lambda: lib.exp(h, 100, kernel=sg.KERNEL_PERSISTENT), "gfd": lambda: lib.backward(h, sg.BWD_GFD, 100),
           "gradx": lambda: lib.backward(h, sg.BWD_EP, 100, grad_X=gx), "pi_exp": lambda: lib.pi_exp(h, 100),
           "pi_backward": lambda: lib.pi_backward(h, 100),
           "update": lambda: lib.L.sg_mesh_update_vertices(h, fake_hip.ptr(X), len(X)),
           "create": lambda: lib.L.sg_mesh_create(fake_hip.ptr(X), len(X), fake_hip.ptr(F), len(F), None, None, 1,
                                                  C.byref(C.c_void_p()))}[call]
    lib.L.fake_malloc_limit(0)
    try:
        assert run() == sg.SG_E_OOM
    finally:
        lib.L.fake_malloc_limit(2 ** 63)
    assert lib.exp(h, 100, kernel=sg.KERNEL_PLAIN) == 0
    assert run() == 0


@pytest.mark.parametrize("kind,open_mesh", [("closed", False), ("one hole", False), ("holes", True), ("mobius", True)])
def test_schedule_of_meshes_with_boundaries(lib, kind, open_mesh):
    """Where many rays end at a boundary the walks take one direction class and refill
    at 32 idle lanes: neither a class's rays nor a query's walks end together there."""
    X, F = _canonical("mobius" if kind == "mobius" else "icosphere")
    if kind in ("one hole", "holes"):
        X, F = M.canonical(*M.remove_faces(*M.icosphere(3), [5] if kind == "one hole" else [0, 97, 194, 291, 388, 485]))
    h, seen = lib.mesh(X, F), {}

    def launch(name, dev, args):
        if name == "k_walk_bwd":
            seen["refill"] = _int(args, 6)
        if name == "k_walk":   # QueueRanges: the buckets of a range follow its pointer
            seen["stride"] = C.cast(args[2], C.POINTER(C.c_int32))[2]

    with lib.on_launch(launch):
        assert lib.exp(h, 800000, kernel=sg.KERNEL_PERSISTENT) == 0   # (four rays per lane and more)
        assert lib.backward(h, sg.BWD_GFD, 1000) == 0   # (a batch that fits the walk's lanes: whole waves)
        assert seen["refill"] in (63, 64)
        assert lib.backward(h, sg.BWD_GFD, 300000) == 0
        got = dict(seen)
        assert lib.backward(h, sg.BWD_GFD, 1000, refill_min=17) == 0
    assert seen["refill"] == 17
    assert got == dict(refill=32 if open_mesh else 63, stride=1024 if open_mesh else 1008)


@pytest.mark.parametrize("kind,wait", [("closed", 16), ("one hole", 16), ("holes", 48), ("sheet", 48)])
def test_wait_of_an_odd_step(lib, kind, wait):
    """With hole avoidance a lane waits for others that meet a boundary: a third as long
    where few do.  (The word behind the mesh's twin pointer; 0 where rays stop.)"""
    holes = {"one hole": [5], "holes": [0, 97, 194, 291, 388, 485]}.get(kind)
    X, F = M.canonical(*(M.remove_faces(*M.icosphere(3), holes) if holes else
                         M.mobius_strip(500, 400) if kind == "sheet" else M.icosphere(3)))   # (1,000 of 400,000)
    h, seen = lib.mesh(X, F), []
    with lib.on_launch(lambda name, dev, args: name in ("k_exp_plain", "k_walk") and
                       seen.append(C.cast(args[0] + 112, C.POINTER(C.c_int32))[0]) or 0):
        for kernel in (sg.KERNEL_PLAIN, sg.KERNEL_PERSISTENT):
            for mode in (sg.BOUNDARY_STOP, sg.BOUNDARY_AVOID):
                assert lib.exp(h, 100, kernel=kernel, boundary_mode=mode) == 0
    assert seen == [0, wait, 0, wait]


@pytest.mark.parametrize("first,then", [(0.01, 0.5), (0.5, 0.01)])
def test_projection_with_the_other_cells(lib, first, then):
    """Calls of short and of long steps (from 0.02 on) have grids of their own.  A call whose
    grid is not built yet takes the other's where it cannot build it: while a graph is
    recorded, and without memory."""
    h, cells = lib.mesh(*_canonical("icosphere")), []

    def launch(name, dev, args):
        _extents(name, dev, args)
        if name == "k_pi_exp_grid":   # PiMesh: the grids' address
            cells.append(C.cast(args[0], C.POINTER(C.c_uint64))[1])

    with lib.on_launch(launch):
        assert lib.pi_exp(h, 100, first) == 0
        lib.L.fake_set_capturing(1)
        try:
            assert lib.pi_exp(h, 100, then) == 0 and lib.pi_exp(h, 100, first) == 0
        finally:
            lib.L.fake_set_capturing(0)
        lib.L.fake_malloc_limit(0)
        try:
            assert lib.pi_exp(h, 100, then) == 0
        finally:
            lib.L.fake_malloc_limit(2 ** 63)
        assert len(set(cells)) == 1
        assert lib.pi_exp(h, 100, then) == 0 and lib.pi_exp(h, 100, first) == 0
    assert cells[-2] != cells[0] == cells[-1]
