"""LDS of the vertex gradient's and the projection's kernels (CPU only): it decides how
many of their blocks a compute unit holds, which their block counts are measured for."""
import re

from test_build_resources import remarks  # noqa: F401  (the fixture compiles the kernels)

CU_LDS = 160 << 10

# kernel, its template arguments: bytes per block, blocks that have to fit a compute unit
LDS = {
    ("k_adjoint_walk", "Li256E"): (52240, 3),
    ("k_adjoint_walk", "Li1024E"): (79888, 2),
    ("k_gs_group", ""): (4096, 8),
    ("k_gs_reduce", "Li1024ELi512E"): (40960, 4),
    ("k_gs_reduce", "Li4096ELi1024E"): (163840, 1),
    ("k_pi_exp_grid", ""): (8192, 2),
}


def test_lds_per_block(remarks):  # noqa: F811
    seen = set()
    for name, (_, lds) in remarks.items():
        m = re.match(r"_ZN2sg12_GLOBAL__N_1\d+(k_[a-z0-9_]+?)(I|E)", name)
        for (kernel, args), (size, blocks) in LDS.items():
            if m and m.group(1) == kernel and args in name:
                seen.add((kernel, args))
                assert lds == size and blocks * lds <= CU_LDS, (name, lds)
    assert seen == set(LDS), set(LDS) - seen
