"""Launch rules of the direct-space list kernels, on the host: a cap on the work-groups per
compute unit (mbd_shape.pair_wg_per_cu) holds for the launch as a whole, also where a
group's candidates are split into parts and the right-hand sides into slices."""
import os

import pytest

from paper_2307_02278_amd import _lib as L

pytestmark = pytest.mark.skipif(not os.path.exists(L.HOSTCHECK_PATH),
                                reason="libmbd_hostcheck.so not built")


@pytest.mark.parametrize("ngroups", [1, 7, 8, 38, 188, 513, 1500, 60000])
@pytest.mark.parametrize("parts,slices", [(1, 1), (1, 2), (6, 1), (16, 1), (5, 4)])
def test_residency_cap_counts_every_work_group(ngroups, parts, slices):
    grid = L.hostcheck().mbdh_pair_grid
    every = -(-ngroups // 8) * 8
    assert grid(ngroups, parts, slices, 0) == every
    for wg_per_cu in (1, 2, 3, 64):
        cap = 256 * wg_per_cu
        x = grid(ngroups, parts, slices, cap)
        assert x % 8 == 0 and 8 <= x <= every
        assert x * parts * slices <= max(cap, 8 * parts * slices)
        # no smaller than the cap asks for
        assert x == every or (x + 8) * parts * slices > cap
