"""The volume-reading passes at every width where their variant changes (under
16 voxels, multiples of 16, rows that end inside a quad, on either side of 400
voxels), with brick layers cut in z and y and without, against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

WIDTHS = [1, 3, 4, 15, 16, 17, 48, 63, 384, 400, 403, 496, 500, 512, 516, 1040]
TYPES = [(np.uint8, 256), (np.uint16, 4096), (np.uint16, 65536)]


@pytest.mark.parametrize("dtype,levels", TYPES)
@pytest.mark.parametrize("nx", WIDTHS)
def test_bricks_and_plain(nx, dtype, levels):
    import paper_2407_21552_amd as pdm
    r = np.random.default_rng(nx + levels)
    for nz, ny in ((8, 12), (7, 10), (5, 3), (2, 9), (6, 1)):
        # values near a border of the opacity's support, so that bricks differ
        vol = r.integers(levels // 4, levels // 2 + levels // 16, (nz, ny, nx)).astype(dtype)
        vol[r.random(vol.shape) < 0.02] = levels - 1
        bounds = np.array([0, levels // 3, levels], np.int32)
        alpha = np.zeros(levels, np.float32)
        alpha[levels // 2: levels // 2 + levels // 32] = 0.5
        v = pdm.Volume(pdm.to_device(vol), levels, bounds, voxel_dtype=dtype)
        v.build()
        bmin, bmax = oracle.bricks(vol)
        assert np.array_equal(pdm.from_device(v.bmin, dtype), bmin)
        assert np.array_equal(pdm.from_device(v.bmax, dtype), bmax)
        v.full_recompute(alpha)
        assert np.array_equal(pdm.from_device(v.dist), oracle.full_recompute(vol, alpha, levels))
        if levels > 16384:
            continue
        e = pdm.Volume(pdm.to_device(vol), levels, bounds, voxel_dtype=dtype, mode=pdm.EXACT)
        e.full_recompute(alpha)
        assert np.array_equal(pdm.from_device(e.dist),
                              oracle.full_recompute(vol, alpha, levels, mode=oracle.EXACT))


@pytest.mark.parametrize("dtype,levels,n", [(np.uint8, 256, 5), (np.uint16, 4096, 40), (np.uint16, 4096, 200)])
@pytest.mark.parametrize("nx", [3, 15, 16, 31, 624, 640, 643, 1024])
def test_exact_build(nx, dtype, levels, n):
    import paper_2407_21552_amd as pdm
    r = np.random.default_rng(nx + n)
    bounds = np.array([(p * levels) // n for p in range(n + 1)], np.int32)
    for nz, ny in ((7, 10), (18, 7), (2, 9), (18, 3)):  # cut layers, with the look-ahead's slices and thin
        vol = np.zeros((nz, ny, nx), dtype)
        at = r.integers(0, vol.size, max(2, vol.size // 100))
        vol.reshape(-1)[at] = r.integers(0, levels, len(at))
        v = pdm.Volume(pdm.to_device(vol), levels, bounds, voxel_dtype=dtype, mode=pdm.EXACT)
        v.build()
        assert np.array_equal(pdm.from_device(v.pdms), oracle.pdms(vol, bounds, levels, mode=oracle.EXACT))
