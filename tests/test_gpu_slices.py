"""The y pass over slices (two waves to a slice, rows in registers) against the
line scans: a plain recompute equals its x pass followed by pdm_distance_yz,
which always runs the scans, and so does a build too small for the sweeps, at
row counts on either side of every chunk and at row widths of every lane count."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ROWS = [2, 3, 15, 16, 31, 32, 33, 34, 64, 65, 97, 128, 129, 161, 193, 225, 254, 255, 256]
WIDTHS = [4, 5, 7, 8, 13, 16, 31, 64, 101, 128, 130, 255, 256]


def _volume(bx, by, bz, voxels):
    g = torch.Generator(device="cuda").manual_seed(bx + 1000 * by + voxels)
    v = torch.zeros((4 * bz, 4 * by, 4 * bx), dtype=torch.uint8, device="cuda")
    at = torch.randint(0, v.numel(), (voxels,), generator=g, device="cuda")
    v.view(-1)[at] = torch.randint(1, 256, (voxels,), generator=g, device="cuda").to(torch.uint8)
    return v


def _check(bx, by, bz, voxels):
    import paper_2407_21552_amd as pdm
    vol = _volume(bx, by, bz, voxels)
    bounds = np.array([0, 100, 200, 256], np.int32)
    v = pdm.Volume(vol, 256, bounds)
    v.build()
    pdms = torch.empty_like(v.pdms)
    pdm.pom_distance_x(v.desc, v.bmin, v.bmax, bounds, pdms)
    pdm.distance_yz(v.desc, pdms, 3)
    assert torch.equal(v.pdms, pdms)
    alpha = np.zeros(256, np.float32)
    alpha[120:] = 1.0
    dist = torch.empty_like(v.dist)
    pdm.plain_distance_x(v.desc, vol, alpha, dist)
    pdm.distance_yz(v.desc, dist, 1)
    v.full_recompute(alpha)
    assert torch.equal(v.dist, dist)


@pytest.mark.parametrize("by", ROWS)
@pytest.mark.parametrize("voxels", [0, 5, 3000])
def test_row_counts(by, voxels):
    _check(37, by, 5, voxels)
    _check(32, by, 8, voxels)


@pytest.mark.parametrize("bx", WIDTHS)
@pytest.mark.parametrize("voxels", [1, 2000])
def test_row_widths(bx, voxels):
    for by in (30, 131):
        _check(bx, by, 17, voxels)
