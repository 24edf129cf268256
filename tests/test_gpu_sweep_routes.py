"""The raster sweeps where the rules choose them (asserted), at every number of
maps to a wave, against the x pass followed by pdm_distance_yz, which always
runs the line scans."""
import numpy as np
import pytest

import route_rules as R

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _sparse(shape, seed, voxels):
    g = torch.Generator(device="cuda").manual_seed(seed)
    vol = torch.zeros(shape, dtype=torch.uint8, device="cuda")
    at = torch.randint(0, vol.numel(), (voxels,), generator=g, device="cuda")
    vol.view(-1)[at] = torch.randint(0, 256, (voxels,), generator=g, device="cuda").to(torch.uint8)
    return vol


def _scans(v):
    want = torch.empty_like(v.pdms)
    import paper_2407_21552_amd as pdm
    pdm.pom_distance_x(v.desc, v.bmin, v.bmax, v.bounds, want)
    pdm.distance_yz(v.desc, want, v.n)
    return want


def _resident(shape, n, seed, voxels):
    import paper_2407_21552_amd as pdm
    return pdm.Volume(_sparse(shape, seed, voxels), 256, np.array([(p * 256) // n for p in range(n + 1)], np.int32))


@pytest.mark.parametrize("shape,n", R.SWEEP_CASES)
@pytest.mark.parametrize("voxels", [40, 20000])
def test_build(shape, n, voxels):
    assert R.sweep_fits(*R.bricks(shape, n))
    v = _resident(shape, n, n + voxels, voxels)
    v.build()
    assert torch.equal(v.pdms, _scans(v))


def test_batch():
    import paper_2407_21552_amd as pdm
    assert R.batch_fits([R.bricks(s, n) for s, n in R.SWEEP_BATCH])
    vols = [_resident(s, n, k, 400) for k, (s, n) in enumerate(R.SWEEP_BATCH)]
    for v in vols:
        v.pdms.fill_(7)
    ws = torch.zeros(pdm.batch_workspace_bytes(len(vols)), dtype=torch.uint8, device="cuda")
    pdm.batch_build([(v.desc, v.volume, v.bmin, v.bmax, v.bounds, v.pdms) for v in vols], ws)
    for v in vols:
        assert torch.equal(v.pdms, _scans(v)), v.volume.shape
