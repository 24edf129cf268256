"""Builds that take the raster sweeps against the line scans: the PDMs of
pdm_build_partitions* equal those of the x pass followed by pdm_distance_yz,
which always runs the scans, at row widths, row counts and map counts that
reach every variant of the sweep kernel."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _volume(shape, levels, dtype, seed, voxels):
    g = torch.Generator(device="cuda").manual_seed(seed)
    v = torch.zeros(shape, dtype=dtype, device="cuda")
    at = torch.randint(0, v.numel(), (voxels,), generator=g, device="cuda")
    v.view(-1)[at] = torch.randint(0, levels, (voxels,), generator=g, device="cuda").to(dtype)
    return v


# (nz, ny, nx), partitions: whole quads and lanes; padded lanes; rows that end
# inside a quad; rows and maps that are no multiple of anything, 2 and 4 maps
# to a wave
CASES = [((512, 1024, 1024), 64), ((384, 384, 400), 256), ((384, 384, 404), 256),
         ((500, 1013, 1010), 64), ((797, 811, 199), 255)]


@pytest.mark.parametrize("shape,n", CASES)
@pytest.mark.parametrize("voxels", [60, 20000])
def test_build_equals_scans(shape, n, voxels):
    import paper_2407_21552_amd as pdm
    vol = _volume(shape, 256, torch.uint8, 1 + n + voxels, voxels)
    bounds = np.array([(p * 256) // n for p in range(n + 1)], np.int32)
    v = pdm.Volume(vol, 256, bounds)
    v.build()
    want = torch.empty_like(v.pdms)
    pdm.pom_distance_x(v.desc, v.bmin, v.bmax, bounds, want)
    pdm.distance_yz(v.desc, want, n)
    assert torch.equal(v.pdms, want)


def test_exact_build_equals_scans():
    import paper_2407_21552_amd as pdm
    vol = _volume((500, 1013, 1010), 4096, torch.int16, 5, 5000)
    bounds = np.array([(p * 4096) // 64 for p in range(65)], np.int32)
    v = pdm.Volume(vol, 4096, bounds, mode=pdm.EXACT)
    v.build()
    want = torch.empty_like(v.pdms)
    pdm.pom_exact_distance_x(v.desc, vol, bounds, want)
    pdm.distance_yz(v.desc, want, 64)
    assert torch.equal(v.pdms, want)


def test_batch_equals_single_builds():
    """A batch large enough for the sweeps, with volumes narrower than a quad,
    flat ones and ones of few planes among them."""
    import paper_2407_21552_amd as pdm
    r = np.random.default_rng(3)
    shapes = [tuple(int(x) for x in r.integers(230, 430, 3)) for _ in range(40)]
    shapes += [(300, 300, 9), (1, 300, 300), (40, 420, 260), (300, 1, 300), (5, 7, 3)]
    items, vols = [], []
    for k, s in enumerate(shapes):
        vol = _volume(s, 256, torch.uint8, k, 300)
        n = int(r.choice([32, 64, 61]))
        bounds = np.array([(p * 256) // n for p in range(n + 1)], np.int32)
        v = pdm.Volume(vol, 256, bounds)
        v.pdms.fill_(7)
        vols.append(v)
        items.append((v.desc, v.volume, v.bmin, v.bmax, v.bounds, v.pdms))
    ws = torch.zeros(pdm.batch_workspace_bytes(len(items)), dtype=torch.uint8, device="cuda")
    pdm.batch_build(items, ws)
    for v in vols:
        want = torch.empty_like(v.pdms)
        pdm.pom_distance_x(v.desc, v.bmin, v.bmax, v.bounds, want)
        pdm.distance_yz(v.desc, want, v.n)
        assert torch.equal(v.pdms, want), v.volume.shape
