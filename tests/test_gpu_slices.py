"""The y pass over slices (two waves to a slice, rows in registers) against the
line scans: a plain recompute equals its x pass followed by pdm_distance_yz,
which always runs the scans, and so does a build too small for the sweeps, at
row counts on either side of every chunk and at row widths of every lane count.
Then the builds on the sweeps' side of the rule, at grids that reach every
variant of the sweep kernel, and batches on either side of it."""
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


# (nz, ny, nx), partitions, all where the sweeps are the faster ones: whole
# quads and lanes; padded lanes; an odd map count; rows that end inside a quad
@pytest.mark.parametrize("shape,n", [((512, 512, 512), 256), ((512, 512, 496), 256), ((512, 504, 512), 255),
                                     ((500, 509, 506), 254), ((795, 1010, 1024), 64)])
@pytest.mark.parametrize("voxels", [60, 20000])
def test_sweep_side(shape, n, voxels):
    import paper_2407_21552_amd as pdm
    g = torch.Generator(device="cuda").manual_seed(n + voxels)
    vol = torch.zeros(shape, dtype=torch.uint8, device="cuda")
    at = torch.randint(0, vol.numel(), (voxels,), generator=g, device="cuda")
    vol.view(-1)[at] = torch.randint(0, 256, (voxels,), generator=g, device="cuda").to(torch.uint8)
    bounds = np.array([(p * 256) // n for p in range(n + 1)], np.int32)
    v = pdm.Volume(vol, 256, bounds)
    v.build()
    want = torch.empty_like(v.pdms)
    pdm.pom_distance_x(v.desc, v.bmin, v.bmax, bounds, want)
    pdm.distance_yz(v.desc, want, n)
    assert torch.equal(v.pdms, want)


# large volumes (sweeps); mixed ones (slices, scans of every class of lengths,
# rows narrower than a quad, single rows and planes)
@pytest.mark.parametrize("shapes,n", [([(800, 1000, 1010), (900, 1024, 1024), (60, 700, 9), (7, 1, 640)], 64),
                                      ([(90, 70, 66), (300, 421, 130), (500, 60, 257), (1020, 40, 33),
                                        (64, 1024, 5), (1, 300, 300), (200, 1, 90), (3, 2, 1), (70, 90, 15)], 37)])
def test_batch_sides(shapes, n):
    import paper_2407_21552_amd as pdm
    items, want = [], []
    for k, s in enumerate(shapes):
        g = torch.Generator(device="cuda").manual_seed(k)
        vol = torch.zeros(s, dtype=torch.uint8, device="cuda")
        at = torch.randint(0, vol.numel(), (400,), generator=g, device="cuda")
        vol.view(-1)[at] = torch.randint(0, 256, (400,), generator=g, device="cuda").to(torch.uint8)
        bounds = np.array([(p * 256) // n for p in range(n + 1)], np.int32)
        v = pdm.Volume(vol, 256, bounds)
        pdms = torch.empty_like(v.pdms)
        v.bmin.fill_(3)
        v.bmax.fill_(3)
        pdm.build_bricks(v.desc, vol, v.bmin, v.bmax)
        pdm.pom_distance_x(v.desc, v.bmin, v.bmax, bounds, pdms)
        pdm.distance_yz(v.desc, pdms, n)
        want.append(pdms)
        v.pdms.fill_(7)
        items.append((v.desc, v.volume, v.bmin, v.bmax, v.bounds, v.pdms))
    for cfg in (None, {"single_launch": 1, "lines_mult": 3}):
        ws = torch.zeros(pdm.batch_workspace_bytes(len(items)), dtype=torch.uint8, device="cuda")
        pdm.batch_build(items, ws, cfg)
        torch.cuda.synchronize()
        for it, w in zip(items, want):
            assert torch.equal(it[5], w)
            it[5].fill_(7)


@pytest.mark.parametrize("off", [1, 2, 3])
@pytest.mark.parametrize("bx,by,bz,n", [(32, 40, 9, 3), (37, 33, 5, 3), (128, 128, 127, 256)])
def test_any_alignment(off, bx, by, bz, n):
    """Maps at any byte address, slices and sweeps; bytes around them stay."""
    import paper_2407_21552_amd as pdm
    vol = _volume(bx, by, bz, 500)
    bounds = np.array([(p * 256) // n for p in range(n + 1)], np.int32)
    v = pdm.Volume(vol, 256, bounds)
    v.build()
    G = v.dist.numel()
    buf = torch.full((n * G + 8,), 77, dtype=torch.uint8, device="cuda")
    pdm.build_partitions(v.desc, v.bmin, v.bmax, bounds, buf[off:off + n * G])
    assert torch.equal(buf[off:off + n * G], v.pdms.reshape(-1))
    assert (buf[:off] == 77).all() and (buf[off + n * G:] == 77).all()
    alpha = np.zeros(256, np.float32)
    alpha[120:] = 1.0
    v.full_recompute(alpha)
    buf.fill_(77)
    pdm.full_recompute(v.desc, vol, alpha, buf[off:off + G])
    assert torch.equal(buf[off:off + G], v.dist.reshape(-1))
    assert (buf[:off] == 77).all() and (buf[off + G:] == 77).all()
