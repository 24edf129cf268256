"""The cases that the GPU tests mean for the sweeps are on the sweeps' side of
the rules, and reach every variant of the kernels."""
import pytest

import route_rules as R

# (n, Bx, By, Bz), measured microseconds of the y and z passes by the sweeps and
# by slices and z scans, where these differ by more than a fifth
TALL = [((64, 64, 64, 3000), 3895, 2113), ((32, 64, 64, 8000), 10691, 2866), ((64, 128, 128, 300), 583, 887),
        ((64, 128, 128, 600), 1143, 1848), ((64, 256, 256, 257), 1147, 2904), ((32, 256, 256, 400), 1514, 2454),
        ((64, 256, 64, 500), 694, 1510), ((16, 256, 64, 2000), 2654, 1362), ((128, 100, 100, 700), 1417, 2698),
        ((12, 256, 256, 300), 1073, 621), ((128, 16, 16, 4000), 3266, 555), ((255, 4, 4, 8000), 5801, 961)]

# the same for rows of several maps to a wave, by more than a twelfth
NARROW = [((255, 24, 128, 600), 2616, 1528), ((255, 31, 127, 300), 1259, 1022), ((255, 60, 128, 200), 786, 609),
          ((255, 60, 160, 200), 945, 743), ((255, 64, 256, 256), 1646, 1479), ((255, 64, 128, 256), 898, 776),
          ((255, 61, 127, 255), 979, 806), ((255, 64, 200, 128), 631, 462), ((128, 100, 256, 256), 1342, 1228),
          ((255, 128, 256, 128), 856, 1080), ((255, 100, 128, 300), 956, 2913), ((255, 101, 129, 301), 1034, 3100),
          ((256, 128, 128, 128), 424, 571), ((128, 130, 96, 256), 548, 595)]


@pytest.mark.parametrize("grid,sweeps,lines", NARROW)
def test_narrow_rows_take_the_faster(grid, sweeps, lines):
    assert R.sweep_fits(*grid) == (sweeps < lines)


@pytest.mark.parametrize("grid,sweeps,lines", TALL)
def test_tall_grids_take_the_faster(grid, sweeps, lines):
    assert R.sweep_fits(*grid) == (sweeps < lines)



# batches, (nx, ny, nz) voxels and how many with n partitions; measured
# microseconds of the build with all volumes of at least 4 bricks a row swept and
# with none, where these differ by more than a twentieth
BATCHES = [([((56, 1000, 1000), 24)], 64, 5250, 4001), ([((64, 1000, 1000), 24)], 64, 4645, 4252),
           ([((80, 1000, 1000), 24)], 64, 5924, 5607), ([((124, 1000, 1000), 24)], 64, 7655, 8155),
           ([((128, 1000, 1000), 24)], 64, 6120, 7184), ([((64, 500, 500), 48)], 64, 2721, 1758),
           ([((96, 500, 500), 48)], 64, 3006, 2534), ([((128, 500, 500), 48)], 64, 3126, 2851),
           ([((64, 1000, 300), 48)], 64, 2968, 2018), ([((96, 1000, 300), 48)], 64, 3453, 2993),
           ([((128, 1000, 300), 48)], 64, 3355, 3176), ([((64, 1024, 1024), 24)], 64, 2976, 3908),
           ([((64, 640, 640), 48)], 64, 2521, 2680), ([((64, 1024, 1024), 48)], 64, 5842, 7821),
           ([((128, 640, 640), 48)], 64, 3858, 4563), ([((128, 1024, 1024), 20)], 64, 5557, 5825),
           ([((128, 512, 1024), 24)], 64, 2741, 3518), ([((128, 1024, 1024), 48)], 32, 6658, 7690),
           ([((32, 1024, 1024), 24)], 64, 4465, 2280), ([((16, 1000, 1000), 24)], 64, 7646, 1492),
           ([((48, 1000, 1000), 24)], 64, 4673, 3540), ([((68, 500, 500), 48)], 64, 2610, 2055),
           ([((160, 1000, 1000), 24)], 64, 7596, 10150), ([((250, 640, 640), 24)], 64, 4534, 5076),
           ([((132, 1000, 1000), 24)], 64, 7139, 8786), ([((300, 1024, 1024), 6)], 64, 4187, 4729),
           ([((1024, 1024, 795), 1), ((12, 1000, 1000), 20)], 64, 2577, 3059),
           ([((1024, 64, 1024), 24)], 64, 2918, 3498), ([((1024, 1024, 795), 2)], 64, 2054, 3227)]
MIXED = [([((1024, 1024, 795), 2), ((32, 1000, 1000), 20)], 64), ([((1024, 1024, 795), 2), ((20, 1000, 1000), 12)], 64),
         ([((1024, 1024, 795), 2), ((16, 1000, 1000), 4), ((30, 700, 900), 4), ((24, 1024, 1024), 4)], 64),
         ([((1024, 1024, 795), 2), ((36, 1000, 1000), 16)], 64)]


def _grids(sizes, n):
    return [R.bricks(s[::-1], n) for s, count in sizes for _ in range(count)]


@pytest.mark.parametrize("sizes,n,sweeps,lines", BATCHES)
def test_batches_take_the_faster(sizes, n, sweeps, lines):
    assert R.batch_fits(_grids(sizes, n)) == (sweeps < lines)


@pytest.mark.parametrize("sizes,n", MIXED)
def test_narrow_volumes_of_a_swept_batch_keep_the_scans(sizes, n):
    grids = _grids(sizes, n)
    assert R.batch_fits(grids)
    assert [R.volume_sweeps(g) for g in grids] == [g[1] > 32 for g in grids]


# (n, Bx, By, Bz), measured microseconds of the y pass by slices and by line
# scans, where these differ by more than a twentieth
Y_PASS = [((64, 8, 16, 4000), 46.6, 30.3), ((64, 8, 64, 1953), 61.6, 57.7), ((64, 4, 16, 4000), 33.0, 26.3),
          ((64, 12, 64, 1302), 65.1, 48.9), ((64, 12, 32, 2604), 64.0, 48.9), ((64, 8, 32, 3906), 61.1, 51.7),
          ((64, 33, 2, 4000), 103.8, 81.5), ((64, 33, 16, 1893), 61.0, 54.6), ((64, 17, 4, 4000), 58.0, 51.3),
          ((64, 4, 17, 4000), 28.6, 47.5), ((64, 5, 64, 3125), 103.6, 134.2), ((64, 8, 100, 1250), 58.2, 65.7),
          ((64, 16, 16, 3906), 35.5, 52.0), ((64, 17, 32, 1838), 42.2, 60.9), ((64, 33, 17, 1782), 58.0, 82.2),
          ((64, 48, 4, 4000), 109.7, 129.7), ((64, 64, 2, 4000), 102.2, 139.0), ((64, 128, 128, 61), 23.6, 57.4),
          ((64, 100, 8, 1250), 74.8, 93.0), ((64, 8, 64, 244), 10.5, 16.5), ((64, 4, 32, 976), 15.4, 20.6),
          ((128, 4, 256, 1907), 362.6, 341.4), ((128, 8, 256, 953), 233.1, 251.4), ((128, 12, 192, 847), 242.9, 228.4),
          ((1, 128, 128, 64), 7.2, 10.0), ((1, 33, 8, 64), 3.0, 4.6),
          ((1, 100, 2, 64), 4.3, 3.6), ((3, 33, 2, 60), 4.2, 3.4), ((1, 17, 3, 64), 4.2, 3.9), ((1, 8, 2, 64), 3.2, 3.4),
          ((6, 256, 2, 200), 5.6, 7.2)]


@pytest.mark.parametrize("grid,slices,scans", Y_PASS)
def test_y_pass_takes_the_faster(grid, slices, scans):
    assert R.slice_y_wins(*grid) == (slices < scans)


def test_single_cases_take_the_sweeps():
    seen = set()
    for shape, n in R.SWEEP_CASES:
        g = R.bricks(shape, n)
        assert R.sweep_fits(*g), (shape, n)
        W = R.lib().row_lanes(g[1])
        ragged, pad = g[1] % 4 != 0, 4 * W != g[1] or n % (64 // W) != 0
        seen.add((W, ragged, pad, g[2] % 4 == 0))
    assert {w for w, _, _, _ in seen} == {16, 32, 64}
    # ragged; whole blocks of rows with and without padding; padded lanes over other row counts
    assert any(r for _, r, _, _ in seen) and any((not r) and (not p) and e for _, r, p, e in seen)
    assert any((not r) and p and e for _, r, p, e in seen) and any((not r) and not e for _, r, _, e in seen)


def test_batch_takes_the_sweeps():
    grids = [R.bricks(s, n) for s, n in R.SWEEP_BATCH]
    assert R.batch_fits(grids)
    swept = [g for g in grids if R.volume_sweeps(g)]
    lanes = {R.lib().row_lanes(g[1]) for g in swept}
    assert {4, 8, 16, 32, 64} <= lanes
    assert any(g[1] >= 4 and not R.volume_sweeps(g) for g in grids)
    assert {R.lib().rows_class(g[2]) for g in swept} == {0, 1}
    assert any(R.lib().parts(g[3]) == 1 and g[2] > 1 for g in swept)
    for ragged in (False, True):  # several maps to a wave, the last wave not full
        assert any((g[1] % 4 != 0) == ragged and g[0] % (64 // R.lib().row_lanes(g[1])) != 0 for g in swept)
