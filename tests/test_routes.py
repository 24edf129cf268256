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
    assert {8, 16, 32, 64} <= lanes
    assert {R.lib().rows_class(g[2]) for g in swept} == {0, 1}
    assert any(R.lib().parts(g[3]) == 1 and g[2] > 1 for g in swept)
    for ragged in (False, True):  # several maps to a wave, the last wave not full
        assert any((g[1] % 4 != 0) == ragged and g[0] % (64 // R.lib().row_lanes(g[1])) != 0 for g in swept)
