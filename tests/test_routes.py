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
