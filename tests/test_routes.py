"""The cases that the GPU tests mean for the sweeps are on the sweeps' side of
the rules, and reach every variant of the kernels."""
import route_rules as R


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
