"""The packed x pass (64/W rows to a wave) against the oracle: row widths on
either side of every lane count, quads cut by the row end, rows that do not
fill the last wave, and partitions that reach the largest 16-bit value (where a
lane without bricks must not count as occupied)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

WIDTHS = [1, 3, 4, 9, 15, 16, 17, 30, 61, 64, 65, 126, 129, 254, 257, 508, 513, 1021, 1024]


def _volume(nx, dtype, levels, seed):
    r = np.random.default_rng(seed)
    v = np.zeros((7, 21, nx), dtype)
    at = r.integers(0, v.size, max(2, v.size // 150))
    v.reshape(-1)[at] = r.integers(0, levels, len(at))
    return v


@pytest.mark.parametrize("nx", WIDTHS)
@pytest.mark.parametrize("dtype,levels,parts", [(np.uint8, 256, (1, 5)), (np.uint16, 65536, (1, 3)),
                                                (np.uint16, 4096, (40,))])
def test_pdms(nx, dtype, levels, parts):
    import paper_2407_21552_amd as pdm
    vol = _volume(nx, dtype, levels, nx + levels)
    for n in parts:
        bounds = np.array([(p * levels) // n for p in range(n + 1)], np.int32)
        v = pdm.Volume(pdm.to_device(vol), levels, bounds)
        v.build()
        want = oracle.pdms(vol, bounds, levels, brick_minmax=oracle.bricks(vol))
        assert np.array_equal(pdm.from_device(v.pdms), want), n


@pytest.mark.parametrize("nx", WIDTHS)
@pytest.mark.parametrize("dtype,levels,n", [(np.uint8, 256, 5), (np.uint16, 4096, 40), (np.uint8, 256, 256)])
def test_pdms_exact(nx, dtype, levels, n):
    import paper_2407_21552_amd as pdm
    vol = _volume(nx, dtype, levels, nx + n)
    bounds = np.array([(p * levels) // n for p in range(n + 1)], np.int32)
    v = pdm.Volume(pdm.to_device(vol), levels, bounds, mode=pdm.EXACT)
    v.build()
    want = oracle.pdms(vol, bounds, levels, mode=oracle.EXACT)
    assert np.array_equal(pdm.from_device(v.pdms), want)
    alpha = np.zeros(levels, np.float32)
    alpha[levels // 3: levels // 2] = 0.5
    v.full_recompute(alpha)
    assert np.array_equal(pdm.from_device(v.dist), oracle.full_recompute(vol, alpha, levels,
                                                                         mode=oracle.EXACT))
