"""CPU model of the raster sweeps' schedule (pdm_sweep.hip): waves that run two
blocks of rows behind one another through rings of rows, two parts in z, rows
past the plane's end, and the padding of the last block, against the
definition.  Every ring entry carries the plane and row it holds, so a row read
before it is written, or after it is overwritten, fails here."""
import random

import numpy as np
import pytest

LAG = 2
CAP = 255


def x_distance(occ):
    d = np.where(occ, 0, CAP)
    r = d.copy()
    for s in range(1, d.shape[2]):
        f = np.maximum(d, s)
        r[:, :, s:] = np.minimum(r[:, :, s:], f[:, :, :-s])
        r[:, :, :-s] = np.minimum(r[:, :, :-s], f[:, :, s:])
    return np.minimum(r, CAP)


def distance(occ):
    """The definition, one axis after the other."""
    d = np.where(occ, 0, CAP)
    for ax in range(3):
        r = np.full_like(d, CAP)
        m = d.shape[ax]
        for s in range(m):
            f = np.maximum(d, s)
            lo, hi = [slice(None)] * 3, [slice(None)] * 3
            lo[ax], hi[ax] = slice(0, m - s), slice(s, None)
            lo, hi = tuple(lo), tuple(hi)
            r[hi] = np.minimum(r[hi], f[lo])
            r[lo] = np.minimum(r[lo], f[hi])
        d = np.minimum(r, CAP)
    return d


def spread(m):
    """1 + the minimum over x-1, x, x+1 (outside the row: above every distance)."""
    p = np.concatenate([[511], m[:-1]])
    n = np.concatenate([m[1:], [511]])
    return np.minimum(np.minimum(p, m), n) + 1


def sweeps(maps, NW, parts, RB, rng):
    bz, by, bx = maps.shape
    A = maps.copy()
    split = (bz + 1) // 2 if parts == 2 else bz
    nblk = (by + RB - 1) // RB
    period = max(nblk, LAG * NW)
    cap = np.full(bx, CAP)
    for ph in (0, 1):
        order = list(range(parts))
        rng.shuffle(order)  # the parts of one launch run in any order
        for part in order:
            up = (ph == 0) == (part == 0)
            ahead = 1 if ph == 1 and parts == 2 else 0
            z_lo, z_hi = (0, split) if part == 0 else (split, bz)
            planes = z_hi - z_lo + ahead
            zs = 1 if up else -1
            z0 = (z_lo if up else z_hi - 1) - zs * ahead
            y0, ys = (0, 1) if ph == 0 else (by - 1, -1)
            steps = ((planes + NW - 1) // NW - 1) * period + nblk + LAG * (NW - 1)
            size = [LAG] * NW
            size[NW - 1] = period - LAG * NW + LAG
            ring = [[None] * (size[w] * RB) for w in range(NW)]
            h = A.copy()
            st = [dict(k=w, b=-LAG * w, X=cap, Pm=cap, pw=[((-1, None), cap)] * RB) for w in range(NW)]
            for t in range(steps + 3):  # the kernel runs a multiple of four steps
                for w in rng.sample(range(NW), NW):  # the waves of a step run in any order
                    q = st[w]
                    k, b = q["k"], q["b"]
                    src, size_r = ring[(w - 1) % NW], size[(w - 1) % NW]
                    act = 0 <= b < nblk and k < planes
                    after = src[((t + 1) % size_r) * RB]
                    if b + 1 >= nblk or k == 0:
                        after = q["pw"][RB - 1]
                    if act and k > 0:
                        want = [b * RB + r for r in range(RB)] + [min((b + 1) * RB, nblk * RB - 1)]
                        for entry, j in zip(q["pw"] + [after], want):
                            assert entry is not None and entry[0] == (k - 1, j)
                    if b == 0:
                        q["X"] = q["Pm"] = cap
                    P0 = q["pw"][0][1] if q["pw"][0] else None
                    for r in range(RB):
                        at = (t % size[w]) * RB + r
                        if not act:
                            ring[w][at] = (("none", t), np.zeros(bx, int))
                            continue
                        j = b * RB + r
                        P1 = (q["pw"][r + 1] if r + 1 < RB else after)[1]
                        m = np.minimum(np.minimum(q["Pm"], P0), P1)
                        # rows past the last one take the last one's values
                        S = np.minimum(np.minimum(h[z0 + zs * k, y0 + ys * min(j, by - 1)], q["X"]), m)
                        q["X"] = spread(S)
                        q["Pm"], P0 = P0, P1
                        ring[w][at] = ((k, j), q["X"])
                        if j < by and k >= ahead:
                            A[z0 + zs * k, y0 + ys * j] = S
                    q["b"] += 1
                    if q["b"] == period:
                        q["b"] = 0
                        q["k"] += NW
                    # read at the end of the step, for the next one
                    if q["k"] > 0:
                        q["pw"] = [src[((t + 1) % size_r) * RB + r] for r in range(RB)]
    return A


@pytest.mark.parametrize("RB", [4, 8])
@pytest.mark.parametrize("NW", [1, 2, 3, 5, 8])
def test_sweeps_are_exact(NW, RB):
    rng = random.Random(100 * NW + RB)
    g = np.random.default_rng(100 * NW + RB)
    for _ in range(12):
        shape = tuple(int(x) for x in g.integers(1, 30, 3))
        occ = g.random(shape) < g.choice([0.0, 0.002, 0.02, 0.2])
        want = distance(occ)
        for parts in (1, 2) if shape[0] > 1 else (1,):
            got = sweeps(x_distance(occ), NW, parts, RB, rng)
            assert np.array_equal(got, want), (shape, parts)


def test_other_part_before_or_after_its_second_sweep():
    """The second sweep of a part may read any mixture of the other part's
    rows before and after that part's own second sweep."""
    rng = random.Random(1)
    g = np.random.default_rng(1)
    for _ in range(40):
        shape = tuple(int(x) for x in g.integers(2, 14, 3))
        occ = g.random(shape) < 0.02
        want = distance(occ)
        # the first sweep of both parts, by raster order
        h, split = x_distance(occ), (shape[0] + 1) // 2
        A = h.copy()
        for zs in (list(range(split)), list(range(shape[0] - 1, split - 1, -1))):
            prev = None
            for z in zs:
                for y in range(shape[1]):
                    m = A[z, y]
                    if y > 0:
                        m = np.minimum(m, spread(A[z, y - 1]))
                    if prev is not None:
                        for yy in range(max(0, y - 1), min(shape[1], y + 2)):
                            m = np.minimum(m, spread(A[prev, yy]))
                    A[z, y] = m
                prev = z
        # the second sweep of the lower part from a mixture of A and the final map
        mix = np.where(g.random(shape) < rng.random(), A, want)
        low, prev = A.copy(), mix[split].copy()
        for z in range(split - 1, -1, -1):
            for y in range(shape[1] - 1, -1, -1):
                m = low[z, y]
                if y + 1 < shape[1]:
                    m = np.minimum(m, spread(low[z, y + 1]))
                for yy in range(max(0, y - 1), min(shape[1], y + 2)):
                    m = np.minimum(m, spread(prev[yy]))
                low[z, y] = m
            prev = low[z].copy()
        assert np.array_equal(low[:split], want[:split])
