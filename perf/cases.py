"""The workloads this library is timed on: its public calls, as a program that
renders or serves volumes makes them.

A case is a dict of plain values.  Fields:

    kind     which call one pass makes:
               build             Volume.build (brick [min,max] and every PDM)
               update            Volume.update_tf (D' of a new opacity table)
               recompute         Volume.full_recompute (plain method, D)
               recompute_cached  Volume.full_recompute_cached
               table             Volume.build_range_table
               update_ranges     Volume.update_tf_ranges
               batch_build       batch_build over `count` volumes
               batch_update      batch_tf_update_prepared over `count` volumes
    nx ny nz, levels, n, mode ("range" or "exact")
    content  what the volume holds: "ellipsoids" (a few solids on a zero
             background, with noise), "tubes" (a sparse tree of capsules, almost
             all voxels near 0) or "ct" (air, tissue cylinder, bones, 5% salt)
    tf       the opacity ramps' supports as fractions of the level range,
             "a-d,a-d": opacity is non-zero strictly between a and d
    count, dims_lo, dims_hi, spec
             batches only: volumes, range of their axes, seed of their sizes

Voxels, opacities and their heights are drawn from the seed on the GPU.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2407_21552_amd as pdm

# supports of the opacity ramps used by the listed cases
TF_TWO = "0.12-0.24,0.55-0.70"             # two ramps
TF_THREE = "0.03-0.13,0.31-0.42,0.80-0.95"  # three ramps


def listed():
    return [
        # The smallest calls (a 64^3 u8 volume, 8 partitions): an interactive
        # preview, where launches and host time are what a user waits for.
        dict(name="update_64", kind="update", nx=64, ny=64, nz=64, levels=256, n=8, mode="range",
             content="ellipsoids", tf=TF_TWO),
        dict(name="recompute_64", kind="recompute", nx=64, ny=64, nz=64, levels=256, n=8, mode="range",
             content="ellipsoids", tf=TF_TWO),
        dict(name="build_64", kind="build", nx=64, ny=64, nz=64, levels=256, n=8, mode="range",
             content="ellipsoids", tf=TF_TWO),
        # A TF change on a large resident volume (1024x1024x795 u8 tube tree,
        # 64 partitions) by the partitioned update, the library's main call.
        dict(name="update_1024", kind="update", nx=1024, ny=1024, nz=795, levels=256, n=64, mode="range",
             content="tubes", tf=TF_THREE),
        # The same TF change by the plain method: from the voxels, and from the
        # brick ranges kept since the volume was loaded.
        dict(name="recompute_1024", kind="recompute", nx=1024, ny=1024, nz=795, levels=256, n=64,
             mode="range", content="tubes", tf=TF_THREE),
        dict(name="recompute_cached_1024", kind="recompute_cached", nx=1024, ny=1024, nz=795, levels=256,
             n=64, mode="range", content="tubes", tf=TF_THREE),
        # Loading that volume: brick ranges and all 64 PDMs.
        dict(name="build_1024", kind="build", nx=1024, ny=1024, nz=795, levels=256, n=64, mode="range",
             content="tubes", tf=TF_THREE),
        # Loading a 12-bit CT scan (512x512x460 u16, 32 partitions).
        dict(name="build_ct", kind="build", nx=512, ny=512, nz=460, levels=4096, n=32, mode="range",
             content="ct", tf=TF_TWO),
        # A scan cropped to odd sizes: rows that are no multiple of anything,
        # bricks cut on all three far faces; the per-voxel (EXACT) reading of
        # the build, and the plain method from the cached ranges.
        dict(name="build_exact_crop", kind="build", nx=509, ny=487, nz=451, levels=4096, n=32,
             mode="exact", content="ct", tf=TF_TWO),
        dict(name="recompute_cached_crop", kind="recompute_cached", nx=509, ny=487, nz=451, levels=4096,
             n=32, mode="range", content="ct", tf=TF_TWO),
        # A server that loads a catalogue: 48 volumes of mixed sizes (96..640
        # per axis, mostly odd), u8 and 12-bit u16, 16 to 64 partitions, built
        # together, and the TF updates of all of them in one call.
        dict(name="batch_build_48", kind="batch_build", count=48, dims_lo=96, dims_hi=640, spec=4,
             tf=TF_TWO),
        dict(name="batch_update_48", kind="batch_update", count=48, dims_lo=96, dims_hi=640, spec=4,
             tf=TF_TWO),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    tf = []
    for _ in range(rng.randint(1, 4)):
        w = rng.uniform(1 / 32, 1 / 4)
        a = rng.uniform(0, 1 - w)
        tf.append("%.3f-%.3f" % (a, a + w))
    tf = ",".join(tf)
    kind = rng.choice(["build", "build", "update", "recompute", "recompute_cached", "table",
                       "update_ranges", "batch_build", "batch_update"])
    if kind.startswith("batch"):
        lo = _log_int(rng, 24, 200)
        return dict(kind=kind, count=rng.randint(2, 40), dims_lo=lo, dims_hi=min(640, lo + _log_int(rng, 8, 400)),
                    spec=rng.randint(1, 10**6), tf=tf)
    mode = "exact" if kind in ("build", "recompute") and rng.random() < 0.3 else "range"
    content = rng.choice(["ellipsoids", "tubes", "ct"])
    levels = rng.choice([256, 256, rng.randint(40, 256)])
    if content == "ct":
        levels = 4096 if mode == "exact" else rng.choice([4096, 4096, 65536])
    while True:
        nx, ny, nz = (_log_int(rng, 24, 1024) for _ in range(3))
        n = _log_int(rng, 1, 256)
        n = max(min(n, levels), 2 if kind == "table" else 1)
        if rng.random() < 0.3:
            nx = max(16, nx // 16 * 16)  # whole quads: many scans are padded to this
        case = dict(kind=kind, nx=nx, ny=ny, nz=nz, levels=levels, n=n, mode=mode, content=content, tf=tf)
        maps = n + (_table_maps(n, 8) if kind in ("table", "update_ranges") else 0)
        if _voxels(case) <= 300_000_000 and maps * _grid(case)[3] <= 600_000_000:
            return case


# ---------------------------------------------------------------- geometry
def _voxels(c):
    return c["nx"] * c["ny"] * c["nz"]


def _grid(c):
    b = [(c[k] + 3) // 4 for k in ("nz", "ny", "nx")]
    return b[0], b[1], b[2], b[0] * b[1] * b[2]


def _bytes(c):
    return 1 if c["levels"] <= 256 else 2


def _bounds(c):
    return np.array([(p * c["levels"]) // c["n"] for p in range(c["n"] + 1)], np.int32)


def _table_maps(n, max_level):
    maps, k = 0, 1
    while k <= max_level and (1 << k) <= n:
        maps += n - (1 << k) + 1
        k += 1
    return maps


def _batch(c):
    """The volumes of a batch case, as single-volume cases."""
    r = random.Random(c["spec"])
    out = []
    for k in range(c["count"]):
        nx, ny, nz = (r.randint(c["dims_lo"], c["dims_hi"]) for _ in range(3))
        u8 = k < c["count"] // 2
        out.append(dict(nx=nx, ny=ny, nz=nz, levels=256 if u8 else 4096, n=r.choice([16, 32, 64]),
                        mode="range", content="ellipsoids" if u8 else "ct", tf=c["tf"]))
    return out


def _support(c):
    """Levels of non-zero opacity."""
    on = np.zeros(c["levels"], bool)
    for part in c["tf"].split(","):
        a, d = (float(x) * c["levels"] for x in part.split("-"))
        i = np.arange(c["levels"])
        on |= (i > a) & (i < d)
    return on


def _active(c):
    on, b = _support(c), _bounds(c)
    return [p for p in range(c["n"]) if on[b[p]:b[p + 1]].any()]


def _alpha(c, seed):
    rng = np.random.default_rng(seed)
    a = np.zeros(c["levels"], np.float32)
    on = _support(c)
    a[on] = rng.uniform(0.05, 1.0, int(on.sum())).astype(np.float32)
    return a


# ------------------------------------------------------------------ inputs
def _solid(vol, gen_np, kind, scale):
    """Writes one solid of a random value into vol (float32, [z][y][x])."""
    shape = vol.shape
    dev = vol.device
    if kind == "ellipsoid":
        p0 = p1 = [gen_np.uniform(0, s) for s in shape]
        semi = [gen_np.uniform(4, 20) * scale for _ in range(3)]
        pad = semi
    else:
        p0 = [gen_np.uniform(0, s) for s in shape]
        d = gen_np.normal(size=3)
        d *= gen_np.uniform(80, 400) * scale / np.linalg.norm(d)
        p1 = [min(max(p0[k] + d[k], 0.0), shape[k] - 1.0) for k in range(3)]
        r = max(1.0, gen_np.uniform(2, 12) * scale)
        pad = [r] * 3
    lo = [max(0, int(min(p0[k], p1[k]) - pad[k])) for k in range(3)]
    hi = [min(shape[k], int(max(p0[k], p1[k]) + pad[k]) + 2) for k in range(3)]
    if any(l >= h for l, h in zip(lo, hi)):
        return
    ax = [torch.arange(l, h, device=dev, dtype=torch.float32).view([-1 if j == k else 1 for j in range(3)])
          for k, (l, h) in enumerate(zip(lo, hi))]
    sub = vol[lo[0]:hi[0], lo[1]:hi[1], lo[2]:hi[2]]
    value = float(gen_np.integers(60, 241))
    if kind == "ellipsoid":
        inside = sum(((ax[k] - p0[k]) / semi[k]) ** 2 for k in range(3)) <= 1.0
    else:
        v = [p1[k] - p0[k] for k in range(3)]
        t = sum((ax[k] - p0[k]) * v[k] for k in range(3)) / max(1e-6, sum(x * x for x in v))
        t = t.clamp(0.0, 1.0)
        inside = sum((ax[k] - p0[k] - t * v[k]) ** 2 for k in range(3)) <= r * r
    sub.masked_fill_(inside, value)


def _volume(c, seed):
    """The voxels on the GPU: uint8, or int16 holding the bits of uint16."""
    shape = (c["nz"], c["ny"], c["nx"])
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    gnp = np.random.default_rng(seed)
    out = torch.empty(shape, dtype=torch.uint8 if _bytes(c) == 1 else torch.int16, device=dev)
    top = c["levels"] - 1
    base = torch.zeros(shape, dtype=torch.float16, device=dev)
    scale = min(shape) / 64.0 if c["content"] == "ellipsoids" else min(1.0, min(shape) / 512.0)
    if c["content"] == "ellipsoids":
        for _ in range(6):
            _solid(base, gnp, "ellipsoid", scale)
    elif c["content"] == "tubes":
        for _ in range(40):
            _solid(base, gnp, "tube", scale)
    else:
        for _ in range(20):
            _solid(base, gnp, "ellipsoid", 2.0 * scale)
    step = max(1, (1 << 26) // (shape[1] * shape[2]))
    y = torch.arange(shape[1], device=dev, dtype=torch.float32)[:, None] - (shape[1] - 1) / 2
    x = torch.arange(shape[2], device=dev, dtype=torch.float32)[None, :] - (shape[2] - 1) / 2
    disk = y * y + x * x <= (0.45 * min(shape[1:])) ** 2
    for z0 in range(0, shape[0], step):
        b = base[z0:z0 + step].float()
        noise = torch.randn(b.shape, generator=gen, device=dev)
        if c["content"] == "ct":  # 12-bit values, spread over the level range
            u = top / 4095.0
            v = torch.where(disk, 1000.0 + 40.0 * noise, (8.0 * noise).abs())
            v = torch.where(b > 0, 1500.0 + 6.0 * b, v) * u
            v = torch.where(torch.rand(b.shape, generator=gen, device=dev) < 0.05, float(top), v)
        else:
            v = (b + (2.0 if c["content"] == "tubes" else 3.0) * noise) * (top / 255.0)
        v = v.round().clamp(0, top).to(torch.int32)
        out[z0:z0 + step] = v.to(out.dtype)
    if c["content"] != "ct":  # hot detector pixels: 200 voxels of any value
        at = torch.from_numpy(gnp.integers(0, out.numel(), 200)).to(dev)
        out.view(-1)[at] = torch.from_numpy(gnp.integers(0, top + 1, 200)).to(dev).to(out.dtype)
    return out


def _resident(c, seed):
    v = pdm.Volume(_volume(c, seed), c["levels"], _bounds(c), mode=c["mode"])
    return v


class _Arena:
    """One device buffer cut into pieces that start at multiples of 512 bytes,
    as a server lays its outputs out."""

    def __init__(self, sizes):
        self.first, total = [], 0
        for s in sizes:
            self.first.append(total)
            total += (s + 511) // 512 * 512
        self.buf = torch.zeros(max(total, 512), dtype=torch.uint8, device="cuda")
        self.sizes = sizes

    def piece(self, k):
        return self.buf[self.first[k]:self.first[k] + self.sizes[k]]

    def fill(self, parts):
        for k, t in enumerate(parts):
            self.piece(k).copy_(t.contiguous().view(-1).view(torch.uint8))
        return self.buf


def _arenas(case):
    """Brick minima and maxima, PDMs and outputs of a batch."""
    cs = _batch(case)
    ranges = [_grid(c)[3] * _bytes(c) for c in cs]
    return (_Arena(ranges), _Arena(ranges), _Arena([c["n"] * _grid(c)[3] for c in cs]),
            _Arena([_grid(c)[3] for c in cs]))


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("batch_build", "batch_update"):
        cs = _batch(case)
        mn, mx, maps, dist = _arenas(case)
        items = []
        for k, c in enumerate(cs):
            vol = _volume(c, seed * 1000 + k)
            desc = pdm.volume_desc(vol.shape, np.uint8 if _bytes(c) == 1 else np.uint16, c["levels"])
            items.append((desc, vol, mn.piece(k), mx.piece(k), _bounds(c), maps.piece(k)))
        ws = torch.zeros(pdm.batch_workspace_bytes(len(items)), dtype=torch.uint8, device="cuda")
        st = dict(kind=kind, items=items, ws=ws, bmin=mn.buf, bmax=mx.buf, pdms=maps.buf, dist=dist.buf)
        if kind == "batch_update":
            pdm.batch_build(items, ws)
            st["entries"] = [(pdm.PreparedVolume(it[0], it[5], it[4]), _alpha(c, seed * 1000 + k), dist.piece(k))
                             for k, (c, it) in enumerate(zip(cs, items))]
        return st
    v = _resident(case, seed)
    st = dict(kind=kind, vol=v, alpha=_alpha(case, seed))
    if kind in ("update", "update_ranges", "table", "recompute_cached"):
        v.build()
    if kind == "update_ranges":
        v.build_range_table()
    return st


def run(state):
    kind = state["kind"]
    if kind == "batch_build":
        pdm.batch_build(state["items"], state["ws"])
        return dict(bmin=state["bmin"], bmax=state["bmax"], pdms=state["pdms"])
    if kind == "batch_update":
        masks = pdm.batch_tf_update_prepared(state["entries"])
        return dict(mask=masks.view(np.int64), dist=state["dist"])
    v = state["vol"]
    if kind == "build":
        v.build()
        return dict(bmin=v.bmin, bmax=v.bmax, pdms=v.pdms)
    if kind == "update":
        mask = v.update_tf(state["alpha"])
        return dict(mask=mask.view(np.int64), dist=v.dist)
    if kind == "update_ranges":
        mask = v.update_tf_ranges(state["alpha"])
        return dict(mask=mask.view(np.int64), dist=v.dist)
    if kind == "table":
        v.build_range_table()
        return dict(table=v.table)
    if kind == "recompute":
        v.full_recompute(state["alpha"])
    else:
        v.full_recompute_cached(state["alpha"])
    return dict(dist=v.dist)


def _cover(case):
    """Maps read through the range table: one or two per run of active partitions."""
    act, maps, k = _active(case), 0, 0
    while k < len(act):
        j = k
        while j + 1 < len(act) and act[j + 1] == act[j] + 1:
            j += 1
        length = j - k + 1
        maps += 1 if length & (length - 1) == 0 else 2
        k = j + 1
    return maps


def work(case):
    kind = case["kind"]
    if kind in ("batch_build", "batch_update"):
        one = kind.split("_")[1]
        return dict(bytes=sum(work(dict(c, kind=one))["bytes"] for c in _batch(case)), flops=0)
    V, G, s, n = _voxels(case), _grid(case)[3], _bytes(case), case["n"]
    b = {
        "build": V * s + 2 * G * s + n * G,
        "update": (len(_active(case)) + 1) * G,
        "update_ranges": (_cover(case) + 1) * G,
        "table": (n + _table_maps(n, 8)) * G,
        "recompute": V * s + G,
        "recompute_cached": 2 * G * s + G,
    }[kind]
    return dict(bytes=b, flops=0)


# ------------------------------------------------- the same by plain tensors
def _levels_of(t):
    return t.to(torch.int32) & 0xFFFF


def _brick_minmax(c, vol):
    bz, by, bx, _ = _grid(c)
    mn = torch.empty((bz, by, bx), dtype=torch.int32, device=vol.device)
    mx = torch.empty_like(mn)
    for z in range(bz):
        v = _levels_of(vol[4 * z:4 * z + 4])
        pad = (0, 4 * bx - c["nx"], 0, 4 * by - c["ny"])
        lo = torch.nn.functional.pad(v.amin(0), pad, value=1 << 20).view(by, 4, bx, 4)
        hi = torch.nn.functional.pad(v.amax(0), pad, value=-1).view(by, 4, bx, 4)
        mn[z], mx[z] = lo.amin((1, 3)), hi.amax((1, 3))
    return mn, mx


def _any_in_brick(c, hit):
    """hit(z0, z1) -> bool voxels; True where some voxel of the brick is."""
    bz, by, bx, _ = _grid(c)
    out = []
    for z in range(bz):
        v = hit(4 * z, 4 * z + 4).any(0)
        v = torch.nn.functional.pad(v, (0, 4 * bx - c["nx"], 0, 4 * by - c["ny"]))
        out.append(v.view(by, 4, bx, 4).any(3).any(1))
    return torch.stack(out)


def _distance(occ):
    """Chessboard distance to the nearest True, clamped at 255 (uint8)."""
    d = torch.where(occ, 0, 255).to(torch.uint8)
    for ax in (2, 1, 0):
        m = d.shape[ax]
        r = d.clone()
        for s in range(1, min(256, m)):
            if s % 8 == 1 and s >= int(r.max()):
                break
            f = d.clamp(min=s)
            a, b = r.narrow(ax, s, m - s), r.narrow(ax, 0, m - s)
            torch.minimum(a, f.narrow(ax, 0, m - s), out=a)
            torch.minimum(b, f.narrow(ax, s, m - s), out=b)
        d = r
    return d


def _occupied(c, vol, mn, mx, lo, hi):
    if c["mode"] == "exact":
        return _any_in_brick(c, lambda a, b: (_levels_of(vol[a:b]) >= lo) & (_levels_of(vol[a:b]) <= hi))
    return (mn <= hi) & (mx >= lo)


def _exact_one(c, vol, alpha):
    kind = c["kind"]
    mn, mx = _brick_minmax(c, vol)
    if kind in ("recompute", "recompute_cached"):
        on = torch.from_numpy(alpha != 0).to(vol.device)
        if c["mode"] == "exact":
            occ = _any_in_brick(c, lambda a, b: on[_levels_of(vol[a:b]).long()])
        else:
            pre = torch.cat([torch.zeros(1, dtype=torch.int64, device=vol.device), on.long().cumsum(0)])
            occ = pre[mx.long() + 1] > pre[mn.long()]
        return dict(dist=_distance(occ))
    b = _bounds(c)
    t = torch.uint8 if _bytes(c) == 1 else torch.int16

    def one(p):
        return _distance(_occupied(c, vol, mn, mx, int(b[p]), int(b[p + 1]) - 1))

    if kind == "build":
        pdms = torch.stack([one(p) for p in range(c["n"])])
        return dict(bmin=mn.to(t), bmax=mx.to(t), pdms=pdms)
    if kind == "table":
        level, out, k = torch.stack([one(p) for p in range(c["n"])]), [], 1
        while k <= 8 and (1 << k) <= c["n"]:
            h = 1 << (k - 1)
            level = torch.minimum(level[:-h], level[h:])
            out.append(level)
            k += 1
        return dict(table=torch.cat(out) if out else None)
    dist = torch.full(mn.shape, 255, dtype=torch.uint8, device=vol.device)
    mask = np.zeros(4, np.uint64)
    for p in range(c["n"]):
        if (alpha[b[p]:b[p + 1]] != 0).any():
            mask[p >> 6] |= np.uint64(1 << (p & 63))
            dist = torch.minimum(dist, one(p))
    return dict(mask=mask.view(np.int64), dist=dist)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("batch_build", "batch_update"):
        outs = []
        for k, c in enumerate(_batch(case)):
            c = dict(c, kind=kind.split("_")[1])
            outs.append(_exact_one(c, _volume(c, seed * 1000 + k), _alpha(c, seed * 1000 + k)))
        mn, mx, maps, dist = _arenas(case)
        if kind == "batch_build":
            return dict(bmin=mn.fill([o["bmin"] for o in outs]), bmax=mx.fill([o["bmax"] for o in outs]),
                        pdms=maps.fill([o["pdms"] for o in outs]))
        return dict(mask=np.stack([o["mask"] for o in outs]), dist=dist.fill([o["dist"] for o in outs]))
    return _exact_one(case, _volume(case, seed), _alpha(case, seed))
