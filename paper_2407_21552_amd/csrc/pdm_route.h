// pdm_route.h -- which kernels take the y and z passes of a build or recompute,
// and the launch shapes that the choice is made on.  Host code without HIP, so
// that it can be compiled and tested on its own.
#pragma once
#include <stdint.h>

#include <algorithm>

namespace pdm {

constexpr int kRowLanes = 64;  // a wave
// Rows per step of a wave (between two barriers).  8 measured within 3% for
// 256-row planes and 7% slower for 96 (fewer blocks than the lag of 16 waves
// needs).
constexpr int kSweepRows = 4;
constexpr int kSweepWaves = 16;       // most waves of a work-group
constexpr int kSweepBatchWaves = 8;   // waves of a batch's work-groups
constexpr int kSweepMinPlanes = 16;   // fewer planes are not cut in two parts in a batch

// The maps of one volume: n grids of Bx x By x Bz bricks.
struct RouteGrid {
    int n, Bx, By, Bz;
};

// Lanes per row, 4 bricks each: the power of two with 4W >= Bx.
inline int row_lanes(int Bx) {
    int W = 1;
    while (4 * W < Bx) W *= 2;
    return W;
}

// Whether k_slice_y can take the y pass of these grids: whole quads of bricks in
// a wave, rows in registers.
inline bool slice_y_fits(int Bx, int By) { return Bx >= 4 && Bx <= 256 && By >= 2 && By <= 256; }

// Scans over at most this many lines run two lanes per line or stage them in
// LDS: they cannot fill the chip's 1024 SIMDs with more than a few waves each,
// so per-wave latency matters more than occupancy.
constexpr int64_t kStagedMaxLines = 1 << 18;

// Whether it takes the y pass of `count` maps, and not the line scans.  It is
// the faster one for few lines (one map of 256x256x199 13 us against 24), but
// for those of 2 or 3 bricks, which are a launch either way (one map of
// 100x2x64 4.3 us against 3.6, 33x2x200 4.0 and 3.4; 8x2x64 3.2 and 3.4), and on
// most grids (64 MB of maps: 128x128 planes 24 us against 57, 33x32 36 against
// 51).  Not, with many lines, on
//  - planes of at most 16 rows that leave two fifths of a row's lanes without a
//    brick: the waves work on 32 rows and 4W bricks whatever the plane has
//    (33x4 112 us against 93, 17x2 55 against 44, 132x8 1.13 times; but 48x4
//    110 against 130, 200x16 0.75 times, 33x20 0.67 times);
//  - planes of whole 64-byte blocks with rows of 4, 8 or 12 bricks: 16 to 64
//    slices to a wave, each of its accesses in a cache line of its own at one
//    alignment (8x16 47 us against 30, 12x64 65 against 49, 4x16 33 against 26;
//    but 8x20 0.76 times, 5x16 31 against 32, 16x16 36 against 52); the scans'
//    tables grow with the line, so 8 and 12 bricks up to 192 rows (250 MB:
//    12x192 243 against 228, 8x256 233 against 251, 4x256 363 against 341).
inline bool slice_y_wins(int count, int Bx, int By, int Bz) {
    if (!slice_y_fits(Bx, By)) return false;
    const int64_t lines = (int64_t)count * Bx * Bz;
    if (lines <= kStagedMaxLines) return Bx <= 16 || By > 3 || lines > kStagedMaxLines / 2;
    const int W = row_lanes(Bx);
    if (W >= 8 && By <= 16 && 5 * Bx <= 12 * W) return false;
    return !(Bx % 4 == 0 && Bx <= 12 && (Bx * By) % 64 == 0 && (Bx == 4 || By <= 192));
}

// Steps of one sweep over np planes of By rows with NW waves.
inline int64_t sweep_steps(int np, int By, int NW) {
    const int nblk = (By + kSweepRows - 1) / kSweepRows;
    const int period = std::max(nblk, 2 * NW);
    return (int64_t)((np + NW - 1) / NW - 1) * period + nblk + 2 * (NW - 1);
}

// Waves of a work-group: the fewest steps.
inline int sweep_waves(int np, int By) {
    int best = 1;
    for (int nw = 2; nw <= kSweepWaves; ++nw)
        if (sweep_steps(np, By, nw) < sweep_steps(np, By, best)) best = nw;
    return best;
}

// Microseconds the line scans take per megabyte of maps, one pass over lines
// of m bricks (fits of measured passes: 0.67 at 96 bricks, 0.74 at 128, 0.91
// at 199, 1.04 at 256: the longer the line, the larger its table and the fewer
// the waves of a compute unit).  Over 256 bricks another kernel takes the pass
// (k_dist_global), whose tables do not grow with the line: 2.1 to 2.6 measured
// from 257 to 8000 bricks.
inline double scan_us_per_mb(int m) { return m > 256 ? 2.3 : 0.45 + 0.0023 * m; }

// Microseconds per step of a sweep over `groups` work-groups: 0.8 of issue, and
// more the more work-groups' rows are in flight, above all where a wave's rows
// are those of several maps, each in cache lines of its own.  Measured: W 64:
// 0.80 (24 work-groups), 0.88 (64), 0.95 (128, no more at 256 and 510); W 32:
// 0.83 (64), 1.11 (128), 1.15 to 1.36 (256); W 16: 1.15 (64), 1.1 to 1.56 (128).
inline double sweep_step_us(int W, int64_t groups) {
    if (W >= 64) return 0.8 + 0.0012 * (double)std::min<int64_t>(groups, 128);
    return 0.8 + (W == 32 ? 0.0022 : 0.0055) * (double)std::min<int64_t>(groups, 256);
}

// Whether the sweeps take all maps of a grid, and not the slices (0.36 us per
// megabyte) and the z scans.  They run one work-group per group of 64/W maps
// and half of the planes, each a chain of steps, so they win where there are
// many bytes for few steps: 64 maps of 256x256x199 bricks 901 us against 1217,
// 256 maps of 128x128x128 424 against 571; but 64 maps of 256x256x128 607
// against 598, of 175x175x175 593 against 485, 256 of 75x75x75 185 against 130.
// Tall grids: 64 maps of 128x128x600 1143 against 1848, of 64x64x3000 3895
// against 2113, 32 of 128x128x1200 2000 against 1691.  Narrow rows: 255 maps of
// 60x128x200 786 against 609, 128 of 100x256x256 1342 against 1228; with 8 maps
// to a wave (32 bricks and fewer) no size measured wins: 255 of 32x128x300 947
// against 959, of 24x128x600 2616 against 1528.
inline bool sweep_fits(int count, int Bx, int By, int Bz) {
    if (Bx <= 32 || Bx > 256 || By > 256 || Bz < 2) return false;
    const int W = row_lanes(Bx), per = kRowLanes / W;
    const int64_t G = (int64_t)Bx * By * Bz;
    if (G * std::min(per, count) > INT32_MAX) return false;  // 32-bit offsets within a group
    const int np = (Bz + 1) / 2 + 1, nw = sweep_waves(np, By);
    const int64_t groups = 2 * (int64_t)((count + per - 1) / per);
    const double rounds = std::max(1.0, (double)groups / 256.0);
    const double t_sweep = 2.0 * (sweep_step_us(W, groups) * (double)sweep_steps(np, By, nw) * rounds + 8.0);
    const double mb = 1e-6 * (double)G * count;
    return t_sweep < mb * (0.36 + scan_us_per_mb(Bz));
}

inline int batch_sweep_parts(int Bz) { return Bz >= kSweepMinPlanes ? 2 : 1; }

// Launch a volume's sweeps are in: planes of more than 104 rows (0) apart from
// the others (1).  A launch's rings are sized for its highest plane, 2 KB per 4
// rows: up to 104 rows (52 KB) three work-groups share a compute unit's LDS.
inline int batch_sweep_class(int By) { return By > 104 ? 0 : 1; }

// Microseconds of slices and z scans for a volume of a batch, and of a brick row
// of its sweeps (64/W maps at once).  The rows of a wave's maps lie in cache
// lines of their own, so narrow rows cost more, and rows of at most 16 bricks
// twice as much again where planes are no whole cache lines and neighbouring
// waves share them.  Per thousand rows, from batches of one size by both
// routes: 0.17 to 0.28 (W 4, whole lines), 0.36 to 0.6 (W 4, others), 0.2 to
// 0.37 (W 8), about 2 (W 2) and 4.5 (W 1); 0.2 for the wider ones.
inline double batch_lines_us(const RouteGrid& g) {
    return 1e-6 * (double)g.Bx * g.By * g.Bz * g.n * (0.46 + 1.3 * scan_us_per_mb(g.Bz));
}
inline double batch_sweep_row_us(const RouteGrid& g) {
    const int W = row_lanes(g.Bx);
    if (W >= 16) return 0.2e-3;
    if (W == 8) return 0.33e-3;
    if (W == 4) return (g.Bx * g.By) % 128 == 0 ? 0.23e-3 : 0.45e-3;
    return W == 2 ? 2e-3 : 4.5e-3;
}
inline double batch_sweep_rows(const RouteGrid& g) {
    const int per = kRowLanes / row_lanes(g.Bx);
    return (double)((g.n + per - 1) / per) * g.By * g.Bz;
}

// Whether a volume's y and z passes are sweeps in a batch that takes them: rows
// of at most 32 bricks only where their sweeps cost less than their slices and
// scans (2 volumes of 1024x1024x795 voxels with 12 of 20x1000x1000: 8715 us
// with all swept, 4532 with none).
inline bool batch_volume_sweeps(const RouteGrid& g) {
    if (g.Bx < 4) return false;
    return g.Bx > 32 || batch_sweep_row_us(g) * batch_sweep_rows(g) < batch_lines_us(g);
}

// Whether the sweeps take the y and z phases of a batch's volumes, as far as
// batch_volume_sweeps lets them, and not the slices and the z scans: their time
// follows all rows and the longest chain of steps, that of the others the bytes
// (fits of the measured batches, sweeps against slices and scans: 4 volumes of
// 900..1024 voxels per axis 2645 us against 3780, 12 of 400..1000 2340 against
// 3230; 48 of 96..640 1833 against 1780, 6 of 300..640 571 against 319, 48 of
// 60..200 194 against 92; whole builds of 24 of 64x1000x1000 4645 against 4252,
// of 80x1000x1000 5923 against 5607, of 128x1000x1000 6120 against 7184).
inline bool batch_sweep_fits(const RouteGrid* g, int count) {
    double rows = 0.0, t_lines = 0.0;
    int64_t chain = 0;
    for (int k = 0; k < count; ++k) {
        if (!batch_volume_sweeps(g[k])) continue;
        const int parts = batch_sweep_parts(g[k].Bz);
        rows += batch_sweep_row_us(g[k]) * batch_sweep_rows(g[k]);
        chain = std::max(chain, sweep_steps((g[k].Bz + parts - 1) / parts, g[k].By, kSweepBatchWaves));
        t_lines += batch_lines_us(g[k]);
    }
    return rows + 0.8 * (double)chain + 30.0 < t_lines;
}

}  // namespace pdm
