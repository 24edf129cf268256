// pdm_sweep.hip -- x distances -> full chessboard distances by two raster
// sweeps over brick rows, for builds that cover many maps.
//
// What it relies on.  The input rows hold distances along x: where a value is
// 1 or more, a neighbour is one less.  For such a row h, 1 + min(h(x-1), h(x),
// h(x+1)) = max(h, 1), so a candidate that is r rows away, max(r, h(x)), is
// reached by r steps of "one more than the smallest of the three neighbours".
// Chessboard distance over rows (y, z) is then a chamfer with unit weights,
// and two raster sweeps of it are exact: the first takes each row from
// (y-1, z) and (y-1 .. y+1, z-1), the second from (y+1, z) and
// (y-1 .. y+1, z+1).  No per-line table and no search: a row of 256 bricks
// costs 15 vector instructions per sweep, where a line scan spends 9 per step
// of 64 bricks and pass (4 x 9 x 2 for the same bricks in y and z), with two
// dependent LDS accesses in each.
//
// General maps, whose rows are not distances, keep the line scans of
// pdm_kernels.hip (pdm_distance_yz promises their definition on any input).
//
// Parallelism.  A work-group takes up to 64/W maps (W lanes per row, 4 bricks
// each).  Its waves run plane after plane, wave w plane w, w + NW, ..., each
// two blocks of kSweepRows rows behind the wave before it, from which it gets
// that plane's rows through a ring in LDS; one barrier per block.  The planes
// are cut in two parts with a work-group each: the first sweep runs z towards
// the middle in both, the second away from it, starting from the other part's
// nearest plane.  That is still exact: the first sweep covers the paths whose
// y ascends in a plane and whose z moves towards the middle, the second those
// whose y descends and whose z moves away from it; a path to the other part
// takes its +y steps in its first plane, then crosses, then takes its -y
// steps.  The second sweep of one part may find the other part's plane before
// or after that part's own second sweep of it (both run in one launch, and
// each byte is one or the other): any value between the first sweep's result
// and the final distance gives the same distances, since the final ones never
// exceed one more than their neighbours' and the first sweep's are enough.
//
// Bound, where fewer work-groups than compute units run, by their number, and
// on a unit by a mix: about 40 instructions per row and wave in all, of which
// one issues per SIMD and 4 cycles.  64 maps of 256x256x199 (128 work-groups on
// 256 units): a wave issues in 32% of its cycles, waits to issue in 33% and
// waits for its barrier, ring or loads in 34%; 23% of the chip's vector slots.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "pdm_launch.h"
#include "pdm_packed.h"

namespace pdm {

constexpr int kWave = 64;
constexpr int kBufferRaw = 0x00020000;     // raw buffer, 32-bit data format (gfx9 family)
constexpr uint32_t kBeyond = 0x01FF01FFu;  // a neighbour outside the row: above every distance
constexpr uint32_t kCap2 = 0x00FF00FFu;    // two capped distances

// 4 bricks of a row: bytes 0, 2 and bytes 1, 3 as 16-bit pairs
struct RowQuad {
    uint32_t e, o;
};

// Packed 16-bit minimum of three.  The values are below 0x0400, i.e. positive
// half-precision subnormals, whose order is that of the integers (subnormals
// are kept: the default mode of HIP kernels).
__device__ __forceinline__ uint32_t pk_min3(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    __asm__("v_pk_minimum3_f16 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
// One row.  In: the row's values h, x = 1 + min3x(previous row of the sweep),
// q = the same for the three rows of the plane before.  S = min(h, x, q);
// out: the packed row, and x = 1 + min3x(S) with min3x the minimum over x-1,
// x, x+1.  One block, so that the two wait states between a VALU write and
// its cross-lane read are filled with the row's own work.
__device__ __forceinline__ uint32_t sweep_row(uint32_t he, uint32_t ho, const RowQuad q, RowQuad& x,
                                              uint32_t edge_l, uint32_t edge_r) {
    uint32_t w, se, so, l, r, xe, xo;
    __asm__(
        "v_pk_minimum3_f16 %[so], %[ho], %[xo], %[qo]\n\t"
        "v_pk_minimum3_f16 %[se], %[he], %[xe], %[qe]\n\t"
        "v_lshl_or_b32 %[w], %[so], 8, %[se]\n\t"
        "v_or_b32_dpp %[l], %[so], %[el] wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_or_b32_dpp %[r], %[se], %[er] wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_alignbit_b32 %[l], %[so], %[l], 16\n\t"
        "v_alignbit_b32 %[r], %[r], %[se], 16\n\t"
        "v_pk_minimum3_f16 %[l], %[se], %[so], %[l]\n\t"
        "v_pk_minimum3_f16 %[r], %[so], %[se], %[r]\n\t"
        "v_pk_add_u16 %[ne], %[l], 1 op_sel_hi:[1,0]\n\t"
        "v_pk_add_u16 %[no], %[r], 1 op_sel_hi:[1,0]"
        : [w] "=&v"(w), [se] "=&v"(se), [so] "=&v"(so), [l] "=&v"(l), [r] "=&v"(r), [ne] "=&v"(xe),
          [no] "=&v"(xo)
        : [he] "v"(he), [ho] "v"(ho), [xe] "v"(x.e), [xo] "v"(x.o), [qe] "v"(q.e), [qo] "v"(q.o),
          [el] "v"(edge_l), [er] "v"(edge_r));
    x.e = xe;
    x.o = xo;
    return w;
}

__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// What one work-group sweeps: up to 64/W maps side by side in its lanes (each
// in a segment of W lanes), planes [z_lo, z_hi).
struct SweepTask {
    uint8_t* base;      // first map
    int64_t G;
    int maps;           // maps present in the lanes
    int Bx, By, Bz, W;
    int part, parts, split;
};

// One sweep of a work-group over its planes.  PH 0: first sweep, y ascending;
// PH 1: second sweep, y descending.
// EVEN: By is a multiple of kSweepRows.
// PAD: some lanes hold no brick (4W > Bx, or fewer maps than the wave takes).
// RAGGED: rows end inside a quad, or rows are not 4-byte aligned.
template <int PH, bool EVEN, bool PAD, bool RAGGED>
__device__ __forceinline__ void sweep(const SweepTask& a, RowQuad* lds) {
    constexpr int RB = kSweepRows;
    constexpr int kBlock = RB * kWave;  // entries of one block of rows
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int NW = blockDim.x / kWave;
    const int seg = lane / a.W, q = lane & (a.W - 1);
    const int nb = seg < a.maps ? max(0, min(4, a.Bx - 4 * q)) : 0;
    const uint32_t pad = PAD && nb < 4 ? ~0u << (8 * nb) : 0u;
    const uint32_t pad_e = even_bytes(pad), pad_o = odd_bytes(pad);
    const uint32_t edge_l = q == 0 ? kBeyond : 0u, edge_r = q == a.W - 1 ? kBeyond : 0u;
    // a quad cut by the row end is the row's last 4 bytes, shifted
    const bool cut = RAGGED && nb > 0 && nb < 4;
    const int shift = cut ? 8 * (4 - nb) : 0;
    // lanes without bricks address past the buffer: their loads return 0 and
    // their stores are dropped
    const int voff = nb > 0 ? (int)(seg * a.G) + 4 * q - shift / 8 : -4;
    const int records = (int)(a.maps * a.G);
    const int Bx = a.Bx, By = a.By, plane = Bx * By;
    const int nblk = (By + RB - 1) / RB;
    const int period = max(nblk, 2 * NW);
    // rings: two blocks between neighbouring waves; between the last wave and
    // wave 0 as many as the last wave runs ahead
    const int last_ring = (period - 2 * NW + 2) * kBlock;
    const int ring_w = wave == NW - 1 ? last_ring : 2 * kBlock, ring_r = wave == 0 ? last_ring : 2 * kBlock;
    RowQuad* const out_ring = lds + wave * (2 * kBlock) + lane;
    const RowQuad* const in_ring = lds + (wave == 0 ? NW - 1 : wave - 1) * (2 * kBlock) + lane;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(a.base, (short)0, records, kBufferRaw);
    const bool up = (PH == 0) == (a.part == 0);  // z ascending
    // with two parts the second sweep starts from the other part's nearest
    // plane, which it reads but does not write
    const int ahead = PH == 1 && a.parts == 2 ? 1 : 0;
    const int z_lo = a.part == 0 ? 0 : a.split, z_hi = a.part == 0 ? a.split : a.Bz;
    const int np = z_hi - z_lo + ahead;
    // offsets of the first plane's first row in sweep order, and from plane to plane
    const int first = ((up ? z_lo - ahead : z_hi - 1 + ahead) * By + (PH == 0 ? 0 : By - 1)) * Bx;
    const int zstep = up ? plane : -plane;
    const int ystep = PH == 0 ? Bx : -Bx, last_row = (By - 1) * ystep;
    const int steps = ((np + NW - 1) / NW - 1) * period + nblk + 2 * (NW - 1);

    // Row r of the block at offset `at` of the plane that ends at `end`; every
    // offset is inside the maps.  Rows past the last: the last again.
    auto load_row = [&](int at, int end) -> uint32_t {
        if (!EVEN) at = PH == 0 ? min(at, end) : max(at, end);
        return __builtin_amdgcn_raw_buffer_load_b32(rs, voff, at, 0);
    };
    // plane and block (kf, bf), three steps ahead of this wave's: the next to be requested
    int kf = wave, bf = -2 * wave;
    auto ahead_at = [&](int& end) -> int {
        const int p = first + min(kf, np - 1) * zstep;
        end = p + last_row;
        return p + max(0, min(bf, nblk - 1)) * (RB * ystep);
    };
    auto advance = [&]() {
        if (++bf == period) {
            bf = 0;
            kf += NW;
        }
    };
    uint32_t rows[4][RB];  // loaded blocks: one in use, three in flight
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        int end, at = ahead_at(end);
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            rows[i][r] = load_row(at, end);
            at += ystep;
        }
        advance();
    }
    lds_barrier();
    RowQuad X = {kCap2, kCap2}, Pm = X;
    RowQuad pw[RB];                   // rows of the plane before: the block's rows 0 .. RB-1
    int k = wave, b = -2 * wave;      // plane and block of this wave in this step
    int slot_w = 0, slot_r = kBlock;  // ring slots written and read in this step
#pragma unroll
    for (int r = 0; r < RB; ++r) pw[r] = {kCap2, kCap2};  // wave 0: nothing before the first plane
    // One step.  A wave without work in it (before its first block, between
    // planes, past its last plane) runs the same code on any rows, and its
    // stores are dropped: no branch, so that the waits for the loads count
    // exactly the loads and stores issued since.
    auto step = [&](const uint32_t (&in)[RB], uint32_t (&fetch)[RB]) {
        int end, at = ahead_at(end);
        // rows of this block to be stored (those of the other part's plane are not)
        const int left = b >= 0 && b < nblk && k < np && k >= ahead ? By - b * RB : 0;
        int off = first + k * zstep + b * (RB * ystep);
        const int rec = left > 0 ? records : 0;
        // the next block's first row of the plane before; past its end the last row again
        RowQuad after = in_ring[slot_r];
        if (b + 1 >= nblk || k == 0) after = pw[RB - 1];
        if (b == 0) {
            X = {kCap2, kCap2};
            Pm = X;
        }
        RowQuad* out = out_ring + slot_w;
        RowQuad P0 = pw[0];
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            fetch[r] = load_row(at, end);
            at += ystep;
            const RowQuad P1 = r + 1 < RB ? pw[r + 1] : after;
            const RowQuad m = {pk_min3(Pm.e, P0.e, P1.e), pk_min3(Pm.o, P0.o, P1.o)};
            uint32_t h = in[r];
            if (RAGGED) h >>= shift;
            uint32_t w = sweep_row(even_bytes(h) | pad_e, odd_bytes(h) | pad_o, m, X, edge_l, edge_r);
            Pm = P0;
            P0 = P1;
            out[r * kWave] = X;
            if constexpr (RAGGED) {
                const uint32_t prev = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x138, 0xf, 0xf, true);
                w = cut ? (uint32_t)((((uint64_t)w << 32) | prev) >> (32 - shift)) : w;
            }
            // rows past the last one go nowhere
            const __amdgpu_buffer_rsrc_t ws = __builtin_amdgcn_make_buffer_rsrc(
                a.base, (short)0, EVEN ? rec : r < left ? records : 0, kBufferRaw);
            __builtin_amdgcn_raw_buffer_store_b32(w, ws, voff, off, 0);
            off += ystep;
            __builtin_amdgcn_sched_barrier(0);
        }
        advance();
        if (++b == period) {
            b = 0;
            k += NW;
        }
        if (k > 0) {  // plane 0 has none before it
            const RowQuad* p = in_ring + slot_r;
#pragma unroll
            for (int r = 0; r < RB; ++r) pw[r] = p[r * kWave];
        }
        slot_w += kBlock;
        if (slot_w == ring_w) slot_w = 0;
        slot_r += kBlock;
        if (slot_r == ring_r) slot_r = 0;
        lds_barrier();
    };
    for (int t = 0; t < steps; t += 4) {
        step(rows[0], rows[3]);
        step(rows[1], rows[0]);
        step(rows[2], rows[1]);
        step(rows[3], rows[2]);
    }
}

template <int PH, bool EVEN, bool PAD, bool RAGGED>
__global__ void __launch_bounds__(64 * kSweepWaves) k_sweep(uint8_t* __restrict__ maps, SweepArgs a) {
    extern __shared__ __align__(16) RowQuad lds[];
    const int per = kWave / a.W, group = blockIdx.x / 2;
    SweepTask t;
    t.base = maps + (int64_t)group * per * a.G;
    t.G = a.G;
    t.maps = min(per, a.count - group * per);
    t.Bx = a.Bx;
    t.By = a.By;
    t.Bz = a.Bz;
    t.W = a.W;
    t.parts = 2;
    t.part = blockIdx.x % 2;
    t.split = (a.Bz + 1) / 2;
    sweep<PH, EVEN, PAD, RAGGED>(t, lds);
}

// The same over the volumes of a batched build: one sweep of the work-groups
// of class cls (see BatchVol), in descriptor order.
template <int PH>
__global__ void __launch_bounds__(64 * kSweepBatchWaves) k_batch_sweep(const BatchVol* __restrict__ vols, int count,
                                                                  int cls) {
    extern __shared__ __align__(16) RowQuad lds[];
    int lo = 0, hi = count - 1;  // last volume whose first work-group is <= this one
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (vols[mid].sweep_first[cls] <= (int)blockIdx.x)
            lo = mid;
        else
            hi = mid - 1;
    }
    const BatchVol& d = vols[lo];
    const int local = (int)blockIdx.x - d.sweep_first[cls];
    SweepTask t;
    t.parts = d.Bz >= kSweepMinPlanes ? 2 : 1;
    t.part = local % t.parts;
    t.split = t.parts == 2 ? (d.Bz + 1) / 2 : d.Bz;
    t.G = d.G;
    t.Bx = d.Bx;
    t.By = d.By;
    t.Bz = d.Bz;
    t.W = d.row_lanes;
    const int per = kWave / t.W, group = local / t.parts;
    t.maps = min(per, d.n - group * per);
    t.base = d.pdms + (int64_t)group * per * d.G;
    if (d.store_vec)
        sweep<PH, false, true, false>(t, lds);
    else
        sweep<PH, false, true, true>(t, lds);
}

// ---------------------------------------------------------------------------
// k_slice_y: the y pass over slices (rows of x distances), in place, two waves
// to a slice (64/W slices side by side in the lanes), each with its half of
// the rows in registers: each sweeps its half from the outside in, the waves
// exchange the row that the next one would build on, and each sweeps back
// from the inside out over its own results.  A one-sided sweep over the other
// direction's results, started from the other half's last row, is the
// two-sided pass.  No table, no LDS but for the exchange, and a slice is a
// work-group of its own: enough of them for one map already.
//
// NCH: chunks of 16 rows a wave's half spans.  A half of fewer rows starts with
// rows outside the grid, at the cap: they change nothing.
// Bound by the waves' chain of 2 x By/2 rows (13 vector instructions each) for
// one map, by memory for many.  Measured against the line scans: 32 maps of
// 128x128x115 57 -> 21 us (5.7 TB/s read and written), one map of 256x256x199
// 24 -> 13 us, of 128x122x113 11 -> 7 us.
// ---------------------------------------------------------------------------
template <int NCH, bool GENERAL>
__device__ __forceinline__ void slice_y(uint8_t* maps, int64_t slices, int64_t s0, int Bx, int By, int W,
                                        RowQuad (&inner)[2][kWave]) {
    constexpr int NR = 16 * NCH;
    const int lane = threadIdx.x & (kWave - 1);
    const int half = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int per = kWave / W, seg = lane / W, q = lane & (W - 1);
    const int here = (int)(slices - s0 < per ? slices - s0 : per);
    const int plane = Bx * By;
    const int nb = seg < here ? max(0, min(4, Bx - 4 * q)) : 0;
    const uint32_t pad = GENERAL && nb < 4 ? ~0u << (8 * nb) : 0u;
    const uint32_t edge_l = q == 0 ? kBeyond : 0u, edge_r = q == W - 1 ? kBeyond : 0u;
    const bool cut = GENERAL && nb > 0 && nb < 4;  // the row's last 4 bytes, shifted
    const int shift = cut ? 8 * (4 - nb) : 0;
    const int voff = nb > 0 ? seg * plane + 4 * q - shift / 8 : -4;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(maps + s0 * plane, (short)0, here * plane, kBufferRaw);
    const int rows = half == 0 ? By / 2 : By - By / 2;
    const int out = NR - rows;  // rows outside the grid, first
    const int ystep = half == 0 ? Bx : -Bx;
    int off = half == 0 ? 0 : (By - 1) * Bx;
    uint32_t w[NR], all = ~0u;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        w[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, voff, off, 0);
        off += i < 16 && i < out ? 0 : ystep;
    }
    const RowQuad cap = {kCap2, kCap2};
    RowQuad X = cap;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        uint32_t h = w[i];
        if (GENERAL) h = (h >> shift) | pad;
        if (i < 16) h |= i < out ? ~0u : 0u;
        all &= h;
        w[i] = sweep_row(even_bytes(h), odd_bytes(h), cap, X, edge_l, edge_r);
    }
    inner[half][lane] = X;
    __syncthreads();
    X = inner[1 - half][lane];
    // no brick in the slices: everything stays at the cap
    if (__ballot(all != ~0u || pk_min16(pk_min16(X.e, X.o), kCap2) != kCap2) == 0ull) return;
    __asm__("" : "+s"(off));  // one running offset, not a register for each row's
#pragma unroll
    for (int i = NR - 1; i >= 0; --i) {
        uint32_t v = sweep_row(even_bytes(w[i]), odd_bytes(w[i]), cap, X, edge_l, edge_r);
        if constexpr (GENERAL) {
            const uint32_t prev = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, true);
            v = cut ? (uint32_t)((((uint64_t)v << 32) | prev) >> (32 - shift)) : v;
        }
        off -= ystep;
        if (i >= 16 || i >= out) __builtin_amdgcn_raw_buffer_store_b32(v, rs, voff, off, 0);
    }
}

template <int NCH, bool GENERAL>
__global__ void __launch_bounds__(2 * kWave) k_slice_y(uint8_t* __restrict__ maps, int64_t slices, int Bx,
                                                       int By, int W) {
    __shared__ RowQuad inner[2][kWave];
    slice_y<NCH, GENERAL>(maps, slices, (int64_t)blockIdx.x * (kWave / W), Bx, By, W, inner);
}

// The volumes of a batch with 16 * LO + 1 .. 16 * HI rows to a half.
template <int LO, int HI>
__global__ void __launch_bounds__(2 * kWave) k_batch_slice_y(const BatchVol* __restrict__ vols, BatchBlocks b) {
    __shared__ RowQuad inner[2][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    // the last volume whose first work-group is not after this one
    const uint64_t before = __ballot(lane < b.count && b.first[lane] <= (int)blockIdx.x);
    const int k = 63 - __clzll((long long)before);
    const BatchVol& d = vols[k];
    const int W = d.row_lanes, Bx = d.Bx, By = d.By;
    const int64_t s0 = (int64_t)((int)blockIdx.x - b.first[k]) * (kWave / W), slices = (int64_t)d.n * d.Bz;
    switch (((By + 1) / 2 + 15) / 16) {
#define PDM_SLICE_CASE(N)                                                       \
    case N:                                                                     \
        if constexpr (N > LO && N <= HI)                                        \
            slice_y<N, true>(d.pdms, slices, s0, Bx, By, W, inner);             \
        break;
        PDM_SLICE_CASE(1) PDM_SLICE_CASE(2) PDM_SLICE_CASE(3) PDM_SLICE_CASE(4)
        PDM_SLICE_CASE(5) PDM_SLICE_CASE(6) PDM_SLICE_CASE(7) PDM_SLICE_CASE(8)
#undef PDM_SLICE_CASE
        default: break;
    }
}

hipError_t launch_slice_y(uint8_t* maps, int count, int Bx, int By, int Bz, hipStream_t s) {
    const int W = row_lanes(Bx), per = kWave / W;
    const int64_t slices = (int64_t)count * Bz, blocks = (slices + per - 1) / per;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    const int nch = ((By + 1) / 2 + 15) / 16;
    const bool general = 4 * W != Bx || slices % per != 0;
    switch (nch) {
#define PDM_SLICE_CASE(N)                                                                              \
    case N:                                                                                            \
        if (general)                                                                                   \
            k_slice_y<N, true><<<(unsigned)blocks, 2 * kWave, 0, s>>>(maps, slices, Bx, By, W);        \
        else                                                                                           \
            k_slice_y<N, false><<<(unsigned)blocks, 2 * kWave, 0, s>>>(maps, slices, Bx, By, W);       \
        break;
        PDM_SLICE_CASE(1) PDM_SLICE_CASE(2) PDM_SLICE_CASE(3) PDM_SLICE_CASE(4)
        PDM_SLICE_CASE(5) PDM_SLICE_CASE(6) PDM_SLICE_CASE(7) PDM_SLICE_CASE(8)
#undef PDM_SLICE_CASE
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int LO, int HI>
static hipError_t launch_batch_slices(const BatchVol* h_vols, int count, const BatchVol* d_vols, hipStream_t s) {
    BatchBlocks b;
    int64_t blocks = 0;
    b.count = count;
    for (int k = 0; k < count; ++k) {
        const BatchVol& d = h_vols[k];
        const int nch = ((d.By + 1) / 2 + 15) / 16, per = kWave / d.row_lanes;
        b.first[k] = (int32_t)blocks;
        if (d.slices && nch > LO && nch <= HI) blocks += ((int64_t)d.n * d.Bz + per - 1) / per;
    }
    if (blocks == 0) return hipSuccess;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    k_batch_slice_y<LO, HI><<<(unsigned)blocks, 2 * kWave, 0, s>>>(d_vols, b);
    return hipGetLastError();
}

hipError_t launch_batch_slice_y(const BatchVol* h_vols, int count, const BatchVol* d_vols, hipStream_t s) {
    const hipError_t e = launch_batch_slices<0, 4>(h_vols, count, d_vols, s);
    return e == hipSuccess ? launch_batch_slices<4, 8>(h_vols, count, d_vols, s) : e;
}

// LDS of a work-group: the rings hold one period of blocks in all.
static size_t sweep_lds(int By, int NW) {
    const int nblk = (By + kSweepRows - 1) / kSweepRows;
    return (size_t)std::max(nblk, 2 * NW) * kSweepRows * kWave * sizeof(RowQuad);
}

// Sweep work-groups of the volumes that take them, in their launch's order.
void batch_sweep_items(BatchVol* vols, int count) {
    int32_t first[2] = {0, 0};
    for (int k = 0; k < count; ++k) {
        BatchVol& d = vols[k];
        const int per = kWave / d.row_lanes, cls = batch_sweep_class(d.By);
        d.sweep_first[0] = first[0];
        d.sweep_first[1] = first[1];
        if (!batch_volume_sweeps({d.n, d.Bx, d.By, d.Bz})) continue;
        d.sweep_items[cls] = (d.n + per - 1) / per * batch_sweep_parts(d.Bz);
        first[cls] += d.sweep_items[cls];
        d.items[1] = d.items[2] = 0;
    }
}

hipError_t launch_batch_sweep(const BatchVol* h_vols, int count, const BatchVol* d_vols, hipStream_t s) {
    for (int ph = 0; ph < 2; ++ph)
        for (int cls = 0; cls < 2; ++cls) {
            int64_t total = 0;
            int by = 0;
            for (int k = 0; k < count; ++k) {
                total += h_vols[k].sweep_items[cls];
                if (h_vols[k].sweep_items[cls] > 0) by = std::max(by, h_vols[k].By);
            }
            if (total == 0) continue;
            if (total > INT32_MAX) return hipErrorInvalidValue;
            const size_t lds = sweep_lds(by, kSweepBatchWaves);
            if (ph == 0)
                k_batch_sweep<0><<<(unsigned)total, kSweepBatchWaves * kWave, lds, s>>>(d_vols, count, cls);
            else
                k_batch_sweep<1><<<(unsigned)total, kSweepBatchWaves * kWave, lds, s>>>(d_vols, count, cls);
        }
    return hipGetLastError();
}

template <int PH>
static void launch_sweep_phase(uint8_t* maps, const SweepArgs& a, unsigned grid, int nw, bool pad, bool ragged,
                               hipStream_t s) {
    const bool even = a.By % kSweepRows == 0;
    const size_t lds = sweep_lds(a.By, nw);
    if (ragged)
        k_sweep<PH, false, true, true><<<grid, nw * kWave, lds, s>>>(maps, a);
    else if (even && !pad)
        k_sweep<PH, true, false, false><<<grid, nw * kWave, lds, s>>>(maps, a);
    else if (even)
        k_sweep<PH, true, true, false><<<grid, nw * kWave, lds, s>>>(maps, a);
    else
        k_sweep<PH, false, true, false><<<grid, nw * kWave, lds, s>>>(maps, a);
}

hipError_t launch_sweep(uint8_t* maps, int count, int Bx, int By, int Bz, hipStream_t s) {
    SweepArgs a;
    a.G = (int64_t)Bx * By * Bz;
    a.count = count;
    a.Bx = Bx;
    a.By = By;
    a.Bz = Bz;
    a.W = row_lanes(Bx);
    const int per = kWave / a.W;
    const unsigned grid = 2u * (unsigned)((count + per - 1) / per);
    const int nw = sweep_waves((Bz + 1) / 2 + 1, By);
    const bool ragged = Bx % 4 != 0 || ((uintptr_t)maps & 3) != 0;
    const bool pad = 4 * a.W != Bx || count % per != 0;
    launch_sweep_phase<0>(maps, a, grid, nw, pad, ragged, s);
    launch_sweep_phase<1>(maps, a, grid, nw, pad, ragged, s);
    return hipGetLastError();
}

}  // namespace pdm
