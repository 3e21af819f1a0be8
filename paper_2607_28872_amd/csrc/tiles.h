// Column-aligned particle chunks and their LDS neighbour windows.
//
// The cell-sorted particles of one (x, y) cell column (2-D: one x column) are
// split into chunks of at most kChunk consecutive particles.  Every neighbour
// of a chunk's particles lies in the chunk's window: the 3^(d-1) columns
// around its own, restricted to the z cells spanned by the chunk widened by
// one cell on each side.  Each of those columns contributes one contiguous
// range of sorted indices, and the ranges are concatenated in increasing order
// of their first index.  A work-group stages the window's particle records in
// LDS once; neighbour lists stored as 16-bit window offsets then index LDS
// directly.  The window depends only on the grid, the cell table and the
// chunk, so the neighbour search and every consumer derive the same one.
#pragma once

#include "common.h"

namespace vct {

constexpr int kChunk = 64;        // particles per chunk
constexpr int kMaxRanges = 9;     // 3 x 3 columns in 3-D, 3 in 2-D

// Mean row length up to which a set takes the kernels' short-row shapes, whose
// register slots hold 32 entries of a row in 2-D (the FP64 apply 28) and 64 in
// 3-D: above the mean rows of the supports in use that fit them (2-D: 26 at
// R = 3 d0, 20 at 2.4 d0; 3-D: 57 at 2.4 d0).  The next supports up (3-D: 103 at
// 3 d0) would run most of each row outside the slots; at mean rows of 29 and 30
// the FP64 apply's last entries take the loop after them.
template <int D> constexpr int64_t short_row() { return D == 2 ? 30 : 62; }
// The mean row length the neighbour search left in the list (nnz unset: long).
inline int64_t mean_row(const vct_nlist* nl) {
    return nl->nnz > 0 && nl->n > 0 ? nl->nnz / nl->n : INT32_MAX;
}

// Window particles of a cell column up to which the adjoint's push form holds
// the column's records and two-word sums (and R2's records, fields and sums) in
// LDS.  The search counts the particles of wider columns into
// nl->wide_particles, as 1 + their number (0: a list without the count).
constexpr int kPushWindow = 3200;

// Chunk table: chunk b covers sorted particles [start[b], start[b+1]) of
// column info[b].x, z cells [info[b].y, info[b].z].
struct ChunkTable {
    const int32_t* start;   // [nchunks + 1]
    const int4* info;       // [nchunks]: column, zlo, zhi, unused
    const int64_t* count;   // device scalar: number of chunks
};

// The chunk of this work-group, one per block; false for the blocks past the
// last chunk.  The launches size their grid by an upper bound (columns + n /
// 64 + 1): the count stays on the device.  The chunks themselves, not the
// blocks, are shared out over the XCDs: dealt out by the grid, the last XCDs
// hold the blocks that return at once, and the others take 11% more chunks
// than their share in 3-D at R = 3 d0 (four and a half chunks a column), 30%
// more for the cubic spline (two and a half).  Sharing out the chunks, one
// MI355X: FP64 apply 1.18 -> 1.09 ms (2,097,152 particles) and 0.56 -> 0.49 ms
// (1,048,352), with the cubic spline 0.90 -> 0.77 ms; moment sweeps 5.51 ->
// 5.16 ms (8,388,608).
__device__ __forceinline__ bool chunk_of_block(const int64_t* __restrict__ nchunks, uint32_t& b) {
    const uint32_t n = (uint32_t)*nchunks;
    if (blockIdx.x >= n) return false;
    b = xcd_tile(blockIdx.x, n);
    return true;
}

template <int D> struct WindowT {
    int nr;
    int64_t gstart[kMaxRanges];
    int off[kMaxRanges + 1];
};

// Columns are numbered c0 * nc1 + c1 in 3-D and c0 in 2-D; z is the last axis.
template <int D>
__device__ __forceinline__ int64_t col_key(const Grid& g, int64_t col, int64_t z) {
    if (D == 3) return col * g.nc[2] + z;
    return col * g.nc[1] + z;
}

template <int D>
__device__ __forceinline__ int64_t grid_nz(const Grid& g) { return D == 3 ? g.nc[2] : g.nc[1]; }

template <int D>
__device__ __forceinline__ int64_t grid_ncols(const Grid& g) { return D == 3 ? g.nc[0] * g.nc[1] : g.nc[0]; }

// Window of a chunk (same result in every thread that calls it).
template <int D>
__device__ __forceinline__ void chunk_window(const Grid& g, const int64_t* __restrict__ cs, int4 info,
                                             WindowT<D>& w) {
    const int64_t nz = grid_nz<D>(g);
    const int64_t zlo = info.y > 0 ? info.y - 1 : 0;
    const int64_t zhi = info.z + 1 < nz ? info.z + 1 : nz - 1;
    int64_t cx, cy = 0;
    if (D == 3) { cx = info.x / g.nc[1]; cy = info.x % g.nc[1]; }
    else cx = info.x;
    w.nr = 0;
    int acc = 0;
    for (int dx = -1; dx <= 1; ++dx) {
        const int64_t x = cx + dx;
        if (x < 0 || x >= g.nc[0]) continue;
        for (int dy = (D == 3 ? -1 : 0); dy <= (D == 3 ? 1 : 0); ++dy) {
            int64_t colid;
            if (D == 3) {
                const int64_t y = cy + dy;
                if (y < 0 || y >= g.nc[1]) continue;
                colid = x * g.nc[1] + y;
            } else {
                colid = x;
            }
            const int64_t a = cs[col_key<D>(g, colid, zlo)], b = cs[col_key<D>(g, colid, zhi) + 1];
            w.gstart[w.nr] = a;
            w.off[w.nr] = acc;
            acc += (int)(b - a);
            ++w.nr;
        }
    }
    w.off[w.nr] = acc;
}

// The same window computed by one whole wave in parallel: lane r handles the
// r-th column of the 3^(d-1) (in the order of chunk_window), the ranges are
// compacted with a ballot and their offsets formed with a prefix sum over
// lanes.  Every lane of the calling wave must call it.
template <int D>
__device__ __forceinline__ void chunk_window_wave(const Grid& g, const int64_t* __restrict__ cs, int4 info,
                                                  WindowT<D>& w) {
    const int lane = threadIdx.x % kWave;
    const int64_t nz = grid_nz<D>(g);
    const int64_t zlo = info.y > 0 ? info.y - 1 : 0;
    const int64_t zhi = info.z + 1 < nz ? info.z + 1 : nz - 1;
    constexpr int ncand = D == 3 ? 9 : 3;
    int64_t x, y = 0, colid;
    if (D == 3) {
        const int nc1 = (int)g.nc[1];   // columns are numbered in 32 bits
        x = info.x / nc1 + lane / 3 - 1;
        y = info.x % nc1 + lane % 3 - 1;
        colid = x * g.nc[1] + y;
    } else {
        x = info.x + lane - 1;
        colid = x;
    }
    const bool in = lane < ncand && x >= 0 && x < g.nc[0] && (D == 2 || (y >= 0 && y < g.nc[1]));
    int64_t a = 0;
    int len = 0;
    if (in) {
        a = cs[col_key<D>(g, colid, zlo)];
        len = (int)(cs[col_key<D>(g, colid, zhi) + 1] - a);
    }
    const uint64_t m = (uint64_t)__ballot(in);
    const int slot = __popcll(m & ((1ull << lane) - 1ull));
    int incl = len;
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
        const int v = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += v;
    }
    const int total = __shfl(incl, ncand - 1, kWave);
    if (in) {
        w.gstart[slot] = a;
        w.off[slot] = incl - len;
    }
    if (lane == 0) {
        w.nr = __popcll(m);
        w.off[__popcll(m)] = total;
    }
}

// Stored windows: chunk b's WindowT at tab + 32 b (int32 words).
static_assert(sizeof(WindowT<3>) <= 32 * sizeof(int32_t), "a stored window fits 32 words");
static_assert(sizeof(WindowT<2>) == sizeof(WindowT<3>), "one stored layout for both dimensions");

// Store (lanes 0..31 of the wave that formed w) or load (lanes 0..31 of any
// wave) a window as 32 int32 words.
template <int D>
__device__ __forceinline__ void window_store(const WindowT<D>& w, int32_t* __restrict__ tab, uint32_t b) {
    const int lane = threadIdx.x % kWave;
    if (lane < (int)(sizeof(WindowT<D>) / 4)) tab[(int64_t)b * 32 + lane] = reinterpret_cast<const int32_t*>(&w)[lane];
}
template <int D>
__device__ __forceinline__ void window_load(const int32_t* __restrict__ tab, uint32_t b, WindowT<D>& w) {
    const int lane = threadIdx.x % kWave;
    if (lane < (int)(sizeof(WindowT<D>) / 4)) reinterpret_cast<int32_t*>(&w)[lane] = tab[(int64_t)b * 32 + lane];
}

// global sorted index of window offset t
template <int D>
__device__ __forceinline__ int64_t window_global(const WindowT<D>& w, int t) {
    t = dcheck(t, w.off[w.nr], kChkWindow);
    int r = 0;
#pragma unroll
    for (int k = 1; k < kMaxRanges; ++k)
        if (k < w.nr && t >= w.off[k]) r = k;
    return w.gstart[r] + (t - w.off[r]);
}

// ------------------------------------------------------------------ row sweeps

// Launch shapes of the one-sweep kernels (conventional operators, pressure
// right-hand side, corrector and diagonal): lanes per particle, row entries a
// lane holds in registers, LDS window (records) and waves per SIMD, by class of
// the mean row length (short_row).  The offsets of a row are read once, up
// front, and the records one slot ahead of the arithmetic; read entry by entry
// inside the loop they cost a trip to the L2 per entry.
enum { kRowsLong = 0, kRowsShort3 = 1, kRowsShort2 = 2 };
template <int C> struct RowShape;
template <> struct RowShape<kRowsLong> { static constexpr int lanes = 8, slots = 14, win = 1400, waves = 4; };
template <> struct RowShape<kRowsShort3> { static constexpr int lanes = 4, slots = 16, win = 1184, waves = 3; };
template <> struct RowShape<kRowsShort2> { static constexpr int lanes = 4, slots = 8, win = 448, waves = 4; };

// A lane's share of a row: entries rb + lane + LANES s, s < SLOTS, two 16-bit
// window offsets per register (slots past the row's end repeat its first).
template <int LANES, int SLOTS> struct RowSlots {
    uint32_t pk[(SLOTS + 1) / 2];
    int n = 0;   // filled slots
    int64_t tail, end;
    __device__ __forceinline__ RowSlots(const uint16_t* __restrict__ col16, int64_t rb, int64_t re, int lane) {
        const int len = (int)(re - rb);
        const uint16_t* c = col16 + rb + lane;
        const uint32_t first = len > 0 ? (uint32_t)col16[rb] : 0u;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const bool in = lane + LANES * s < len;
            const uint32_t v = in ? (uint32_t)c[LANES * s] : first;
            n += in ? 1 : 0;
            if (s % 2 == 0) pk[s / 2] = v;
            else pk[s / 2] |= v << 16;
        }
        tail = rb + lane + (int64_t)LANES * SLOTS;
        end = re;
    }
    __device__ __forceinline__ int at(int s, int W) const {
        return dcheck((int)((pk[s / 2] >> (16 * (s % 2))) & 0xffffu), W, kChkWindow);
    }
};

// Stages the records of window offsets [0, W), W <= WIN: every load of a thread
// before its first LDS store.
template <int WIN, int THREADS, class Load, class Store>
__device__ __forceinline__ void stage_window(int W, Load&& load, Store&& store) {
    constexpr int kRep = (WIN + THREADS - 1) / THREADS;
    decltype(load(0)) v[kRep];
#pragma unroll
    for (int k = 0; k < kRep; ++k) {
        const int t = threadIdx.x + k * THREADS;
        if (t < W) v[k] = load(t);   // lanes past the window load nothing (whole waves skip)
    }
#pragma unroll
    for (int k = 0; k < kRep; ++k) {
        const int t = threadIdx.x + k * THREADS;
        if (t < W) store(t, v[k]);
    }
}

// Visits every entry of a row: REC rec(t) of each window offset t, the records
// of the register slots requested one slot ahead, then the entries past them.
// in_lds (uniform): rec reads LDS, else memory (the whole row in the last loop,
// its offsets one entry ahead: 240,000 particles in 2-D with rows of 775, moment
// sweeps 2.06 -> 1.81 ms).
template <int LANES, int SLOTS, class Rec, class Body>
__device__ __forceinline__ void sweep_row(const RowSlots<LANES, SLOTS>& rs, const uint16_t* __restrict__ col16, int W,
                                          bool in_lds, Rec&& rec, Body&& body) {
    if (in_lds) {
        auto next = rec(rs.at(0, W));
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const auto q = next;
            if (s + 1 < SLOTS) next = rec(rs.at(s + 1, W));
            __builtin_amdgcn_sched_barrier(0);
            if (s < rs.n) body(q);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // (from memory the whole row by its offsets: a loop over the slots would
    // index the registers by a variable, which puts them in scratch memory)
    const int64_t e0 = in_lds ? rs.tail : rs.tail - (int64_t)LANES * SLOTS;
    uint32_t next = e0 < rs.end ? (uint32_t)col16[e0] : 0u;   // the offsets one entry ahead
    for (int64_t e = e0; e < rs.end; e += LANES) {
        const uint32_t t = next;
        if (e + LANES < rs.end) next = (uint32_t)col16[e + LANES];
        body(rec(dcheck((int)t, W, kChkWindow)));
    }
}

}  // namespace vct
