// Background-cell sort and neighbour lists (paper Sec. 3.1, Eq. SPH_neighbor_set;
// neighbour searches with background cells, Sec. 3.4).
//
// Cells are at least R wide, so every neighbour of a particle lies in the
// 3^d cells around its own.  Particles are sorted by (cell key, original index)
// with a counting sort; z is the fastest cell axis, so the three z-adjacent
// cells of one (x, y) column are contiguous in memory and each particle's
// candidates form 3^(d-1) contiguous ranges, visited in increasing order.
#include "common.h"
#include "tiles.h"

namespace vct {

// ------------------------------------------------------------------ small kernels

__global__ void k_fill_i64(int64_t* p, int64_t n, int64_t v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

static int fill_i64(int64_t* p, int64_t n, int64_t v, hipStream_t s) {
    if (n <= 0) return VCT_OK;
    VCT_LAUNCH("k_fill_i64", k_fill_i64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
    VCT_LAUNCH_CHECK();
    return VCT_OK;
}

// p[0..n) = 0 and q[0..m) = 0, m <= 256
__global__ void k_fill_i32(int32_t* p, int64_t n, int32_t* q, int m) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
    if (i < m) q[i] = 0;
}

static int zero_i32(int32_t* p, int64_t n, int32_t* q, int m, hipStream_t s) {
    VCT_LAUNCH("k_fill_i32", k_fill_i32, dim3((unsigned)((n > m ? n : m) + 255) / 256), dim3(256), 0, s, p, n, q, m);
    VCT_LAUNCH_CHECK();
    return VCT_OK;
}

// ------------------------------------------------------------------ exclusive scan

// out[i] = sum_{k<i} in[k] for i in [0, n], int32 -> int64.  Up to kScanOne
// values one work-group does it in one launch.  Beyond, per-tile sums and
// per-tile scans, each tile adding up the sums of the tiles before it by
// itself (up to kScanSelf tiles: at most 32 values per thread, from the L2; 8.4M
// values are 4,096 tiles); beyond that a single-block scan of the tile sums
// stands between the two.  A launch costs about as much as scanning 100,000
// values, and a small geometry is five scans: with three launches each they
// took 97 of the 280 us of its kernels (4,096 particles in 2-D).
constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;
constexpr int kScanOneThreads = 1024;
constexpr int kScanOne = kScanOneThreads * 16;
constexpr int kScanSelf = 8192;

template <int THREADS>
__device__ int64_t block_exclusive_scan(int64_t v, int64_t* lds_waves, int64_t* total) {
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
    int64_t inc = v;
    for (int o = 1; o < kWave; o <<= 1) {
        int64_t t = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += t;
    }
    if (lane == kWave - 1) lds_waves[wv] = inc;
    __syncthreads();
    int64_t wbase = 0, tot = 0;
    for (int k = 0; k < THREADS / kWave; ++k) {
        if (k < wv) wbase += lds_waves[k];
        tot += lds_waves[k];
    }
    __syncthreads();
    *total = tot;
    return wbase + inc - v;
}

// ITEMS consecutive values of a thread, as 16-byte loads where whole (in is
// 16-byte aligned, base a multiple of ITEMS)
template <int ITEMS>
__device__ __forceinline__ int64_t scan_load(const int32_t* __restrict__ in, int64_t n, int64_t base, int (&v)[ITEMS]) {
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < ITEMS; k += 4) {
        if (base + k + 4 <= n) {
            const int4 q = *reinterpret_cast<const int4*>(in + base + k);
            v[k] = q.x; v[k + 1] = q.y; v[k + 2] = q.z; v[k + 3] = q.w;
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) v[k + u] = base + k + u < n ? in[base + k + u] : 0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) s += v[k + u];
    }
    return s;
}

__global__ __launch_bounds__(kScanOneThreads) void k_scan_one(const int32_t* in, int64_t n, int64_t* out,
                                                             int64_t* total) {
    constexpr int kItems = kScanOne / kScanOneThreads;
    __shared__ int64_t lw[kScanOneThreads / kWave];
    const int64_t base = (int64_t)threadIdx.x * kItems;
    int v[kItems];
    const int64_t s = scan_load(in, n, base, v);
    int64_t tot;
    int64_t run = block_exclusive_scan<kScanOneThreads>(s, lw, &tot);
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        if (base + k < n) out[base + k] = run;
        run += v[k];
    }
    if (threadIdx.x == 0) {
        out[n] = tot;
        if (total) *total = tot;
    }
}

__global__ __launch_bounds__(kScanThreads) void k_scan_tiles(const int32_t* in, int64_t n, int64_t* tile_sums) {
    __shared__ int64_t lw[kScanThreads / kWave];
    int v[kScanItems];
    const int64_t s = scan_load(in, n, (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems, v);
    int64_t tot;
    block_exclusive_scan<kScanThreads>(s, lw, &tot);
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = tot;
}

__global__ void k_scan_sums(int64_t* sums, int64_t ntiles) {
    __shared__ int64_t lw[kScanThreads / kWave];
    int64_t carry = 0;
    for (int64_t b = 0; b < ntiles; b += kScanThreads) {
        int64_t i = b + threadIdx.x;
        int64_t v = i < ntiles ? sums[i] : 0;
        int64_t tot;
        int64_t ex = block_exclusive_scan<kScanThreads>(v, lw, &tot);
        if (i < ntiles) sums[i] = carry + ex;
        carry += tot;
    }
}

// scanned: tile_sums already holds each tile's offset
__global__ __launch_bounds__(kScanThreads) void k_scan_apply(const int32_t* in, int64_t n,
                                                            const int64_t* __restrict__ tile_sums, bool scanned,
                                                            int64_t* out, int64_t* total) {
    __shared__ int64_t lw[kScanThreads / kWave];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int v[kScanItems];
    const int64_t s = scan_load(in, n, base, v);
    int64_t off = 0, tot;
    if (scanned) {
        off = tile_sums[blockIdx.x];
    } else {
        int64_t before = 0;
        for (int64_t k = threadIdx.x; k < (int64_t)blockIdx.x; k += kScanThreads) before += tile_sums[k];
        block_exclusive_scan<kScanThreads>(before, lw, &off);
    }
    int64_t run = off + block_exclusive_scan<kScanThreads>(s, lw, &tot);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < n) out[base + k] = run;
        run += v[k];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        out[n] = off + tot;
        if (total) *total = off + tot;
    }
}

static size_t scan_ws_bytes(int64_t n) {
    int64_t ntiles = (n + kScanTile - 1) / kScanTile;
    return (size_t)(ntiles > 0 ? ntiles : 1) * sizeof(int64_t);
}

// out has n + 1 entries; out[n] is the total (n > 0: also written to *total when given)
static int exclusive_scan(const int32_t* in, int64_t n, int64_t* out, int64_t* tile_ws, hipStream_t s,
                          int64_t* total = nullptr) {
    if (n == 0) return fill_i64(out, 1, 0, s);
    if (n <= kScanOne) {
        VCT_LAUNCH("k_scan_one", k_scan_one, dim3(1), dim3(kScanOneThreads), 0, s, in, n, out, total);
        VCT_LAUNCH_CHECK();
        return VCT_OK;
    }
    const int64_t ntiles = (n + kScanTile - 1) / kScanTile;
    const bool scanned = ntiles > kScanSelf;
    VCT_LAUNCH("k_scan_tiles", k_scan_tiles, dim3((unsigned)ntiles), dim3(kScanThreads), 0, s, in, n, tile_ws);
    VCT_LAUNCH_CHECK();
    if (scanned) {
        VCT_LAUNCH("k_scan_sums", k_scan_sums, dim3(1), dim3(kScanThreads), 0, s, tile_ws, ntiles);
        VCT_LAUNCH_CHECK();
    }
    VCT_LAUNCH("k_scan_apply", k_scan_apply, dim3((unsigned)ntiles), dim3(kScanThreads), 0, s, in, n, tile_ws,
               scanned, out, total);
    VCT_LAUNCH_CHECK();
    return VCT_OK;
}

// ------------------------------------------------------------------ cell sort

// The key of every particle, and its slot in its cell (the count the atomic
// increment returns; the slots of a cell are a permutation of 0..count-1 in
// an order that varies from run to run, which the per-cell sort removes).
__global__ void k_cell_keys(int dim, int64_t n, const double* __restrict__ pos, Grid g,
                            int32_t* __restrict__ keys, int32_t* __restrict__ slots,
                            int32_t* __restrict__ counts, int32_t* __restrict__ bad) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int64_t c[3] = {0, 0, 0};
    bool finite = true;
    for (int a = 0; a < dim; ++a) {
        double v = pos[a * n + i];
        finite = finite && isfinite(v);
        c[a] = cell_coord(v, g.lo[a], g.inv_cs[a], g.nc[a]);
    }
    if (!finite) atomicAdd(bad, 1);
    int32_t k = (int32_t)cell_key(c[0], c[1], c[2], g);
    keys[i] = k;
    slots[i] = atomicAdd(&counts[k], 1);
}

__global__ void k_cell_scatter(int64_t n, const int32_t* __restrict__ keys, const int32_t* __restrict__ slots,
                               const int64_t* __restrict__ cell_start, int32_t* __restrict__ perm) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    perm[cell_start[keys[i]] + slots[i]] = (int32_t)i;
}

// The scatter leaves each cell's particles in arbitrary order; sorting every
// cell's slice by original index makes the result deterministic.  A slice of
// at most kSortReg entries is sorted in registers by a bitonic network (the
// slots past its end hold INT_MAX and stay at the end); a longer one by
// insertion in place.
constexpr int kSortReg = 64;
__global__ void k_cell_sort(int64_t ncell, const int64_t* __restrict__ cell_start,
                            int32_t* __restrict__ perm) {
    int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncell) return;
    int64_t b = cell_start[c], e = cell_start[c + 1];
    if (e - b <= kSortReg) {
        const int len = (int)(e - b);
        int v[kSortReg];
#pragma unroll
        for (int k = 0; k < kSortReg; ++k) v[k] = k < len ? perm[b + k] : INT_MAX;
#pragma unroll
        for (int size = 2; size <= kSortReg; size <<= 1)
#pragma unroll
            for (int stride = size >> 1; stride > 0; stride >>= 1)
#pragma unroll
                for (int k = 0; k < kSortReg; ++k) {
                    const int l = k ^ stride;
                    if (l > k) {
                        const bool up = (k & size) == 0;   // ascending half
                        const int lo = v[k] < v[l] ? v[k] : v[l], hi = v[k] < v[l] ? v[l] : v[k];
                        v[k] = up ? lo : hi;
                        v[l] = up ? hi : lo;
                    }
                }
#pragma unroll
        for (int k = 0; k < kSortReg; ++k)
            if (k < len) perm[b + k] = v[k];
        return;
    }
    for (int64_t i = b + 1; i < e; ++i) {
        int32_t v = perm[i];
        int64_t j = i - 1;
        while (j >= b && perm[j] > v) {
            perm[j + 1] = perm[j];
            --j;
        }
        perm[j + 1] = v;
    }
}

// Components move in groups of four whose loads are all issued before the
// first store: the scattered side then costs one memory latency per group,
// not one per component.
__global__ void k_gather(int64_t n, int ncomp, const int32_t* __restrict__ perm,
                         const double* __restrict__ src, double* __restrict__ dst) {
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    int64_t o = perm[s];
    for (int c0 = 0; c0 < ncomp; c0 += 4) {
        double v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (c0 + k < ncomp) v[k] = src[(c0 + k) * n + o];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (c0 + k < ncomp) dst[(c0 + k) * n + s] = v[k];
    }
}

__global__ void k_scatter(int64_t n, int ncomp, const int32_t* __restrict__ perm,
                          const double* __restrict__ src, double* __restrict__ dst) {
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    int64_t o = perm[s];
    for (int c0 = 0; c0 < ncomp; c0 += 4) {
        double v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (c0 + k < ncomp) v[k] = src[(c0 + k) * n + s];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (c0 + k < ncomp) dst[(c0 + k) * n + o] = v[k];
    }
}

// ------------------------------------------------------------------ chunk table

// What a search hands to the host: the entries found, whether some window is
// beyond 16-bit offsets, whether an entry had no transpose, whether a window is
// wider than the staged hit words describe, and the particles of columns
// wider than kPushWindow.
struct SearchHead {
    int64_t nnz;
    int32_t overflow, miss, wide, in_wide;
};
// After the head, kSymSlots sums of the transposed-entry map (see k_col_transpose),
// cleared with the head: together zero if the rows are symmetric.
constexpr int kSymSlots = 256;
struct SearchState {
    SearchHead head;
    unsigned long long sym[kSymSlots];
};
__device__ __forceinline__ void clear_state(SearchState* st, int64_t nnz, int64_t t) {
    if (t == 0) st->head = SearchHead{nnz, 0, 0, 0, 0};
    if (t < kSymSlots) st->sym[t] = 0ull;
}

// Chunks of one column: ceil(count / kChunk) pieces of consecutive particles.
template <int D>
__global__ void k_chunk_count(Grid g, const int64_t* __restrict__ cs, int32_t* __restrict__ nch,
                              SearchState* __restrict__ st) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    clear_state(st, 0, c);   // for the search that follows
    if (c >= grid_ncols<D>(g)) return;
    const int64_t nz = grid_nz<D>(g);
    const int64_t cnt = cs[col_key<D>(g, c, nz - 1) + 1] - cs[col_key<D>(g, c, 0)];
    nch[c] = (int32_t)((cnt + kChunk - 1) / kChunk);
}

// z cell of sorted particle p inside column c (largest z with cs[key(c, z)] <= p)
template <int D>
__device__ int64_t z_of(const Grid& g, const int64_t* __restrict__ cs, int64_t c, int64_t p) {
    int64_t lo = 0, hi = grid_nz<D>(g) - 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) / 2;
        if (cs[col_key<D>(g, c, mid)] <= p) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// One column per kFillLanes lanes, each lane every kFillLanes-th chunk of it: a
// 2-D set has few columns of many chunks (1,048,576 particles: 683 columns of
// 25 chunks, each chunk two bisections over the column's cells: 86 us with one
// thread per column, 9 us now; 3-D columns of 5 chunks fill a third of the lanes
// and take what they took, 10 us).  The same lanes add up the columns around,
// for the particles of wide columns.
constexpr int kFillLanes = 16;
template <int D>
__global__ void k_chunk_fill(Grid g, int64_t n, const int64_t* __restrict__ cs, const int64_t* __restrict__ off,
                             int32_t* __restrict__ cstart, int4* __restrict__ cinfo, SearchHead* __restrict__ head) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t c = t / kFillLanes;
    const int lane = (int)(t % kFillLanes);
    const int64_t ncols = grid_ncols<D>(g);
    if (c >= ncols) {
        if (c == ncols && lane == 0) cstart[off[ncols]] = (int32_t)n;
        return;
    }
    const int64_t nz = grid_nz<D>(g);
    const int64_t a = cs[col_key<D>(g, c, 0)], e = cs[col_key<D>(g, c, nz - 1) + 1];
    static_assert(kFillLanes >= kMaxRanges, "a lane per column around");
    {
        const int64_t ny = D == 3 ? g.nc[1] : 1;
        const int64_t x = c / ny + (D == 3 ? lane / 3 : lane) - 1, y = c % ny + (D == 3 ? lane % 3 - 1 : 0);
        const bool in = lane < (D == 3 ? 9 : 3) && x >= 0 && x < g.nc[0] && y >= 0 && y < ny;
        const int64_t q = x * ny + y;
        int win = in ? (int)(cs[col_key<D>(g, q, nz - 1) + 1] - cs[col_key<D>(g, q, 0)]) : 0;
#pragma unroll
        for (int m = kFillLanes / 2; m >= 1; m >>= 1) win += __shfl_xor(win, m, kWave);
        if (lane == 0 && win > kPushWindow && e > a) atomicAdd(&head->in_wide, (int)(e - a));
    }
    int64_t b = off[c] + lane;
    for (int64_t p = a + (int64_t)lane * kChunk; p < e; p += (int64_t)kFillLanes * kChunk, b += kFillLanes) {
        const int64_t q = (p + kChunk < e ? p + kChunk : e) - 1;
        cstart[b] = (int32_t)p;
        cinfo[b] = make_int4((int)c, (int)z_of<D>(g, cs, c, p), (int)z_of<D>(g, cs, c, q), 0);
    }
}

// ------------------------------------------------------------------ neighbours

// The neighbour test of Eq. SPH_neighbor_set: d2 summed left to right in FP64
// with no fused multiply-add (so the sets are reproducible bit for bit).
__device__ __forceinline__ bool within_exact(double dx, double dy, double dz, double R2) {
#pragma clang fp contract(off)
    double d2 = dx * dx;
    d2 = d2 + dy * dy;
    d2 = d2 + dz * dz;
    return d2 < R2;
}

constexpr int kNbWaves = 4;                    // waves per work-group
constexpr int kNbThreads = kNbWaves * kWave;   // one chunk per work-group
constexpr int kNbSeg = 1536;                   // window records per LDS segment (24 KB)
constexpr int kNbBlock = 128;                  // candidates of a matrix block: four words
constexpr int kNbRep = 2;                      // records a thread stages at a time
constexpr float kNbFar = 3e38f;                // |q|^2 of a record that is nobody's neighbour
constexpr int kNbStride = kNbSeg + 16;         // floats between the components (16 mod 64 banks)
constexpr int kNbWords = kNbSeg / 32;          // 32-candidate words per segment
constexpr int kStage = 128;                    // 16-bit staging slots per particle in the workspace
constexpr int kBmWords = kStage / 2;           // hit words per particle slot: windows up to 2048 candidates

// One chunk per work-group, a wave for 16 of its particles.  The window is staged
// in LDS segment by segment as FP32 offsets from the chunk's middle particle in
// units of R, and the squared distances come from the matrix cores: with
// m = -2 f and c = |f|^2 - lim for a particle at offset f,
//     d2 - lim = q_x m_x + q_y m_y + q_z m_z + |q|^2 * 1 + c
// is one 16 x 16 x 4 product of 16 records (x, y, z, |q|^2) and 16 columns
// (m_x, m_y, m_z, 1) on top of c.  A candidate whose FP32 value is inside or
// outside by more than a bound on its rounding error is decided by its sign; the
// few near the support edge are re-tested with the exact FP64 predicate on the
// stored positions.  Hits are collected as one bit per candidate (32-candidate
// words).  The records of a block of 128 candidates are stored so that row i of
// product u holds candidate 32 (i / 4) + 4 u + i % 4: the four results of a
// lane, over the block's eight products, are then the 32 bits of one word, and
// no lane needs another's.
//
// What bounds it: the vector instructions (61% of the busy time at 8,388,608
// particles with five waves on a SIMD; the matrix cores 29%), then the waits of
// the staging.  A candidate costs a lane one shift and half a minimum, next to
// six operations and a 16-byte LDS read per candidate when the lanes test one
// candidate each; two records of a thread staged at a time keep the registers at
// six work-groups per CU (six at a time: 125 registers, 2.1 ms).  8,388,608
// particles: 2.48 -> 2.01 ms; 1,049,800 in 3-D 0.318 -> 0.257; cubic spline,
// 2,097,152: 0.474 -> 0.355; 2-D, 1,048,576: 0.129 -> 0.092.
// MODE 0 writes the counts.  MODE 1 writes the columns at row_ptr (sorted
// indices and/or 16-bit window offsets): the words go to LDS ([word][particle])
// and a per-particle prefix over the waves' hit counts places every wave's
// hits, in ascending window order, in the particle's row.  MODE 2 writes the
// counts and the chunk's hit words, [word][particle] with the chunk's np
// particles per word, at word p0 * kBmWords of `col16` (the staging buffer),
// for k_nb_expand to turn into rows; a window wider than kBmWords * 32
// candidates does not fit there: its chunk is counted only, and head->wide
// tells the host to run the fill pass.  head->overflow flags windows beyond 65535.
template <int D, int MODE>
__global__ __launch_bounds__(kNbThreads, 6) void k_nb_chunk(int64_t n, const double* __restrict__ pos, Grid g,
                                                            double R2, double sc, const int64_t* __restrict__ cs,
                                                            const int32_t* __restrict__ cstart,
                                                            const int4* __restrict__ cinfo,
                                                            const int64_t* __restrict__ nchunks,
                                                            int32_t* __restrict__ counts,
                                                            const int64_t* __restrict__ row_ptr,
                                                            int32_t* __restrict__ col, uint16_t* __restrict__ col16,
                                                            SearchHead* __restrict__ head,
                                                            int32_t* __restrict__ win_tab) {
    constexpr bool FILL = MODE == 1, STAGE = MODE == 2;
    static_assert(kChunk == kWave && kChunk == 16 * kNbWaves, "16 particles to a wave");
    static_assert(kNbSeg % kNbBlock == 0, "segments hold whole blocks");
    __shared__ float win[4][kNbStride];
    __shared__ uint32_t bm[FILL ? kNbWords : 1][kChunk];
    __shared__ int32_t wcnt[kNbWaves][kChunk];
    __shared__ float wmax[kNbWaves];
    __shared__ WindowT<D> w;
    uint32_t b;
    if (!chunk_of_block(nchunks, b)) return;   // uniform over the work-group
    const int64_t p0 = cstart[b], p1 = cstart[b + 1];
    const int np = (int)(p1 - p0);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), pl = threadIdx.x % kWave;
    if (wv == 0) chunk_window_wave<D>(g, cs, cinfo[b], w);
    // the lane's column of the products: one of the wave's 16 particles, and
    // the component (of records and columns) or word (of results) it holds
    const int cpl = 16 * wv + pl % 16, quad = pl / 16;
    const int64_t i = p0 + cpl;
    const bool valid = cpl < np;
    const int64_t ii = valid ? i : p0;
    // the chunk origin: its middle particle, which keeps the offsets (and the
    // rounding of the expanded distance) small
    const int64_t pm = p0 + (np - 1) / 2;
    const double o0 = pos[pm], o1 = pos[n + pm], o2 = (D == 3) ? pos[2 * n + pm] : 0.0;
    const double xi0 = pos[ii], xi1 = pos[n + ii], xi2 = (D == 3) ? pos[2 * n + ii] : 0.0;
    // offsets from the chunk origin in FP32 (the same rounding as the records)
    const float f0 = (float)((xi0 - o0) * sc), f1 = (float)((xi1 - o1) * sc), f2 = (float)((xi2 - o2) * sc);
    const float ff = fmaf(f2, f2, fmaf(f1, f1, f0 * f0));
    const float colv = quad == 0 ? -2.0f * f0 : quad == 1 ? -2.0f * f1 : quad == 2 ? -2.0f * f2 : 1.0f;   // exact
    // MODE 1, lane = particle: the row to fill
    const int64_t rlo = FILL ? row_ptr[p0 + (pl < np ? pl : 0)] : 0;
    const int64_t rlen = FILL ? row_ptr[p0 + (pl < np ? pl : 0) + 1] - rlo : 0;
    __syncthreads();
    const int W = w.off[w.nr];
    if ((FILL || STAGE) && threadIdx.x == 0 && W > 65535) atomicOr(&head->overflow, 1);
    if (win_tab && wv == 0) window_store<D>(w, win_tab, b);   // for the later calls
    // the chunk's and the particle's own window offsets (it is never its own
    // neighbour; the chunk is a run of one range: lane r looks for its start in range r)
    int self_t, run0;
    {
        const int64_t d = pl < w.nr ? p0 - w.gstart[pl] : -1;
        const int len = pl < w.nr ? w.off[pl + 1] - w.off[pl] : 0, at = pl < w.nr ? w.off[pl] + (int)d : 0;
        const uint64_t own = __ballot(d >= 0 && d < len);
        run0 = __builtin_amdgcn_readlane(at, __builtin_ctzll(own));
        self_t = run0 + cpl;
    }
    // the chunk's hit words (MODE 2), np per word; only when they fit its
    // share of the staging buffer (np * kBmWords words)
    const bool words = STAGE && W <= kBmWords * 32;   // uniform
    if (STAGE && !words && threadIdx.x == 0) atomicOr(&head->wide, 1);
    uint32_t* bmg = STAGE ? reinterpret_cast<uint32_t*>(col16) + p0 * kBmWords : nullptr;
    int rowpos = 0;                     // entries of the row found so far (MODE 1)
    int mycnt = 0;                      // hits of this lane's words (MODES 0, 2)
    for (int s0 = 0; s0 < W; s0 += kNbSeg) {
        const int sW = W - s0 < kNbSeg ? W - s0 : kNbSeg;
        const int nb = (sW + kNbBlock - 1) / kNbBlock;
        if (s0 > 0) __syncthreads();   // the previous segment is consumed
        // stage the segment, kNbRep records of a thread at a time (their loads
        // before the first LDS store); the last block is filled up with records
        // far outside
        {
            float mo = 0.0f;   // largest |q|^2
            for (int t0 = 0; t0 < nb * kNbBlock; t0 += kNbRep * kNbThreads) {   // uniform
                double px[kNbRep], py[kNbRep], pz[kNbRep];
#pragma unroll
                for (int k = 0; k < kNbRep; ++k) {
                    const int t = t0 + threadIdx.x + k * kNbThreads;
                    const int64_t j = window_global<D>(w, s0 + (t < sW ? t : 0));
                    px[k] = pos[j];
                    py[k] = pos[n + j];
                    pz[k] = D == 3 ? pos[2 * n + j] : 0.0;
                }
#pragma unroll
                for (int k = 0; k < kNbRep; ++k) {
                    const int t = t0 + threadIdx.x + k * kNbThreads;
                    if (t >= nb * kNbBlock) continue;
                    float q0 = (float)((px[k] - o0) * sc), q1 = (float)((py[k] - o1) * sc);
                    float q2 = D == 3 ? (float)((pz[k] - o2) * sc) : 0.0f;
                    float qq = fmaf(q2, q2, fmaf(q1, q1, q0 * q0));
                    mo = fmaxf(mo, qq);   // (the filling repeats a record of the window)
                    if (t >= sW) qq = kNbFar;
                    if (__any(qq != qq)) {   // rare: a position that is not a number is no neighbour
                        if (qq != qq) {
                            q0 = q1 = q2 = 0.0f;
                            qq = kNbFar;
                        }
                    }
                    const int at = (t & ~(kNbBlock - 1)) + ((t >> 2) & 7) * 16 + ((t >> 5) & 3) * 4 + (t & 3);
                    win[0][at] = q0;
                    win[1][at] = q1;
                    win[2][at] = q2;
                    win[3][at] = qq;
                }
            }
#pragma unroll
            for (int m = kWave / 2; m >= 1; m >>= 1) mo = fmaxf(mo, __shfl_xor(mo, m, kWave));
            if (pl == 0) wmax[wv] = mo;
        }
        __syncthreads();
        // Absolute bound on the error of t against the exact d2 - lim in units
        // of R, with u = 2^-24, Q the largest |q|^2 of the segment, F = |f|^2
        // and T = 2 (Q + F) >= (|q| + |f|)^2: the rounded offsets (at most u |q|
        // and u |f| off), 2 u T; the roundings of |q|^2 and |f|^2, 3 u Q and 3 u F; of |f|^2 - lim, u (F + 1), and of lim, u; the four
        // products and sums of the matrix core, each partial result below
        // T + 1 and taken as truncated (2 u), 8 u (T + 1) and 2 u T.
        // 20 u T + 16 u covers the sum.
        const float seg = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
        const float T = 2.0f * (seg + ff);
        const bool odd = valid && !(T < 1e30f);   // offsets beyond FP32, or not a number: the exact predicate decides all
        const double margin = (20.0 * (double)T + 16.0) * 0x1p-24;
        const float in_lim = (float)(1.0 - margin), out_lim = (float)(1.0 + margin);
        const float cf = valid ? ff - in_lim : kNbFar;   // (an idle column has no hits)
        // t = d2 - in_lim: t < 0 is a certain hit, 0 <= t <= band is the
        // uncertain band (as unsigned integers, exactly the non-negative t up
        // to band: a negative t has its sign bit set), t > band certainly
        // lies outside.  band = out_lim - in_lim, rounded up if the FP32
        // difference is inexact.
        const double band_d = (double)out_lim - (double)in_lim;   // exact in FP64
        float band = (float)band_d;
        if ((double)band < band_d) band = nextafterf(band, INFINITY);
        const uint32_t band_u = __float_as_uint(band);
        using f4 = float __attribute__((ext_vector_type(4)));
        const f4 c4 = {cf, cf, cf, cf};
        const int nblk = 16 * wv < np ? nb : 0;   // uniform: a wave without particles has nothing to test
        for (int blk = 0; blk < nblk; ++blk) {
            const float* ap = &win[quad][blk * kNbBlock + pl % 16];
            float rec[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) rec[u] = ap[16 * u];
            // Hits shift in as the sign bits of t (the first candidate ends in
            // bit 31, reversed below); the smallest t as an unsigned integer
            // tells whether any candidate of the word lies in the band.
            uint32_t bits = 0u, low = 0xffffffffu;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const f4 t = __builtin_amdgcn_mfma_f32_16x16x4f32(rec[u], colv, c4, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const uint32_t tu = __float_as_uint(t[v]);
                    bits = __builtin_amdgcn_alignbit(bits, tu, 31);
                    low = low < tu ? low : tu;
                }
            }
            bits = __builtin_bitreverse32(bits);
            // drop the particle itself (its run's blocks alone)
            const int tb = s0 + blk * kNbBlock + 32 * quad;   // the lane's word
            const int me = self_t - tb;
            if (run0 < s0 + (blk + 1) * kNbBlock && run0 + np > s0 + blk * kNbBlock)   // uniform
                bits &= ~((unsigned)me < 32u ? 1u << me : 0u);
            if (__ballot(low <= band_u || odd)) {   // uniform; rare
                const int left = s0 + sW - tb;
                uint32_t keep = left >= 32 ? 0xffffffffu : left > 0 ? (1u << left) - 1u : 0u;
                if ((unsigned)me < 32u) keep &= ~(1u << me);
                // the words' candidates in the band, from the same products
                // (the empty asm keeps the compiler from carrying the t of the
                // loop above over to here), then the exact FP64 predicate
                float col2 = colv;
                asm volatile("" : "+v"(col2));
                uint32_t amb = 0u;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const f4 t = __builtin_amdgcn_mfma_f32_16x16x4f32(rec[u], col2, c4, 0, 0, 0);
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (__float_as_uint(t[v]) <= band_u) amb |= 1u << (4 * u + v);
                }
                if (odd) {
                    amb = 0xffffffffu;
                    bits = 0u;
                }
                amb &= keep;
                while (amb) {
                    const int u = __builtin_ctz(amb);
                    amb &= amb - 1u;
                    const int64_t j = window_global<D>(w, tb + u);
                    if (within_exact(pos[j] - xi0, pos[n + j] - xi1, D == 3 ? pos[2 * n + j] - xi2 : 0.0, R2))
                        bits |= 1u << u;
                }
            }
            if constexpr (FILL) {
                bm[blk * 4 + quad][cpl] = bits;
            } else {
                if (words && valid && tb < W)
                    bmg[dcheck((tb / 32) * np + cpl, np * kBmWords, kChkCapacity)] = bits;
                mycnt += __popc(bits);
            }
        }
        // MODES 0 and 2 sum the counts once, after the last segment
        if constexpr (FILL) {
            // lane = particle, a quarter of the words to each wave
            __syncthreads();
            const int nw = (sW + 31) / 32;
            const int k0 = wv * nw / kNbWaves, k1 = (wv + 1) * nw / kNbWaves;
            int cnt = 0;
            for (int k = k0; k < k1; ++k) cnt += __popc(bm[k][pl]);
            wcnt[wv][pl] = cnt;
            __syncthreads();
            // place this wave's hits after those of the earlier waves
            int pos0 = rowpos, total = 0;
#pragma unroll
            for (int v = 0; v < kNbWaves; ++v) {
                const int c = wcnt[v][pl];
                if (v < wv) pos0 += c;
                total += c;
            }
            if (pl < np) {
                int at = pos0;
                for (int k = k0; k < k1; ++k) {
                    uint32_t bits = bm[k][pl];
                    while (bits) {
                        const int t = s0 + 32 * k + __builtin_ctz(bits);
                        bits &= bits - 1u;
                        if (at < rlen) {
                            if (col) col[rlo + at] = (int32_t)window_global<D>(w, t);
                            if (col16) col16[rlo + at] = (uint16_t)t;
                        }
                        ++at;
                    }
                }
            }
            rowpos += total;
        }
    }
    if constexpr (!FILL) {
        wcnt[quad][cpl] = mycnt;
        __syncthreads();
        if (wv == 0 && pl < np) {
            int c = 0;
#pragma unroll
            for (int v = 0; v < kNbWaves; ++v) c += wcnt[v][pl];
            counts[p0 + pl] = c;
        }
    }
}

// Turn every chunk's hit words (written by k_nb_chunk in MODE 2) into its
// rows behind row_ptr: 16-bit window offsets, and sorted indices through the
// chunk window when col is wanted.  The words are [word][particle], np
// particles per word.  Lane = particle, and the eight waves take an eighth of
// the words each: every non-empty (word, particle) gets its first output
// position (the row's start, the earlier waves' share of the row, the hits
// before the word) and goes into a list ordered by its number of hits (a
// counting sort in LDS).  Taken in that order, the lanes of a wave expand
// words with about the same number of hits, so the loop over a word's bits
// does not wait for the fullest word of 64.  The positions are fixed before
// the expansion, so its order does not matter.  A list entry is 4 bytes (the
// particle, the word and the hits of the row before it; the word's bits are
// read again from the L2), which keeps the LDS at four work-groups per CU.
// The entries go to the chunk's block in LDS, which the work-group stores
// with unit stride; a chunk whose block exceeds the LDS buffer writes its
// entries to memory directly.
constexpr int kExT = 512;                     // threads of k_nb_expand
constexpr int kExOut = 8192;                  // entries of a chunk's block in LDS (16 KB)
constexpr int kExList = kBmWords * kChunk;    // every (word, particle) of a chunk can be listed (16 KB)
template <int D>
__global__ __launch_bounds__(kExT) void k_nb_expand(Grid g, const int64_t* __restrict__ cs,
                                                    const int32_t* __restrict__ cstart,
                                                    const int4* __restrict__ cinfo,
                                                    const int64_t* __restrict__ nchunks,
                                                    const int64_t* __restrict__ row_ptr,
                                                    const uint32_t* __restrict__ words,
                                                    const int32_t* __restrict__ win_tab,
                                                    int32_t* __restrict__ col, uint16_t* __restrict__ col16,
                                                    uint16_t* __restrict__ range_pos) {
    constexpr int kWaves = kExT / kWave;
    constexpr int kPer = kBmWords / kWaves;   // words of one wave's share
    static_assert(kBmWords % kWaves == 0 && kChunk == kWave, "shares of whole words, lane = particle");
    __shared__ WindowT<D> w;
    __shared__ int64_t rp[kChunk + 1];
    __shared__ int32_t part[kWaves][kChunk];      // each wave's share of every row
    __shared__ uint32_t bucket[33];               // words per hit count (32 - count), then offsets
    __shared__ uint32_t list[kExList];            // particle | word << 6 | hits of the row before it << 12
    __shared__ __align__(16) uint16_t sout[kExOut];
    uint32_t b;
    if (!chunk_of_block(nchunks, b)) return;   // uniform over the work-group
    const int64_t p0 = cstart[b];
    const int np = (int)(cstart[b + 1] - p0);
    const int wv = threadIdx.x / kWave, pl = threadIdx.x % kWave;
    const uint32_t* src = words + p0 * kBmWords;
    const int k0 = wv * kPer;
    const bool lane_on = pl < np;
    // this wave's share of the words, requested with the window and the row
    // pointers: all kBmWords words of the chunk's share of the buffer (np x
    // kBmWords), those past the window (not written by the search) masked
    // once the window is known
    uint32_t v[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) v[u] = lane_on ? src[(k0 + u) * np + pl] : 0u;
    if (wv == 0) {
        if (win_tab) window_load<D>(win_tab, b, w);
        else chunk_window_wave<D>(g, cs, cinfo[b], w);
    }
    if (threadIdx.x <= (unsigned)np) rp[threadIdx.x] = row_ptr[p0 + threadIdx.x];
    if (threadIdx.x < 33) bucket[threadIdx.x] = 0u;
    __syncthreads();
    // at most kBmWords words: the search flags wider windows, and the host
    // then runs the fill pass instead
    const int nw = dcheck((w.off[w.nr] + 31) / 32, kBmWords + 1, kChkCapacity);
    const int64_t e0 = rp[0], e1 = rp[np];
    int before[kPer];   // hits of the row in this wave's share before each word
    {
#pragma unroll
        for (int u = 0; u < kPer; ++u) v[u] = k0 + u < nw ? v[u] : 0u;
        int c = 0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            before[u] = c;
            c += __popc(v[u]);
        }
        part[wv][pl] = c;
    }
    __syncthreads();
    int start = 0;   // hits of the row in the earlier waves' shares
    for (int x = 0; x < wv; ++x) start += part[x][pl];
    if (range_pos) {
        // where each range of the window begins in the row (read by the
        // transposed-entry map), by the wave that holds the range's first word
        for (int r = 1; r < w.nr; ++r) {
            const int o = __builtin_amdgcn_readfirstlane(w.off[r]);
            const int u0 = (o >> 5) - k0;
            if (u0 < 0 || u0 > kPer || (u0 == kPer && wv < kWaves - 1)) continue;   // uniform over the wave
            int at = start + before[kPer - 1] + __popc(v[kPer - 1]);   // past this share: its end
#pragma unroll
            for (int u = 0; u < kPer; ++u)
                if (u == u0) at = start + before[u] + __popc(v[u] & ((1u << (o & 31)) - 1u));
            sout[(kMaxRanges - 1) * pl + r - 1] = (uint16_t)at;
        }
    }
    uint32_t slot[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) slot[u] = v[u] ? atomicAdd(&bucket[32 - __popc(v[u])], 1u) : 0u;
    __syncthreads();
    if (range_pos && (int)threadIdx.x < np)
        reinterpret_cast<uint4*>(range_pos)[p0 + threadIdx.x] = reinterpret_cast<const uint4*>(sout)[threadIdx.x];
    if (wv == 0) {   // exclusive prefix of the 32 bucket sizes; bucket[32] = the total
        const uint32_t t = pl < 32 ? bucket[pl] : 0u;
        uint32_t incl = t;
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
            const uint32_t o = __shfl_up(incl, m, kWave);
            if (pl >= m) incl += o;
        }
        if (pl <= 32) bucket[pl] = incl - t;
    }
    __syncthreads();
    const int nlist = (int)bucket[32];   // the non-empty words (words without hits are not listed)
#pragma unroll
    for (int u = 0; u < kPer; ++u)
        if (v[u])
            list[dcheck((int)(bucket[32 - __popc(v[u])] + slot[u]), kExList, kChkCapacity)] =
                (uint32_t)pl | ((uint32_t)(k0 + u) << 6) | ((uint32_t)(start + before[u]) << 12);
    __syncthreads();
    const bool in_lds = e1 - e0 <= kExOut;
    auto expand = [&](uint32_t bits, int at, int wd) {
        while (bits) {
            const uint16_t t = (uint16_t)(32 * wd + __builtin_ctz(bits));
            bits &= bits - 1u;
            if (in_lds) {
                sout[dcheck(at, kExOut, kChkCapacity)] = t;
            } else {
                if (col16) col16[e0 + at] = t;
                if (col) col[e0 + at] = (int32_t)window_global<D>(w, t);
            }
            ++at;
        }
    };
    for (int li = threadIdx.x; li < nlist; li += kExT) {
        const uint32_t ent = list[li];
        const int q = (int)(ent & 63u), wd = (int)((ent >> 6) & 63u);
        expand(src[wd * np + q], (int)(rp[q] - e0) + (int)(ent >> 12), wd);
    }
    if (!in_lds) return;   // uniform over the work-group
    __syncthreads();
    for (int e = threadIdx.x; e < (int)(e1 - e0); e += kExT) {
        const uint16_t t = sout[e];
        if (col16) col16[e0 + e] = t;
        if (col) col[e0 + e] = (int32_t)window_global<D>(w, t);
    }
}

VCT_CHECKS_TU(checks_cells)

}  // namespace vct

using namespace vct;

// ====================================================================== C ABI

extern "C" int64_t vct_grid_dims(int dim, const double* lo, const double* hi, double R, int64_t* dims) {
    if ((dim != 2 && dim != 3) || !lo || !hi || !(R > 0.0) || !isfinite(R)) return VCT_E_ARG;
    Grid g;
    int64_t total = grid_setup(dim, lo, hi, R, g);
    if (total < 0) return total;
    if (dims) for (int a = 0; a < 3; ++a) dims[a] = g.nc[a];
    return total;
}

extern "C" size_t vct_build_cells_workspace_size(int dim, int64_t n, int64_t ncell) {
    (void)dim;
    if (n < 0 || ncell < 1) return 0;
    return aligned_sum({(size_t)n * 4, (size_t)n * 4, (size_t)ncell * 4, scan_ws_bytes(ncell), 64});
}

extern "C" int vct_build_cells(int dim, int64_t n, const double* pos, const double* lo, const double* hi,
                               double R, int32_t* perm, double* pos_sorted, int64_t* cell_start,
                               int64_t ncell, void* ws, size_t ws_bytes, void* stream) {
    VCT_API_RANGE("vct_build_cells");
    if ((dim != 2 && dim != 3) || n < 0 || n > INT32_MAX || !lo || !hi || !(R > 0.0) || !isfinite(R))
        return VCT_E_ARG;
    Grid g;
    int64_t total = grid_setup(dim, lo, hi, R, g);
    if (total < 0) return (int)total;
    if (ncell != total || !cell_start) return VCT_E_ARG;
    if (n > 0 && (!pos || !perm || !pos_sorted)) return VCT_E_ARG;
    if (!ws || ws_bytes < vct_build_cells_workspace_size(dim, n, ncell)) return VCT_E_WORKSPACE;
    hipStream_t s = as_stream(stream);
    Carver cv(ws, ws_bytes);
    int32_t* keys = cv.take<int32_t>((size_t)n);
    int32_t* slots = cv.take<int32_t>((size_t)n);
    int32_t* counts = cv.take<int32_t>((size_t)ncell);
    int64_t* tiles = cv.take<int64_t>(scan_ws_bytes(ncell) / 8);
    int32_t* bad = cv.take<int32_t>(16);
    int st;
    if ((st = zero_i32(counts, ncell, bad, 1, s))) return st;
    if (n > 0) {
        VCT_LAUNCH("k_cell_keys", k_cell_keys, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, dim, n, pos, g,
                   keys, slots, counts, bad);
        VCT_LAUNCH_CHECK();
    }
    if ((st = exclusive_scan(counts, ncell, cell_start, tiles, s))) return st;
    if (n > 0) {
        VCT_LAUNCH("k_cell_scatter", k_cell_scatter, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, keys,
                   slots, cell_start, perm);
        VCT_LAUNCH_CHECK();
        VCT_LAUNCH("k_cell_sort", k_cell_sort, dim3((unsigned)((ncell + 255) / 256)), dim3(256), 0, s, ncell,
                   cell_start, perm);
        VCT_LAUNCH_CHECK();
        VCT_LAUNCH("k_gather", k_gather, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, dim, perm, pos,
                   pos_sorted);
        VCT_LAUNCH_CHECK();
    }
    int32_t hbad = 0;
    VCT_HIP_CHECK(hipMemcpyAsync(&hbad, bad, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    VCT_HIP_CHECK(hipStreamSynchronize(s));
    return hbad ? VCT_E_NONFINITE : VCT_OK;
}

extern "C" int vct_gather_sorted(int64_t n, int ncomp, const int32_t* perm, const double* src, double* dst,
                                 void* stream) {
    VCT_API_RANGE("vct_gather_sorted");
    if (n < 0 || ncomp < 1 || n > INT32_MAX) return VCT_E_ARG;
    if (n == 0) return VCT_OK;
    if (!perm || !src || !dst || src == dst) return VCT_E_ARG;
    VCT_LAUNCH("k_gather", k_gather, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, as_stream(stream), n, ncomp,
               perm, src, dst);
    VCT_LAUNCH_CHECK();
    return VCT_OK;
}

extern "C" int vct_scatter_sorted(int64_t n, int ncomp, const int32_t* perm, const double* src, double* dst,
                                  void* stream) {
    VCT_API_RANGE("vct_scatter_sorted");
    if (n < 0 || ncomp < 1 || n > INT32_MAX) return VCT_E_ARG;
    if (n == 0) return VCT_OK;
    if (!perm || !src || !dst || src == dst) return VCT_E_ARG;
    VCT_LAUNCH("k_scatter", k_scatter, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, as_stream(stream), n, ncomp,
               perm, src, dst);
    VCT_LAUNCH_CHECK();
    return VCT_OK;
}

extern "C" int64_t vct_chunk_capacity(int dim, int64_t n, int64_t ncell) {
    if ((dim != 2 && dim != 3) || n < 0 || ncell < 1) return 0;
    return n / kChunk + ncell + 1;
}

// Workspace without the staging buffer (enough for the two-pass search).
static size_t nb_ws_base(int64_t n, int64_t ncell) {
    const int64_t m = n > ncell ? n : ncell;
    return aligned_sum({(size_t)m * 4, scan_ws_bytes(m), sizeof(SearchState)});
}

extern "C" size_t vct_neighbors_workspace_size(int64_t n, int64_t ncell) {
    if (n < 0 || ncell < 1) return 0;
    return aligned_sum({nb_ws_base(n, ncell), (size_t)(n > 0 ? n : 1) * kStage * sizeof(uint16_t),
                        (size_t)(n > 0 ? n : 1) * (kMaxRanges - 1) * sizeof(uint16_t)});
}

namespace vct {
// Transposed-entry map: for entry e = (i, j) of row i, the position of (j, i)
// in row j.  The neighbour relation is symmetric (d2 is formed from x_j - x_i,
// whose negation is exact), and a chunk's particles are consecutive sorted
// indices, so the entries of row j that lie in one chunk are consecutive too:
// those of the chunk's particles that have j in their rows, in order.  One
// work-group per chunk therefore marks, in LDS, which of its particles have
// each window candidate (one bit per particle), finds where row j reaches the
// chunk once per candidate, and an entry's transposed position is that plus
// the number of marked particles before its own.  The expansion of the hit
// words leaves where each column's part of every row begins (range_pos, 8
// positions per row); the chunk's entries are then nearly always the first or
// the last of the part in its column, which one read confirms, and a binary
// search finds the others (and all of them where the rows came from the fill
// pass, which leaves no range_pos).
// Bound by the scattered reads of those confirmations and by the map's stores:
// with a binary search per candidate, nine reads instead of one or two, 0.80
// ms, and one search per entry, each lane searching 16 at a time, 2.66 ms, for
// 1,049,800 particles in 3-D (104M entries); now 0.52 ms (0.48 without the check below).  2-D, 1,048,576
// particles: 0.43 -> 0.12 ms.  Windows beyond kTWin candidates are taken in
// parts.
// Those reads confirm the first entry of every run; that each of the others has
// its transpose too is confirmed over the whole set: the sum of
// a(i) b(j) - b(i) a(j) over the entries (i, j), a and b two hash values of 32
// bits (multipliers from the golden ratio and the roots of 2 and 3), in 64-bit
// integers is zero if every entry has its transpose, and with an entry that has
// none it is zero by a chance of about 2^-32.  (Reading every entry of the runs
// as well takes 0.35 ms more.)
struct SymPair {
    uint64_t a, b;
};
__device__ __forceinline__ SymPair sym_pair(int32_t j) {
    uint32_t x = (uint32_t)j * 0x9e3779b9u;
    x ^= x >> 15;
    x *= 0x6a09e667u;
    const uint32_t y = (x ^ x >> 12) * 0xbb67ae85u;
    return {x, y ^ y >> 15};
}
constexpr int kTThreads = 512;
constexpr int kTWin = 1536;   // candidates per part (18 KB of LDS)
template <int D, bool OFFS>
__global__ __launch_bounds__(kTThreads) void k_col_transpose(Grid g, const int64_t* __restrict__ cs,
                                                             const int32_t* __restrict__ cstart,
                                                             const int4* __restrict__ cinfo,
                                                             const int64_t* __restrict__ nchunks,
                                                             const int32_t* __restrict__ win_tab,
                                                             const int64_t* __restrict__ row_ptr,
                                                             const int32_t* __restrict__ col,
                                                             const uint16_t* __restrict__ col16,
                                                             const uint16_t* __restrict__ range_pos,
                                                             int32_t* __restrict__ col_t, SearchState* __restrict__ st) {
    constexpr int kLanes = kTThreads / kChunk;   // lanes per row
    // row entries per lane held in registers: the rows of R = 3 d0 (2-D: with
    // 14 slots, mostly empty, 0.142 instead of 0.121 ms at 1,048,576 particles)
    constexpr int kTSlots = D == 2 ? 4 : 14;
    static_assert(kChunk == 64, "one mask bit per particle of the chunk");
    __shared__ uint32_t mask[2][kTWin];   // particles 0..31 and 32..63 of the chunk
    __shared__ int32_t base[kTWin];
    __shared__ WindowT<D> w;
    __shared__ int s_own[kMaxRanges], s_nr[kMaxRanges];   // per range: the chunk's column and the ranges, seen from it
    uint32_t b;
    if (!chunk_of_block(nchunks, b)) return;   // uniform over the work-group
    const int64_t p0 = cstart[b];
    const int np = (int)(cstart[b + 1] - p0);
    if (threadIdx.x < kWave) {
        if (win_tab) window_load<D>(win_tab, b, w);
        else chunk_window_wave<D>(g, cs, cinfo[b], w);
    } else if (threadIdx.x < 2 * kWave && range_pos) {
        // the columns around this one are the window's ranges; in the windows
        // of such a column this one is range s_own of s_nr
        const int ln = threadIdx.x - kWave;
        const int64_t c = cinfo[b].x, ny = D == 3 ? g.nc[1] : 1;
        const int64_t cx = c / ny, cy = c % ny;
        auto inside = [&](int64_t x, int64_t y) { return x >= 0 && x < g.nc[0] && y >= 0 && y < ny; };
        const int64_t x = cx + (D == 3 ? ln / 3 : ln) - 1, y = cy + (D == 3 ? ln % 3 - 1 : 0);
        const bool in = ln < (D == 3 ? 9 : 3) && inside(x, y);
        const uint64_t mb = (uint64_t)__ballot(in);
        if (in) {
            int own = 0, nr = 0;
            for (int k = 0; k < (D == 3 ? 9 : 3); ++k) {
                const int64_t x2 = x + (D == 3 ? k / 3 : k) - 1, y2 = y + (D == 3 ? k % 3 - 1 : 0);
                if (!inside(x2, y2)) continue;
                if (x2 == cx && y2 == cy) own = nr;
                ++nr;
            }
            const int r = __popcll(mb & ((1ull << ln) - 1ull));
            s_own[r] = own;
            s_nr[r] = nr;
        }
    }
    const int pl = threadIdx.x / kLanes, lane = threadIdx.x % kLanes;
    const int64_t rb = pl < np ? row_ptr[p0 + pl] : 0, re = pl < np ? row_ptr[p0 + pl + 1] : 0;
    __syncthreads();
    const int W = w.off[w.nr];
    // window offset of entry e: stored, or from its sorted index j, whose
    // range is the last one that starts at or before j (the ranges ascend; an
    // empty range never holds j)
    auto offset_of = [&](int64_t e) {
        if constexpr (OFFS) return (int)col16[e];
        const int32_t j = col[e];
        int r = 0;
#pragma unroll
        for (int k = 1; k < kMaxRanges; ++k)
            if (k < w.nr && (int64_t)j >= w.gstart[k] && w.off[k + 1] > w.off[k]) r = k;
        return w.off[r] + (int)((int64_t)j - w.gstart[r]);
    };
    // the first kTSlots entries of a lane stay in registers for both uses
    // (loaded together; longer rows re-read the rest)
    int tt[kTSlots];
#pragma unroll
    for (int s = 0; s < kTSlots; ++s) {
        const int64_t e = rb + lane + (int64_t)kLanes * s;
        tt[s] = e < re ? offset_of(e) : -1;
    }
    const int64_t tail = rb + lane + (int64_t)kLanes * kTSlots;
    bool bad = false;   // an entry that is not in the window, or a run that is not in its place
#pragma unroll
    for (int s = 0; s < kTSlots; ++s)
        bad = bad || (rb + lane + (int64_t)kLanes * s < re && (unsigned)tt[s] >= (unsigned)W);
    for (int64_t e = tail; e < re; e += kLanes) bad = bad || (unsigned)offset_of(e) >= (unsigned)W;
    uint64_t sa = 0, sb = 0;   // sums of a(j) and b(j) over the lane's entries
    for (int s0 = 0; s0 < W; s0 += kTWin) {
        const int sW = W - s0 < kTWin ? W - s0 : kTWin;
        for (int t = threadIdx.x; t < sW; t += kTThreads) {
            mask[0][t] = mask[1][t] = 0u;
            base[t] = (int32_t)window_global<D>(w, s0 + t);   // the candidate j, until its run is found
        }
        __syncthreads();
        auto mark = [&](int t) {
            if ((unsigned)t < (unsigned)sW) {
                atomicOr(&mask[pl >> 5][t], 1u << (pl & 31));
                const SymPair h = sym_pair(base[t]);
                sa += h.a;
                sb += h.b;
            }
        };
#pragma unroll
        for (int s = 0; s < kTSlots; ++s) mark(tt[s] - s0);
        for (int64_t e = tail; e < re; e += kLanes) mark(offset_of(e) - s0);
        __syncthreads();
        for (int t = threadIdx.x; t < sW; t += kTThreads) {
            const unsigned long long m = mask[0][t] | (unsigned long long)mask[1][t] << 32;
            if (!m) continue;
            int r = 0;
#pragma unroll
            for (int q = 1; q < kMaxRanges; ++q)
                if (q < w.nr && s0 + t >= w.off[q]) r = q;
            const int64_t j = base[t];
            int64_t lo = row_ptr[j], hi = row_ptr[j + 1];
            if (range_pos) {   // the part of row j in the chunk's column
                const int own = s_own[r];
                const uint16_t* rp = range_pos + j * (kMaxRanges - 1);
                const int64_t jb = lo;
                if (own + 1 < s_nr[r]) hi = jb + rp[own];
                if (own > 0) lo = jb + rp[own - 1];
            }
            const int cnt = __popcll(m);
            const int32_t first = (int32_t)p0 + __builtin_ctzll(m);
            // nearly always the part begins or ends in this chunk
            int64_t at = lo;
            if (at >= hi || col[at] != first) {
                at = hi - cnt;
                if (at < lo || col[at] != first) {
                    int64_t e = hi;
                    at = lo;
                    while (at < e) {
                        const int64_t mid = (at + e) / 2;
                        if (col[mid] < first) at = mid + 1;
                        else e = mid;
                    }
                    if (at >= hi || col[at] != first) at = hi;   // not there
                }
            }
            const bool ok = at + cnt <= hi;
            bad = bad || !ok;
            base[t] = ok ? (int32_t)at : -1;
        }
        __syncthreads();
        auto store = [&](int64_t e, int t) {
            if ((unsigned)t < (unsigned)sW) {
                const int32_t bt = base[t];
                const uint32_t below = (1u << (pl & 31)) - 1u;
                const int rank = pl < 32 ? __popc(mask[0][t] & below) : __popc(mask[0][t]) + __popc(mask[1][t] & below);
                col_t[e] = bt < 0 ? -1 : bt + rank;
            }
        };
#pragma unroll
        for (int s = 0; s < kTSlots; ++s) store(rb + lane + (int64_t)kLanes * s, tt[s] - s0);
        for (int64_t e = tail; e < re; e += kLanes) store(e, offset_of(e) - s0);
        __syncthreads();   // the part's masks are consumed
    }
    if (bad) atomicOr(&st->head.miss, 1);
    const SymPair hi = sym_pair((int32_t)(p0 + pl));
    unsigned long long sum = hi.a * sb - hi.b * sa;
    for (int m = 1; m < kWave; m <<= 1) sum += __shfl_xor(sum, m, kWave);
    unsigned long long* part = reinterpret_cast<unsigned long long*>(mask);
    if (threadIdx.x % kWave == 0) part[threadIdx.x / kWave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int v = 1; v < kTThreads / kWave; ++v) sum += part[v];
        atomicAdd(&st->sym[b % kSymSlots], sum);
    }
}

int nlist_check(const vct_nlist* nl, Grid& g) {
    if (!nl || (nl->dim != 2 && nl->dim != 3) || nl->n < 0 || nl->n > INT32_MAX || !(nl->R > 0.0) ||
        !isfinite(nl->R) || !nl->cell_start || !nl->row_ptr || !nl->chunk_off || !nl->chunk_start ||
        !nl->chunk_info || (reinterpret_cast<uintptr_t>(nl->col16) & 15u) != 0)
        return VCT_E_ARG;
    const int64_t total = grid_setup(nl->dim, nl->lo, nl->hi, nl->R, g);
    if (total < 0) return (int)total;
    if (total != nl->ncell || nl->chunk_cap < vct_chunk_capacity(nl->dim, nl->n, nl->ncell)) return VCT_E_ARG;
    return VCT_OK;
}
}  // namespace vct

// The workspace of a search and its rows.
struct NbWork {
    int32_t* counts;
    int64_t* tiles;
    SearchState* state;
    SearchHead* head;
    uint16_t* staged;      // hit words
    uint16_t* range_pos;   // per row: where each column's part begins
    NbWork(const vct_nlist* nl, void* p, size_t bytes) {
        const int64_t n = nl->n, m = n > nl->ncell ? n : nl->ncell;
        Carver cv(p, bytes);
        counts = cv.take<int32_t>((size_t)m);
        tiles = cv.take<int64_t>(scan_ws_bytes(m) / 8);
        state = cv.take<SearchState>(1);
        head = &state->head;
        staged = cv.take<uint16_t>((size_t)(n > 0 ? n : 1) * kStage);
        range_pos = cv.take<uint16_t>((size_t)(n > 0 ? n : 1) * (kMaxRanges - 1));
    }
};

template <int D>
static int build_chunks(const vct_nlist* nl, const Grid& g, const NbWork& ws, hipStream_t s) {
    int32_t* tmp = ws.counts;
    const int64_t ncols = D == 3 ? g.nc[0] * g.nc[1] : g.nc[0];
    VCT_LAUNCH("k_chunk_count", (k_chunk_count<D>), dim3((unsigned)((ncols + 255) / 256)), dim3(256), 0, s, g,
               nl->cell_start, tmp, ws.state);
    VCT_LAUNCH_CHECK();
    int st = exclusive_scan(tmp, ncols, nl->chunk_off, ws.tiles, s);
    if (st) return st;
    VCT_LAUNCH("k_chunk_fill", (k_chunk_fill<D>), dim3((unsigned)(((ncols + 1) * kFillLanes + 255) / 256)), dim3(256),
               0, s, g, nl->n, nl->cell_start, nl->chunk_off, nl->chunk_start, reinterpret_cast<int4*>(nl->chunk_info),
               ws.head);
    VCT_LAUNCH_CHECK();
    return VCT_OK;
}

template <int D, int MODE>
static int launch_nb(const vct_nlist* nl, const double* pos, const Grid& g, const NbWork& ws, hipStream_t s) {
    const int64_t ncols = D == 3 ? g.nc[0] * g.nc[1] : g.nc[0];
    const int64_t cap = ncols + nl->n / kChunk + 1;   // upper bound of the chunk count
    const char* name = MODE == 0 ? "k_nb_chunk (count)" : MODE == 1 ? "k_nb_chunk (fill)" : "k_nb_chunk (stage)";
    const int4* cinfo = reinterpret_cast<const int4*>(nl->chunk_info);
    const double R2 = nl->R * nl->R;
    // (the staging search is the counting one too: timed under both names)
    const LaunchTimer counted(MODE == 2 ? "k_nb_chunk (count)" : nullptr, s);
    VCT_LAUNCH(name, (k_nb_chunk<D, MODE>), dim3((unsigned)cap), dim3(kNbThreads), 0, s, nl->n, pos, g,
               R2, 1.0 / sqrt(R2), nl->cell_start, nl->chunk_start, cinfo, nl->chunk_off + ncols,
               MODE == 1 ? nullptr : ws.counts, nl->row_ptr, MODE == 1 ? nl->col : nullptr,
               MODE == 1 ? nl->col16 : ws.staged, ws.head, nl->chunk_win);
    VCT_LAUNCH_CHECK();
    return VCT_OK;
}

template <int D>
static int launch_expand(const vct_nlist* nl, const Grid& g, const NbWork& ws, hipStream_t s) {
    const int64_t ncols = D == 3 ? g.nc[0] * g.nc[1] : g.nc[0];
    const int64_t cap = ncols + nl->n / kChunk + 1;
    VCT_LAUNCH("k_nb_expand", (k_nb_expand<D>), dim3((unsigned)cap), dim3(kExT), 0, s, g, nl->cell_start,
               nl->chunk_start, reinterpret_cast<const int4*>(nl->chunk_info), nl->chunk_off + ncols,
               nl->row_ptr, reinterpret_cast<const uint32_t*>(ws.staged), nl->chunk_win, nl->col, nl->col16,
               nl->col_t ? ws.range_pos : nullptr);
    VCT_LAUNCH_CHECK();
    return VCT_OK;
}

static int nb_check(const vct_nlist* nl, const double* pos, const void* ws, size_t ws_bytes, Grid& g) {
    const int st = nlist_check(nl, g);
    if (st) return st;
    if (nl->n > 0 && !pos) return VCT_E_ARG;
    return !ws || ws_bytes < vct_neighbors_workspace_size(nl->n, nl->ncell) ? VCT_E_WORKSPACE : VCT_OK;
}

// Chunk table, counts and row pointers; with `stage` also the hit words.
template <int D>
static int nb_search(const vct_nlist* nl, const double* pos, const Grid& g, const NbWork& ws, bool stage,
                     hipStream_t s) {
    int st = build_chunks<D>(nl, g, ws, s);
    if (st) return st;
    if (nl->n > 0) {
        st = stage ? launch_nb<D, 2>(nl, pos, g, ws, s) : launch_nb<D, 0>(nl, pos, g, ws, s);
        if (st) return st;
    }
    return exclusive_scan(ws.counts, nl->n, nl->row_ptr, ws.tiles, s, &ws.head->nnz);
}

// The columns behind row_ptr (from the hit words, or by the fill pass) and the
// transposed-entry map.
template <int D>
static int nb_rows(const vct_nlist* nl, const double* pos, const Grid& g, const NbWork& ws, bool words, hipStream_t s) {
    const int64_t n = nl->n;
    if (n == 0) return VCT_OK;
    const int st = words ? launch_expand<D>(nl, g, ws, s) : launch_nb<D, 1>(nl, pos, g, ws, s);
    if (st || !nl->col_t) return st;
    const int64_t ncols = D == 3 ? g.nc[0] * g.nc[1] : g.nc[0];
    const dim3 grid((unsigned)(ncols + n / kChunk + 1));
    const int4* cinfo = reinterpret_cast<const int4*>(nl->chunk_info);
    const uint16_t* range_pos = words ? ws.range_pos : nullptr;
    if (nl->col16)
        VCT_LAUNCH("k_col_transpose", (k_col_transpose<D, true>), grid, dim3(kTThreads), 0, s, g, nl->cell_start,
                   nl->chunk_start, cinfo, nl->chunk_off + ncols, nl->chunk_win, nl->row_ptr, nl->col, nl->col16,
                   range_pos, nl->col_t, ws.state);
    else
        VCT_LAUNCH("k_col_transpose", (k_col_transpose<D, false>), grid, dim3(kTThreads), 0, s, g, nl->cell_start,
                   nl->chunk_start, cinfo, nl->chunk_off + ncols, nl->chunk_win, nl->row_ptr, nl->col, nl->col16,
                   range_pos, nl->col_t, ws.state);
    VCT_LAUNCH_CHECK();
    return VCT_OK;
}

static int read_head(const NbWork& ws, SearchHead& h, hipStream_t s) {
    VCT_HIP_CHECK(hipMemcpyAsync(&h, ws.head, sizeof(h), hipMemcpyDeviceToHost, s));
    VCT_HIP_CHECK(hipStreamSynchronize(s));
    return VCT_OK;
}

__global__ void k_head_given(SearchState* st, const int64_t* nnz) { clear_state(st, *nnz, threadIdx.x); }

// The end of a call that wrote the transposed-entry map: whether every entry
// has its transpose, and the head.
static int read_transposed(const NbWork& ws, SearchHead& h, hipStream_t s) {
    SearchState st;
    VCT_HIP_CHECK(hipMemcpyAsync(&st, ws.state, sizeof(st), hipMemcpyDeviceToHost, s));
    VCT_HIP_CHECK(hipStreamSynchronize(s));
    h = st.head;
    unsigned long long sum = 0;
    for (unsigned long long v : st.sym) sum += v;
    return h.overflow ? VCT_E_WINDOW : h.miss || sum ? VCT_E_HIP : VCT_OK;
}

extern "C" int vct_neighbors(vct_nlist* nl, const double* pos_sorted, int64_t col_cap, int64_t* nnz_out,
                             int reuse_row_ptr, void* ws_p, size_t ws_bytes, void* stream) {
    VCT_API_RANGE("vct_neighbors");
    Grid g;
    if (!nnz_out) {
        const int st = nlist_check(nl, g);
        return st ? st : VCT_E_ARG;
    }
    int st = nb_check(nl, pos_sorted, ws_p, ws_bytes, g);
    if (st) return st;
    hipStream_t s = as_stream(stream);
    const NbWork ws(nl, ws_p, ws_bytes);
    const bool want_cols = nl->col || nl->col16;
    if (reuse_row_ptr) {
        VCT_LAUNCH("k_head_given", k_head_given, dim3(1), dim3(kSymSlots), 0, s, ws.state, nl->row_ptr + nl->n);
        VCT_LAUNCH_CHECK();
    } else {
        st = nl->dim == 2 ? nb_search<2>(nl, pos_sorted, g, ws, want_cols, s)
                          : nb_search<3>(nl, pos_sorted, g, ws, want_cols, s);
        if (st) return st;
    }
    SearchHead h;
    if ((st = read_head(ws, h, s))) return st;
    *nnz_out = h.nnz;
    nl->nnz = h.nnz;
    if (!reuse_row_ptr) nl->wide_particles = 1 + h.in_wide;
    if (!want_cols) return VCT_OK;
    if (col_cap < h.nnz) return VCT_E_CAPACITY;
    if (nl->col_t && (!nl->col || h.nnz > INT32_MAX)) return VCT_E_ARG;
    if (h.overflow) return VCT_E_WINDOW;
    const bool words = !reuse_row_ptr && h.wide == 0;
    st = nl->dim == 2 ? nb_rows<2>(nl, pos_sorted, g, ws, words, s) : nb_rows<3>(nl, pos_sorted, g, ws, words, s);
    if (st) return st;
    if (nl->col_t) return read_transposed(ws, h, s);
    if ((st = read_head(ws, h, s))) return st;
    return h.overflow ? VCT_E_WINDOW : VCT_OK;
}

// what vct_neighbors_search left in the workspace
enum { kStagedFill = 0, kStagedWords = 1, kStagedOverflow = 2 };

extern "C" int vct_neighbors_search(vct_nlist* nl, const double* pos_sorted, int64_t* nnz_out, int* staged, void* ws_p,
                                    size_t ws_bytes, void* stream) {
    VCT_API_RANGE("vct_neighbors_search");
    Grid g;
    if (!nnz_out || !staged) return VCT_E_ARG;
    int st = nb_check(nl, pos_sorted, ws_p, ws_bytes, g);
    if (st) return st;
    hipStream_t s = as_stream(stream);
    const NbWork ws(nl, ws_p, ws_bytes);
    st = nl->dim == 2 ? nb_search<2>(nl, pos_sorted, g, ws, true, s) : nb_search<3>(nl, pos_sorted, g, ws, true, s);
    if (st) return st;
    SearchHead h;
    if ((st = read_head(ws, h, s))) return st;
    *nnz_out = h.nnz;
    nl->nnz = h.nnz;
    nl->wide_particles = 1 + h.in_wide;
    *staged = h.overflow ? kStagedOverflow : h.wide ? kStagedFill : kStagedWords;
    return VCT_OK;
}

extern "C" int vct_neighbors_rows(const vct_nlist* nl, const double* pos_sorted, int64_t col_cap, int staged,
                                  void* ws_p, size_t ws_bytes, void* stream) {
    VCT_API_RANGE("vct_neighbors_rows");
    Grid g;
    int st = nb_check(nl, pos_sorted, ws_p, ws_bytes, g);
    if (st) return st;
    if (staged < kStagedFill || staged > kStagedOverflow || (!nl->col && !nl->col16) || nl->nnz < 0) return VCT_E_ARG;
    if (col_cap < nl->nnz) return VCT_E_CAPACITY;
    if (nl->col_t && (!nl->col || nl->nnz > INT32_MAX)) return VCT_E_ARG;
    if (staged == kStagedOverflow) return VCT_E_WINDOW;
    hipStream_t s = as_stream(stream);
    const NbWork ws(nl, ws_p, ws_bytes);
    const bool words = staged == kStagedWords;
    st = nl->dim == 2 ? nb_rows<2>(nl, pos_sorted, g, ws, words, s) : nb_rows<3>(nl, pos_sorted, g, ws, words, s);
    if (st || !nl->col_t) return st;
    SearchHead h;
    return read_transposed(ws, h, s);
}
