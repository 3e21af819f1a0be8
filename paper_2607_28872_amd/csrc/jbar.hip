// Volume smoothing of the sigma method: the smoothed Jacobian determinant
// Jbar^N of paper Sec. 3.6 (Eq. VCT_bar_a).
//
// With v_i = J_i / Jbar_i (particle i's representative volume in units of V),
// the update of one neighbour pair (i, j) in Eq. VCT_bar_a is a volume
// exchange:
//   c_ij = C_V (r_e - |r^_ij|) / r_e,   dv = c_ij (v_j - v_i),
//   v_i <- v_i + dv,   v_j <- v_j - dv,
// applied along the neighbours j of a target particle i one after the other,
// every exchange seen by the next, and then for the next target.  Every
// particle is a target once; the paper leaves the order of the targets open.
//
// Schedule.  The targets are taken cell by cell in 3^d phases: the cell
// (cx, [cy,] cz) belongs to phase (cx mod 3) + 3 (cy mod 3) + 9 (cz mod 3)
// (2-D: (cx mod 3) + 3 (cz mod 3)), phases in increasing order.  A target
// and its neighbours lie in the 3^d cells around the target's cell, and two
// cells of one phase are at least three cells apart along some axis, so those
// blocks of cells are disjoint and the cells of a phase are independent: one
// work-group per cell.  Within a cell the targets go in sorted order and the
// neighbours of each in the order of its row (ascending sorted index).  The
// result is the sequential definition with the targets ordered by (phase,
// cell, sorted index), up to rounding.
//
// Within one row the neighbours are distinct, so their values are read at
// once, and v_i after the first k exchanges is the composition of the affine
// maps x -> (1 - c_k) x + c_k v_jk: one prefix scan over the lanes (128
// entries at a time, two to a lane) gives v_i before every exchange, and with
// it every neighbour's new value (the scan runs on DPP row shifts and
// broadcasts).  The v values of the cell's block are staged in LDS (blocks
// larger than the LDS area are updated in place in memory by one wave, 64
// entries to a scan, the same maps).  J / Jbar is formed once before the phases and J / v once
// after.
#include "common.h"
#include "map_dev.h"
#include "tiles.h"

namespace vct {

int nlist_check(const vct_nlist* nl, Grid& g);

constexpr int kJCap = 1024;   // block values staged in LDS
// Launch shapes: waves of a cell's work-group, doubles of its LDS area, and the
// block size up to which the neighbours' positions are staged with the values
// (kJLong3: 5 groups to a CU; a block at R = 3 d0 has about 800).  Long rows in
// 3-D take the first, by the mean row length (short_row).
enum { kJLong3 = 0, kJShort3 = 1, kJ2 = 2 };
template <int C> struct JShape;
template <> struct JShape<kJLong3> { static constexpr int kD = 3, kWaves = 3, kArea = 3840, kPos = 960; };
template <> struct JShape<kJShort3> { static constexpr int kD = 3, kWaves = 1, kArea = kJCap, kPos = 0; };
template <> struct JShape<kJ2> { static constexpr int kD = 2, kWaves = 1, kArea = kJCap, kPos = 0; };

struct JbarArgs {
    int64_t n;
    Grid g;
    double cv, re;
    const double* pos;
    const int64_t* row_ptr;
    const uint16_t* col16;
    const int64_t* cs;
    const int64_t* chunk_off;
    const int32_t* cstart;
    const int4* cinfo;
    const int32_t* cwin;
    double* v;   // [n] J / Jbar, updated in place
};

__global__ __launch_bounds__(256) void k_jbar_ratio(int64_t n, const double* __restrict__ a,
                                                   const double* __restrict__ b, double* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = a[i] / b[i];
}

// Orders the LDS accesses of one wave around it (the hardware takes a wave's
// LDS instructions in order, so there is nothing to wait for; the compiler must
// not move or forward across lanes).
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ double lane_of(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// position of sorted index i in a window (the range holding it), or -1
template <int D>
__device__ __forceinline__ int window_offset_of(const WindowT<D>& w, int64_t i) {
    int t = -1;
#pragma unroll
    for (int r = 0; r < kMaxRanges; ++r)
        if (r < w.nr && i >= w.gstart[r] && i < w.gstart[r] + (w.off[r + 1] - w.off[r]))
            t = w.off[r] + (int)(i - w.gstart[r]);
    return t;
}

// A 64-bit value moved across lanes by a DPP control (row shifts, row
// broadcasts, wave shift); lanes without a source, or masked by the row mask,
// take `ID` (1 or 0).  Zero words come with the move itself where every row
// takes part.
template <int CTRL, int ROWMASK, int ID>
__device__ __forceinline__ double dpp_move64(double v) {
    constexpr int id_hi = ID ? 0x3ff00000 : 0;
    constexpr bool zero = ROWMASK == 0xF;
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWMASK, 0xF, zero);
    const int hi = __builtin_amdgcn_update_dpp(id_hi, __double2hiint(v), CTRL, ROWMASK, 0xF, zero && !ID);
    return __hiloint2double(hi, lo);
}

// One step of the inclusive scan of affine maps x -> a x + b over the lanes
// (lane k composes its map after the one the control brings in; the identity
// (1, 0) for lanes without one leaves a and b exactly as they are).
template <int CTRL, int ROWMASK = 0xF>
__device__ __forceinline__ void affine_step(double& a, double& b) {
    const double ao = dpp_move64<CTRL, ROWMASK, 1>(a), bo = dpp_move64<CTRL, ROWMASK, 0>(b);
    b = fma(a, bo, b);
    a = a * ao;
}

// Inclusive scan over the 64 lanes: within rows of 16 by row shifts of 1, 2,
// 4 and 8, then row 0's total into row 1 (and row 2's into row 3) by the
// row-15 broadcast, then the first two rows' total into rows 2 and 3 by the
// row-31 broadcast.
__device__ __forceinline__ void affine_scan(double& a, double& b) {
    affine_step<0x111>(a, b);         // row_shr:1
    affine_step<0x112>(a, b);         // row_shr:2
    affine_step<0x114>(a, b);         // row_shr:4
    affine_step<0x118>(a, b);         // row_shr:8
    affine_step<0x142, 0xA>(a, b);    // row_bcast:15 into rows 1 and 3
    affine_step<0x143, 0xC>(a, b);    // row_bcast:31 into rows 2 and 3
}

constexpr int kJSlots = 2;   // row entries per lane taken together (rows of up to 128 in one pass)
constexpr int kJRows = 64;   // row pointers of a cell held in registers (longer cells reload them)

// Pair weights c = C_V (r_e - |r^_ij|) / r_e and value addresses of the
// entries [e0 + s 64 + lane] of one row (s < kJSlots), decoded through the
// window of the row's chunk; entries past `re` get c = 0 and no address.
template <int D>
__device__ __forceinline__ void row_geometry(const JbarArgs& A, const WindowT<D>& cw, const WindowT<D>& blk, bool fast,
                                             int64_t i, int64_t e0, int64_t re, double (&c)[kJSlots],
                                             int64_t (&jj)[kJSlots]) {
    const int lane = threadIdx.x;
    const int64_t n = A.n;
    double xi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) xi[a] = a < D ? A.pos[a * n + i] : 0.0;
#pragma unroll
    for (int s = 0; s < kJSlots; ++s) {
        const int64_t e = e0 + s * kWave + lane;
        c[s] = 0.0;
        jj[s] = -1;
        if (e < re) {
            const int t = dcheck((int)A.col16[e], cw.off[cw.nr], kChkWindow);
            int r = 0;
#pragma unroll
            for (int k = 1; k < kMaxRanges; ++k)
                if (k < cw.nr && t >= cw.off[k]) r = k;
            const int64_t j = cw.gstart[r] + (t - cw.off[r]);
            // the chunk window and the block list the same columns in the same order
            jj[s] = fast ? blk.off[r] + (j - blk.gstart[r]) : j;
            double r2 = 0.0;
#pragma unroll
            for (int a = 0; a < D; ++a) {
                const double d = A.pos[a * n + j] - xi[a];
                r2 += d * d;
            }
            c[s] = A.cv * (A.re - sqrt(r2)) / A.re;
        }
    }
}

// The exchanges of one cell by one wave (the general form).  FAST: the block's
// values are in LDS (vp = s_v, addressed by block offset); otherwise in
// memory (vp = A.v, addressed by sorted index).  The geometry of the next
// target's row (its window offsets and neighbour positions, which no exchange
// changes) is loaded while the current row's exchanges run.
template <int D, bool FAST>
__device__ __forceinline__ void jbar_cell(const JbarArgs& A, int64_t col, int64_t p0, int64_t p1, double* vp,
                                          const WindowT<D>& blk, WindowT<D> (&cw)[2]) {
    const int lane = threadIdx.x;
    const Grid& g = A.g;
    // row pointers of targets [q0, q0 + 63], lane k holding row_ptr[q0 + k]
    int64_t q0 = p0;
    int64_t rp = A.row_ptr[q0 + lane < p1 ? q0 + lane : p1];
    auto row_ptr_of = [&](int64_t i) {   // uniform i in [q0, q0 + kJRows)
        return __shfl(rp, (int)(i - q0), kWave);
    };
    // chunk of a target: the column's chunks in order
    int64_t bc = A.chunk_off[col];
    auto chunk_of = [&](int64_t i) {
        while (A.cstart[bc + 1] <= i) ++bc;
        return bc;
    };
    auto load_window = [&](int64_t chunk, WindowT<D>& w) {
        if (A.cwin) window_load<D>(A.cwin, (uint32_t)chunk, w);
        else chunk_window_wave<D>(g, A.cs, A.cinfo[chunk], w);
    };

    int cur = 0;
    int64_t bcur = chunk_of(p0);
    load_window(bcur, cw[cur]);
    wave_order();
    int64_t rb = row_ptr_of(p0), re = p0 + 1 - q0 < kJRows ? row_ptr_of(p0 + 1) : A.row_ptr[p0 + 1];
    double c[kJSlots];
    int64_t jj[kJSlots];
    row_geometry<D>(A, cw[cur], blk, FAST, p0, rb, re, c, jj);

    for (int64_t i = p0; i < p1; ++i) {
        // the next target's geometry first
        const bool more = i + 1 < p1;
        int64_t rb1 = 0, re1 = 0;
        int nxt = cur;
        double c1[kJSlots] = {};
        int64_t jj1[kJSlots] = {};
        if (more) {   // uniform
            if (i + 2 - q0 > kJRows) {   // refill the row pointers (uniform)
                q0 = i + 1;
                rp = A.row_ptr[q0 + lane < p1 ? q0 + lane : p1];
            }
            rb1 = row_ptr_of(i + 1);
            re1 = i + 2 - q0 < kJRows ? row_ptr_of(i + 2) : A.row_ptr[i + 2];
            const int64_t b1 = chunk_of(i + 1);
            if (b1 != bcur) {   // uniform: the next target starts a new chunk
                nxt = 1 - cur;
                load_window(b1, cw[nxt]);
                bcur = b1;
                wave_order();
            }
            row_geometry<D>(A, cw[nxt], blk, FAST, i + 1, rb1, re1, c1, jj1);
        }
        const int64_t ii = FAST ? window_offset_of<D>(blk, i) : i;
        double vi = vp[ii];
        for (int64_t e0 = rb; e0 < re; e0 += kWave * kJSlots) {
            if (e0 != rb) row_geometry<D>(A, cw[cur], blk, FAST, i, e0, re, c, jj);   // rows longer than 128
            double vj[kJSlots];
#pragma unroll
            for (int s = 0; s < kJSlots; ++s) vj[s] = jj[s] >= 0 ? vp[jj[s]] : 0.0;
            // slot by slot: the scan of the maps x -> (1 - c) x + c v_j gives
            // v_i before every lane's exchange (padding lanes are the identity)
#pragma unroll
            for (int s = 0; s < kJSlots; ++s) {
                double am = 1.0 - c[s], bm = c[s] * vj[s];
                affine_scan(am, bm);
                const double ap = dpp_move64<0x138, 0xF, 1>(am), bp = dpp_move64<0x138, 0xF, 0>(bm);   // wave_shr:1
                const double xk = fma(ap, vi, bp);
                if (jj[s] >= 0) vp[jj[s]] = vj[s] - c[s] * (vj[s] - xk);
                const double aT = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(am), kWave - 1),
                                                   __builtin_amdgcn_readlane(__double2loint(am), kWave - 1));
                const double bT = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(bm), kWave - 1),
                                                   __builtin_amdgcn_readlane(__double2loint(bm), kWave - 1));
                vi = fma(aT, vi, bT);
            }
        }
        if (lane == 0) vp[ii] = vi;
        if (!FAST) __threadfence_block();
        wave_order();   // this row's values before the next row reads them
        cur = nxt;
        rb = rb1;
        re = re1;
#pragma unroll
        for (int s = 0; s < kJSlots; ++s) {
            c[s] = c1[s];
            jj[s] = jj1[s];
        }
    }
}

constexpr int kJWins = 4;   // chunk windows of one cell held in LDS

// A hand-over between the waves of the group: LDS writes before it are seen by
// LDS reads after it (loads from memory stay in flight across it).
template <int WAVES>
__device__ __forceinline__ void turn_over() {
    if (WAVES == 1) return wave_order();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// sqrt(x), x >= 0, from the hardware's estimate y of 1/sqrt(x): g = x y
// corrected by (x - g^2) y / 2, whose factors stay in range for every x (y^2
// does not below 2^-1022, the square of a distance of 1e-154).
__device__ __forceinline__ double pair_distance(double x) {
    const double y = __builtin_amdgcn_rsq(x), g = x * y;
    return x > 0.0 ? fma(fma(-g, g, x), 0.5 * y, g) : 0.0;
}

// The part of a row's exchanges that no value enters.  Entries 2 lane and
// 2 lane + 1 of up to 128 are the lane's: their weights c (0 past the row's
// end) and LDS places jl (-1 there), and the slopes of the scan over the lanes'
// composed maps x -> (1 - c1) ((1 - c0) x + ..) + ..: before each step, before
// the lane (ap) and of the whole row (aT).
struct RowMaps {
    int len;
    int jl[2];
    double c[2], a[6], ap, aT;
};
__device__ __forceinline__ int row_last(int len) { return len > 64 ? kWave - 1 : len > 32 ? 31 : 15; }
__device__ __forceinline__ void row_slopes(RowMaps& m) {
    m.a[0] = (1.0 - m.c[0]) * (1.0 - m.c[1]);
    m.a[1] = m.a[0] * dpp_move64<0x111, 0xF, 1>(m.a[0]);   // row_shr:1, 2, 4, 8
    m.a[2] = m.a[1] * dpp_move64<0x112, 0xF, 1>(m.a[1]);
    m.a[3] = m.a[2] * dpp_move64<0x114, 0xF, 1>(m.a[2]);
    m.a[4] = m.a[3] * dpp_move64<0x118, 0xF, 1>(m.a[3]);
    m.a[5] = m.a[4];
    if (m.len > 32) m.a[5] *= dpp_move64<0x142, 0xA, 1>(m.a[4]);   // uniform; row_bcast:15 into rows 1 and 3
    double t = m.a[5];
    if (m.len > 64) t *= dpp_move64<0x143, 0xC, 1>(t);   // uniform; row_bcast:31 into rows 2 and 3
    m.ap = dpp_move64<0x138, 0xF, 1>(t);                 // wave_shr:1
    m.aT = lane_of(t, row_last(m.len));
}
// The exchanges of one row from target value vi; returns the target's value
// after them.  The scan gives the target's value before each lane's pair.
__device__ __forceinline__ double exchange_row(double* s_v, const RowMaps& m, double vi) {
    double v[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) v[s] = m.jl[s] >= 0 ? s_v[m.jl[s]] : 0.0;
    double b = fma(1.0 - m.c[1], m.c[0] * v[0], m.c[1] * v[1]);
    b = fma(m.a[0], dpp_move64<0x111, 0xF, 0>(b), b);
    b = fma(m.a[1], dpp_move64<0x112, 0xF, 0>(b), b);
    b = fma(m.a[2], dpp_move64<0x114, 0xF, 0>(b), b);
    b = fma(m.a[3], dpp_move64<0x118, 0xF, 0>(b), b);
    if (m.len > 32) b = fma(m.a[4], dpp_move64<0x142, 0xA, 0>(b), b);
    if (m.len > 64) b = fma(m.a[5], dpp_move64<0x143, 0xC, 0>(b), b);
    const double x0 = fma(m.ap, vi, dpp_move64<0x138, 0xF, 0>(b));
    const double d0 = m.c[0] * (v[0] - x0), d1 = m.c[1] * (v[1] - (x0 + d0));
    if (m.jl[0] >= 0) s_v[m.jl[0]] = v[0] - d0;
    if (m.jl[1] >= 0) s_v[m.jl[1]] = v[1] - d1;
    return fma(m.aT, vi, lane_of(b, row_last(m.len)));
}

// The exchanges of one cell whose block fits the LDS area and whose targets
// lie in at most kJWins chunks (whose windows are all in LDS, cwa[k] for
// chunk b0 + k, starting at sorted index cst[k]; sh[k][r] the shifts of its
// range r from window offset to sorted index and to block offset).  ii0 is the
// first target's place in the block.
// What bounds it: the rows of a cell are a serial chain, and a phase has only
// two or three cells per SIMD, the slowest of which (a cell of 4 planes where
// the others have 3) ends it; per row about 190 vector instructions.  So a row
// costs one scan (two entries per lane composed first) instead of two, all that
// is uniform sits in scalar registers, and where rows are long the waves of the
// group take the rows in turn: each prepares its next row (offsets, positions,
// weights, slopes of the scan) while the others have the turn, and the
// neighbours' positions come from LDS.  2,097,152 particles, R = 3 d0: 0.135 ->
// 0.072 ms a phase (one wave, positions from memory: 0.083); 72,000: 0.109 ->
// 0.028 ms.  Short rows (cubic spline at 2.4 d0, 14 targets a cell; 2-D, 9) keep
// one wave, whose smaller LDS area lets all cells of a phase run at once:
// 1,065,547 particles 0.077 -> 0.048 ms a phase (the long shape 0.054), 2-D,
// 524,288: 0.051 -> 0.039 (three waves 0.045).
template <int C, bool POS>
__device__ __forceinline__ void jbar_cell_shared(const JbarArgs& A, int p0, int p1, double* s_v, int ii0,
                                                 const WindowT<JShape<C>::kD>* cwa, const int (&cst)[kJWins],
                                                 const int2 (*sh)[kMaxRanges]) {
    constexpr int D = JShape<C>::kD, kN = JShape<C>::kWaves, kP = JShape<C>::kPos;
    constexpr int kR = D == 3 ? 9 : 3;
    constexpr int kRow = 2 * kWave;
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t n = A.n;
    const double cvr = A.cv / A.re;
    auto uni = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
    // the window of the target whose positions are loaded next
    int kw = -1, off[kR], wlen = 0;
    auto window_of = [&](int i) {   // uniform
        int k = 0;
#pragma unroll
        for (int q = 1; q < kJWins; ++q) k = i >= cst[q] ? q : k;   // starts past the cell's chunks: p1
        k = uni(k);
        if (k != kw) {
            kw = k;
            const int nr = uni(cwa[k].nr);
            wlen = uni(cwa[k].off[nr]);
#pragma unroll
            for (int q = 0; q < kR; ++q) {
                const int o = uni(cwa[k].off[q]);
                off[q] = q < nr ? o : INT32_MAX;
            }
        }
    };
    // entries of the targets' rows, counted from the cell's first: lane k holds
    // the row start of target q0 + k; asked for in increasing order
    const int64_t e0 = A.row_ptr[p0];
    const int ne = uni((int)(A.row_ptr[p1] - e0));
    if (ne == 0) return;   // uniform over the group
    const uint16_t* c16 = A.col16 + e0;
    int q0 = p0;
    auto row_starts = [&] { return (int)(A.row_ptr[q0 + lane < p1 ? q0 + lane : p1] - e0); };
    int rp = row_starts();
    // and the position of target x0 + k
    int x0 = p0;
    double px[D];
    auto target_pos = [&] {
#pragma unroll
        for (int a = 0; a < D; ++a) px[a] = A.pos[a * n + (x0 + lane < p1 ? x0 + lane : p1 - 1)];
        // waited for here, in the rare branch that reloads them: left in flight, every use would wait for all loads
#pragma unroll
        for (int a = 0; a < D; ++a) asm volatile("" : "+v"(px[a]));
    };
    target_pos();

    // A row on its way.  The loads are issued by every lane (lanes past the
    // row's end read the cell's last entry and the window's first particle): a
    // load under a branch could not stay in flight past it.
    int rb, re, t[2];              // the row whose offsets are under way
    int frb = 0, flen, fjl[2];     // the row whose positions are under way
    double xj[2][D];
    auto start = [&](int i) {   // offsets; rows past the cell's last are empty
        rb = re = 0;
        if (i < p1) {   // uniform
            if (i < q0 || i + 1 - q0 >= kJRows) {   // (back only after a long row)
                q0 = i;
                rp = row_starts();
                asm volatile("" : "+v"(rp));   // waited for here, as the target positions
            }
            rb = __builtin_amdgcn_readlane(rp, i - q0);
            re = __builtin_amdgcn_readlane(rp, i + 1 - q0);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int e = rb + 2 * lane + s;
            t[s] = c16[(unsigned)(e < ne ? e : ne - 1)];
        }
    };
    auto fetch = [&](int i) {   // positions of the started row, target i's
        window_of(i < p1 ? i : p1 - 1);
        frb = rb;
        flen = re - rb;
        bool in[2];
        int tt[2];
        int2 d[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            in[s] = 2 * lane + s < flen;
            tt[s] = dcheck(in[s] ? t[s] : 0, wlen, kChkWindow);
            int r = 0;
#pragma unroll
            for (int q = 1; q < kR; ++q) r += tt[s] >= off[q] ? 1 : 0;
            d[s] = sh[kw][r];
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            // (a window's first particle may lie outside the block: its own place 0 serves as well)
            fjl[s] = in[s] ? tt[s] + d[s].y : -1;
            const int jl = in[s] ? tt[s] + d[s].y : 0;
#pragma unroll
            for (int a = 0; a < D; ++a)
                xj[s][a] = POS ? s_v[(1 + a) * kP + jl] : A.pos[a * n + (unsigned)(tt[s] + d[s].x)];
        }
    };
    // the pair weights c = C_V (r_e - |r^_ij|) / r_e of target i's entries
    auto weights = [&](int i, RowMaps& m) {
        if (i - x0 >= kWave) {   // uniform
            x0 = i;
            target_pos();
        }
        double xi[D];
#pragma unroll
        for (int a = 0; a < D; ++a) xi[a] = lane_of(px[a], i - x0);
        m.len = flen;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            double r2 = 0.0;
#pragma unroll
            for (int a = 0; a < D; ++a) {
                const double d = xj[s][a] - xi[a];
                r2 += d * d;
            }
            m.jl[s] = fjl[s];
            const double c = cvr * (A.re - pair_distance(r2));
            m.c[s] = m.jl[s] >= 0 ? c : 0.0;
        }
        row_slopes(m);
    };

    RowMaps m;
    int mrb;   // first entry of m's row
    // wave w takes targets p0 + w, + kN, ..: its first row complete, the
    // second's positions and the third's offsets under way
    start(p0 + wave);
    fetch(p0 + wave);
    start(p0 + wave + kN);
    weights(p0 + wave < p1 ? p0 + wave : p1 - 1, m);
    mrb = frb;
    fetch(p0 + wave + kN);
    start(p0 + wave + 2 * kN);
    int mine = p0 + wave;
    bool ahead = false;   // the second part of the preparation is still to do
    for (int i = p0; i < p1; ++i) {
        const bool turn = kN == 1 || i == mine;   // uniform per wave
        if (turn) {
            const int ii = ii0 + (i - p0);
            double vi = exchange_row(s_v, m, s_v[ii]);
            if (m.len > kRow) {   // uniform: more entries than the lanes hold; the rest in place
                const int len = m.len;
                for (int eb = kRow; eb < len; eb += kRow) {
                    rb = mrb + eb;
                    re = mrb + len;
#pragma unroll
                    for (int s = 0; s < 2; ++s) t[s] = c16[(unsigned)(rb + 2 * lane + s < ne ? rb + 2 * lane + s : ne - 1)];
                    fetch(i);
                    weights(i, m);
                    wave_order();
                    vi = exchange_row(s_v, m, vi);
                }
                start(i + kN);   // what was under way, again
                fetch(i + kN);
                start(i + 2 * kN);
            }
            if (lane == 0) s_v[ii] = vi;
        }
        turn_over<kN>();   // this row's values before the next row reads them
        // the wave's next rows, while the other waves take their turns
        if (turn) {
            weights(i + kN < p1 ? i + kN : p1 - 1, m);
            mrb = frb;
            mine = i + kN;
        }
        if (kN <= 2 ? turn : ahead) {
            fetch(mine + kN);
            start(mine + 2 * kN);
        }
        ahead = turn;
    }
}

// A block between memory and LDS, range by range (a range is a run of
// consecutive particles of one column), the ranges over the waves: the values,
// and with POS the positions; every load before the first LDS store, as far as
// ranges of up to 128 go.
template <int C, bool POS>
__device__ __forceinline__ void block_load(const WindowT<JShape<C>::kD>& blk, const double* __restrict__ v,
                                           const double* __restrict__ pos, int64_t n, double* s_v) {
    constexpr int D = JShape<C>::kD, kN = JShape<C>::kWaves, kP = JShape<C>::kPos;
    constexpr int kR = D == 3 ? 9 : 3, kRep = (kR + kN - 1) / kN, kA = POS ? 1 + D : 1;
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    double x[kRep][2][kA];
#pragma unroll
    for (int k = 0; k < kRep; ++k) {
        const int r = wave + k * kN;
        const int len = r < blk.nr ? blk.off[r + 1] - blk.off[r] : 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int t = lane + h * kWave;
            if (t < len) {
                const int64_t j = blk.gstart[r] + t;
                x[k][h][0] = v[j];
#pragma unroll
                for (int a = 1; a < kA; ++a) x[k][h][a] = pos[(a - 1) * n + j];
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kRep; ++k) {
        const int r = wave + k * kN;
        const int len = r < blk.nr ? blk.off[r + 1] - blk.off[r] : 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int t = lane + h * kWave;
#pragma unroll
            for (int a = 0; a < kA; ++a)
                if (t < len) s_v[a * kP + blk.off[r] + t] = x[k][h][a];
        }
        for (int t = lane + 2 * kWave; t < len; t += kWave) {
            const int64_t j = blk.gstart[r] + t;
            s_v[blk.off[r] + t] = v[j];
#pragma unroll
            for (int a = 1; a < kA; ++a) s_v[a * kP + blk.off[r] + t] = pos[(a - 1) * n + j];
        }
    }
}

template <int C>
__device__ __forceinline__ void block_store(const WindowT<JShape<C>::kD>& blk, const double* s_v, double* v) {
    const int lane = threadIdx.x % kWave;
    for (int r = threadIdx.x / kWave; r < blk.nr; r += JShape<C>::kWaves) {
        const int len = blk.off[r + 1] - blk.off[r];
        for (int t = lane; t < len; t += kWave) v[blk.gstart[r] + t] = s_v[blk.off[r] + t];
    }
}

// One cell of phase `phase` per work-group.
template <int C>
__global__ __launch_bounds__(kWave* JShape<C>::kWaves) void k_jbar_phase(JbarArgs A, int phase, uint32_t uy, uint32_t uz) {
    constexpr int D = JShape<C>::kD;
    __shared__ double s_v[JShape<C>::kArea];   // the block's values, and its positions
    __shared__ WindowT<D> blk;     // the 3^d cells around the cell
    __shared__ WindowT<D> cw[2];   // windows of the chunks of the current and the next target
    __shared__ WindowT<D> cwa[kJWins];          // windows of the cell's chunks
    __shared__ int2 s_sh[kJWins][kMaxRanges];   // per range: shifts to the sorted index and to the block offset
    const int lane = threadIdx.x % kWave;
    const bool first = threadIdx.x < kWave;   // the wave that fills the tables
    const Grid& g = A.g;
    // the cell: z (last axis) fastest over the phase's cells
    uint32_t b = blockIdx.x;
    int cx, cy = 0, cz;
    if (D == 3) {
        cz = phase / 9 + 3 * (b % uz);
        b /= uz;
        cy = (phase / 3) % 3 + 3 * (b % uy);
        b /= uy;
        cx = phase % 3 + 3 * b;
    } else {
        cz = phase / 3 + 3 * (b % uz);
        b /= uz;
        cx = phase % 3 + 3 * b;
    }
    const int64_t col = D == 3 ? (int64_t)cx * g.nc[1] + cy : cx;
    const int64_t key = col_key<D>(g, col, cz);
    const int64_t p0 = A.cs[key], p1 = A.cs[key + 1];
    int64_t b0 = A.chunk_off[col];
    const int64_t bend = A.chunk_off[col + 1];
    if (p0 == p1) return;   // uniform over the work-group
    // the chunks holding the cell's targets: the column's chunk starts over the
    // lanes, b0 moved up until lane 0 has the chunk of the first target or the
    // rest of the column is in the lanes
    auto starts = [&] { return b0 + lane < bend ? A.cstart[b0 + lane] : INT32_MAX; };
    int st = starts();
    int k0 = __popcll(__ballot(st <= p0)) - 1;
    while (k0 + kJWins >= kWave - 1 && b0 + kWave < bend) {   // uniform; rare (columns of over 59 chunks)
        b0 += k0;
        st = starts();
        k0 = __popcll(__ballot(st <= p0)) - 1;
        if (k0 == 0) break;
    }
    const int nchk = __popcll(__ballot(st < p1)) - k0;
    b0 += k0;
    if (first) chunk_window_wave<D>(g, A.cs, make_int4((int)col, cz, cz, 0), blk);
    __syncthreads();
    const int W = blk.off[blk.nr];
    if (W <= kJCap) {   // uniform
        if (nchk <= kJWins) {   // uniform
            int cst[kJWins];
#pragma unroll
            for (int k = 0; k < kJWins; ++k) {
                cst[k] = k < nchk ? __builtin_amdgcn_readlane(st, k0 + k) : (int)p1;
                if (first && k < nchk) {
                    if (A.cwin) window_load<D>(A.cwin, (uint32_t)(b0 + k), cwa[k]);
                    else chunk_window_wave<D>(g, A.cs, A.cinfo[b0 + k], cwa[k]);
                }
            }
            const bool pos = W <= JShape<C>::kPos;   // uniform
            if constexpr (JShape<C>::kPos > 0) {
                if (pos) block_load<C, true>(blk, A.v, A.pos, A.n, s_v);
            }
            if (!pos) block_load<C, false>(blk, A.v, A.pos, A.n, s_v);
            __syncthreads();
            // per window and range: window offset -> sorted index and -> block
            // offset (the chunk windows and the block list the same columns
            // in the same order)
            if (first && lane < nchk * kMaxRanges) {
                const int k = lane / kMaxRanges, r = lane % kMaxRanges;
                const WindowT<D>& w = cwa[k];
                const int64_t g0 = r < w.nr ? w.gstart[r] - w.off[r] : 0;
                s_sh[k][r] = make_int2((int)g0, r < w.nr ? (int)(g0 - blk.gstart[r]) + blk.off[r] : 0);
            }
            __syncthreads();
            auto uni = [](int64_t x) { return __builtin_amdgcn_readfirstlane((int)x); };
            const int ii0 = uni(window_offset_of<D>(blk, p0));
            if constexpr (JShape<C>::kPos > 0) {
                if (pos) jbar_cell_shared<C, true>(A, uni(p0), uni(p1), s_v, ii0, cwa, cst, s_sh);
            }
            if (!pos) jbar_cell_shared<C, false>(A, uni(p0), uni(p1), s_v, ii0, cwa, cst, s_sh);
        } else {
            block_load<C, false>(blk, A.v, A.pos, A.n, s_v);
            __syncthreads();
            if (first) jbar_cell<D, true>(A, col, p0, p1, s_v, blk, cw);
        }
        __syncthreads();
        block_store<C>(blk, s_v, A.v);
    } else if (first) {
        jbar_cell<D, false>(A, col, p0, p1, A.v, blk, cw);
    }
}

// J = det J = alpha at every particle (Eq. det_jacobi)
__global__ __launch_bounds__(256) void k_map_alpha(int dim, int64_t n, const double* __restrict__ pos, MapParams mp,
                                                   double* __restrict__ alpha) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double x = pos[i], y = dim == 3 ? pos[n + i] : 0.0, zh = pos[(int64_t)(dim - 1) * n + i];
    alpha[i] = map_coef_at(mp, i, x, y, zh).alpha;
}

// projected positions of physical points: x^ = x, y^ = y, z^ = alpha (z + beta) (Eq. VCT)
__global__ __launch_bounds__(256) void k_map_project(int dim, int64_t n, const double* __restrict__ phys, MapParams mp,
                                                     double* __restrict__ proj) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double x = phys[i], y = dim == 3 ? phys[n + i] : 0.0, z = phys[(int64_t)(dim - 1) * n + i];
    const MapCoef<double> c = map_coef_at(mp, i, x, y, 0.0);
    for (int a = 0; a < dim - 1; ++a) proj[(int64_t)a * n + i] = phys[(int64_t)a * n + i];
    proj[(int64_t)(dim - 1) * n + i] = c.alpha * (z + c.beta);
}

VCT_CHECKS_TU(checks_jbar)

}  // namespace vct

using namespace vct;

extern "C" size_t vct_jbar_workspace_size(int64_t n) {
    if (n < 0) return 0;
    return aligned_sum({(size_t)(n > 0 ? n : 1) * sizeof(double)});
}

extern "C" int vct_jbar_smooth(const vct_nlist* nl, const double* pos_sorted, const double* J, double* jbar, double cv,
                               double re, void* ws, size_t ws_bytes, void* stream) {
    VCT_API_RANGE("vct_jbar_smooth");
    Grid g;
    int st = nlist_check(nl, g);
    if (st) return st;
    if (!isfinite(cv) || !(re > 0.0) || !isfinite(re)) return VCT_E_ARG;
    const int64_t n = nl->n;
    if (n == 0) return VCT_OK;
    if (!pos_sorted || !J || !jbar || !nl->col16) return VCT_E_ARG;
    if (!ws || ws_bytes < vct_jbar_workspace_size(n)) return VCT_E_WORKSPACE;
    Carver cv_ws(ws, ws_bytes);
    double* v = cv_ws.take<double>((size_t)n);
    hipStream_t s = as_stream(stream);
    JbarArgs a;
    a.n = n; a.g = g; a.cv = cv; a.re = re; a.pos = pos_sorted; a.row_ptr = nl->row_ptr; a.col16 = nl->col16;
    a.cs = nl->cell_start; a.chunk_off = nl->chunk_off; a.cstart = nl->chunk_start;
    a.cinfo = reinterpret_cast<const int4*>(nl->chunk_info); a.cwin = nl->chunk_win; a.v = v;
    const unsigned nb = (unsigned)((n + 255) / 256);
    VCT_LAUNCH("k_jbar_ratio", k_jbar_ratio, dim3(nb), dim3(256), 0, s, n, J, jbar, v);
    VCT_LAUNCH_CHECK();
    const int dim = nl->dim;
    const int nph = dim == 3 ? 27 : 9;
    const int64_t nx = g.nc[0], ny = dim == 3 ? g.nc[1] : 1, nz = dim == 3 ? g.nc[2] : g.nc[1];
    auto count = [](int64_t nc, int64_t p) { return nc > p ? (nc - p + 2) / 3 : 0; };
    for (int ph = 0; ph < nph; ++ph) {
        const int64_t ux = count(nx, ph % 3);
        const int64_t uy = dim == 3 ? count(ny, (ph / 3) % 3) : 1;
        const int64_t uz = count(nz, dim == 3 ? ph / 9 : ph / 3);
        const int64_t cells = ux * uy * uz;
        if (cells == 0) continue;
        const dim3 gr((unsigned)cells);
        const uint32_t vy = (uint32_t)uy, vz = (uint32_t)uz;
        if (dim == 2) VCT_LAUNCH("k_jbar_phase", k_jbar_phase<kJ2>, gr, dim3(kWave), 0, s, a, ph, vy, vz);
        else if (mean_row(nl) <= short_row<3>())
            VCT_LAUNCH("k_jbar_phase", k_jbar_phase<kJShort3>, gr, dim3(kWave), 0, s, a, ph, vy, vz);
        else
            VCT_LAUNCH("k_jbar_phase", k_jbar_phase<kJLong3>, gr, dim3(kWave * JShape<kJLong3>::kWaves), 0, s, a, ph, vy, vz);
        VCT_LAUNCH_CHECK();
    }
    VCT_LAUNCH("k_jbar_ratio", k_jbar_ratio, dim3(nb), dim3(256), 0, s, n, J, v, jbar);
    VCT_LAUNCH_CHECK();
    return VCT_OK;
}

extern "C" int vct_map_alpha(int dim, int64_t n, const double* pos, const vct_map* map, double* alpha, void* stream) {
    VCT_API_RANGE("vct_map_alpha");
    if ((dim != 2 && dim != 3) || n < 0 || !map) return VCT_E_ARG;
    MapParams mp;
    const int st = map_params_from(map, dim, n, mp);
    if (st) return st;
    if (n == 0) return VCT_OK;
    if (!pos || !alpha) return VCT_E_ARG;
    VCT_LAUNCH("k_map_alpha", k_map_alpha, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, as_stream(stream), dim, n,
               pos, mp, alpha);
    VCT_LAUNCH_CHECK();
    return VCT_OK;
}

extern "C" int vct_map_project(int dim, int64_t n, const double* phys, const vct_map* map, double* proj, void* stream) {
    VCT_API_RANGE("vct_map_project");
    if ((dim != 2 && dim != 3) || n < 0 || !map) return VCT_E_ARG;
    MapParams mp;
    const int st = map_params_from(map, dim, n, mp);
    if (st) return st;
    if (n == 0) return VCT_OK;
    if (!phys || !proj || phys == proj) return VCT_E_ARG;
    VCT_LAUNCH("k_map_project", k_map_project, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, as_stream(stream),
               dim, n, phys, mp, proj);
    VCT_LAUNCH_CHECK();
    return VCT_OK;
}
