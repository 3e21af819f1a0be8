// Operator application (paper Sec. 3.1, Eqs. gra_1st and sec_SPH2; Sec. 2.1,
// Eqs. grad_VCT and lap_VCT): the neighbour sums [a_i; s_i] of each field,
// then out_i = P_i [a_i; s_i] with the per-particle state of vct_moments.
//
// Numerics.  phi_ij is dominated by its first-order part r_ij . grad phi,
// which cancels across a (nearly) symmetric neighbourhood in s_i; rounding the
// individual terms is then amplified by |grad phi| / (R |Hess phi|).  The
// operator is linear and reproduces linear fields exactly, so for any vector
// G, out(phi) = P [a; s](psi) + W G with psi_ij = phi_ij - (x_j - x_i) . G and
// W the response of the output rows to a unit projected gradient (stored by
// vct_moments).  The kernel sums in two passes: pass 1 forms the particle's
// first-order gradient G = L a (d sums), pass 2 sums the residual psi, which
// is second-order small and has a(psi) = 0 up to rounding.  psi is formed in
// FP64 from the FP64 positions and field values; the pair geometry, kernel and
// sums run in the arithmetic type T (FP64, or FP32 for the mixed form).  The
// result is the same linear operator; only the rounding changes.
//
// Work decomposition.  One work-group per chunk (at most 64 consecutive
// particles of one cell column).  The chunk's neighbour window (positions,
// field values, volumes) and its block of 16-bit row entries are staged once
// in LDS with coalesced loads; each particle is served by kLanes lanes that
// hold their share of the row entries in registers and read the pair records
// from LDS, software-pipelined one record ahead.  The group reduces its sums
// with cross-lane shuffles; the products with the state are done with one
// thread per (row, particle) so that the state is read with unit stride.
// Work-groups are remapped so each XCD covers a contiguous range of chunks.
#include <type_traits>

#include "common.h"
#include "tiles.h"

namespace vct {

int nlist_check(const vct_nlist* nl, Grid& g);

// Launch classes, chosen on the host by the mean row length (short_row in
// tiles.h).  A row's entries are spread over `lanes` lanes that hold `slots` of
// them each in registers, and both passes run over every slot, so the slots
// that a set's rows do not fill are work for nothing: the long-row shape (112
// entries, Wendland C2 with R = 3 d0 in 3-D: 103) costs a 2-D set with 26
// neighbours four times the pair terms it needs and reserves five times its
// LDS window, which leaves two work-groups on a CU where six fit.
//   kShort2: 2-D rows up to about 30 entries, 4 lanes x 7 or 8 slots in
//     256-thread groups (8 lanes x 4 slots: 20-40% slower), windows up to 448
//     records (297 at R = 3 d0).  1,048,576 particles, R = 3 d0: FP64 0.385 ->
//     0.127 ms, mixed 0.235 -> 0.096 ms (floor at the copy rate: 0.07 and 0.05
//     ms).
//   kShort3: 3-D rows up to 64 entries (cubic spline, R = 2.4 d0: 57), 4 lanes
//     x 16 slots, row entries read straight into the registers and a window
//     that lets three groups share a CU (53,760 bytes each: LDS comes in
//     pieces of 1,280 bytes).  2,097,152 particles: FP64 1.29 -> 0.91 ms,
//     mixed 0.82 -> 0.64 ms; with 8 lanes x 8 slots and two groups 0.97 and
//     0.70 ms.
// A row longer than its class's slots finishes in a loop over the rest, a
// window larger than the class's reads its records from memory: a set whose
// rows are short on average but not everywhere stays correct.
enum { kLongRows = 0, kShort3 = 1, kShort2 = 2 };

// Lanes per particle, register slots per lane, occupancy target (waves per
// SIMD), LDS window capacity (records) and row entries of a chunk staged in
// LDS (0: read from memory into the slots) of each arithmetic type and class.
// The long-row class runs 512-thread groups (8 lanes per particle) at 4 waves
// per SIMD, two groups per CU; its FP64 form takes a smaller window (about 77
// KB of LDS per group) and fills the 128 VGPRs that 4 waves allow.
template <int LANES, int SLOTS, int WAVES, int WIN, int COLS> struct ApplyShape {
    static constexpr int lanes = LANES, slots = SLOTS, waves = WAVES, win = WIN, cols = COLS;
};
template <class T, int C> struct ApplyCfg;
template <> struct ApplyCfg<float, kLongRows> : ApplyShape<8, 14, 4, 1664, 7168> {};
template <> struct ApplyCfg<double, kLongRows> : ApplyShape<8, 14, 4, 1400, 7168> {};
template <> struct ApplyCfg<float, kShort3> : ApplyShape<4, 16, 3, 1400, 0> {};
template <> struct ApplyCfg<double, kShort3> : ApplyShape<4, 16, 3, 1184, 0> {};
template <> struct ApplyCfg<float, kShort2> : ApplyShape<4, 8, 5, 448, 2304> {};
template <> struct ApplyCfg<double, kShort2> : ApplyShape<4, 7, 5, 448, 2304> {};

// The FP32 sums of the mixed form keep one order in every class, that of eight
// lanes per row: with fewer lanes a lane holds as many partial sums as it
// stands for (entry k of a row belongs to sum k mod 8), combined at the end as
// the eight lanes combine theirs.  A set's class then leaves the bits of the
// mixed form alone (in FP64 the order moves the last digits only).
template <class T, int LANES> constexpr int kParts = sizeof(T) == 4 ? 8 / LANES : 1;

template <class S> struct ApplyArgs {
    int64_t n;
    int nf;
    int nrows;
    double invR;
    Grid g;
    const double* phi;
    const double* pos;
    const double* vol;
    const int64_t* row_ptr;
    const uint16_t* col16;
    const int64_t* cs;
    const int32_t* cstart;
    const int4* cinfo;
    const int32_t* cwin;   // stored windows or NULL
    const int64_t* nchunks;
    const S* state;
    double* out;
    float* g_out;        // [nf][D][n] or NULL: the first pass's G~, written
    const float* g_in;   // [nf][D][n] or NULL: G~ given to the FP64 form (first pass skipped)
    int lap_row;               // the row of the system form (kLap)
    const uint8_t* dirichlet;  // [n] or NULL: its rows that return the field itself
};

// The mixed form keeps positions in units of R (x / R, in FP64): the FP64
// offset is then r~ itself and only needs rounding to FP32.  The FP64 form
// keeps positions as they are, so its offsets are exact differences.
template <class T> struct Scaled {
    static constexpr bool value = std::is_same<T, float>::value;
};

// Pair geometry: FP64 offset dx = x_j - x_i (in units of R for the mixed
// form), r~ = dx / R, q^2 = |r~|^2 and V_j c~(q) in the arithmetic type T;
// with IQ4 also 1 / q^4, both from one reciprocal square root.  An empty
// register slot (use false) takes q^2 = 4, outside the support: c~ = 0
// exactly, 1 / q^4 stays finite, and its terms add zero without a mask on
// each product.
template <int D, int KERNEL, class T, bool IQ4 = false>
__device__ __forceinline__ void pair_geom(const double4& q, T vj, const double (&xi)[3], T invR,
                                          double (&dx)[D], T (&r)[D], T& q2, T& vc, T* iq4 = nullptr,
                                          bool use = true) {
    dx[0] = q.x - xi[0];
    dx[1] = q.y - xi[1];
    if (D == 3) dx[D - 1] = q.z - xi[2];
    q2 = T(0);
#pragma unroll
    for (int a = 0; a < D; ++a) {
        r[a] = Scaled<T>::value ? T(dx[a]) : T(dx[a]) * invR;
        q2 += r[a] * r[a];
    }
    q2 = use ? q2 : T(4);
    if (IQ4) {
        T rs;
        if constexpr (Scaled<T>::value) rs = __builtin_amdgcn_rsqf(q2);
        else rs = vrsq(q2);
        const T rs2 = rs * rs;
        vc = vj * kernel_shape<KERNEL>(q2 * rs);
        *iq4 = rs2 * rs2;
    } else {
        vc = vj * kernel_shape<KERNEL>(vsqrt(q2));
    }
}

// Sums of one pair with residual psi: a~ += V c~ psi r~ and
// s~ += V c~ psi (r~' L~ r~) / |r~|^4 r~ r~' (L2 holds L~ with doubled
// off-diagonal entries), with vq = V c~ / |r~|^4 given.
template <int D, class T, int H>
__device__ __forceinline__ void pair_sums(const T (&r)[D], T vq, T vc, T psi, const T (&L2)[Dims<D>::nL],
                                          T (&acc)[Dims<D>::nk][H], int h) {
    using Dm = Dims<D>;
    T qv[Dm::m];
#pragma unroll
    for (int p = 0; p < Dm::m; ++p) qv[p] = r[pair_a<D>(p)] * r[pair_b<D>(p)];
    T rLr = T(0);
#pragma unroll
    for (int p = 0; p < Dm::nL; ++p) rLr += L2[p] * qv[p];
    const T wa = vc * psi, ws = vq * psi * rLr;
#pragma unroll
    for (int a = 0; a < D; ++a) acc[a][h] += wa * r[a];
#pragma unroll
    for (int p = 0; p < Dm::m; ++p) acc[D + p][h] += ws * qv[p];
}

// Total of a lane group's partial sums, H per lane.
template <int LANES, int H, class T>
__device__ __forceinline__ T group_total(const T (&v)[H]) {
    static_assert(H == 1 || H == 2, "eight lanes' sums on eight or four lanes");
    const T t = group_sum(v[0], LANES);
    if constexpr (H == 1) return t;
    else return t + group_sum(v[1], LANES);
}

// G~ = L~ a~ after the group reduction of a~ (dimensionless).
template <int D, class T, int LANES, int H, class U>
__device__ __forceinline__ void group_gradient(const T (&L2)[Dims<D>::nL], const U (&a1)[D][H], T (&Gt)[D]) {
    T at[D];
#pragma unroll
    for (int a = 0; a < D; ++a) at[a] = T(group_total<LANES>(a1[a]));
#pragma unroll
    for (int a = 0; a < D; ++a) {
        T t = T(0);
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const int p = sym_index<D>(a, c);
            t += (a == c ? L2[p] : T(0.5) * L2[p]) * at[c];
        }
        Gt[a] = t;
    }
}

template <int D, class T, class S>
__device__ __forceinline__ void load_L(const ApplyArgs<S>& A, int64_t ii, T (&L2)[Dims<D>::nL]) {
#pragma unroll
    for (int p = 0; p < Dims<D>::nL; ++p) {
        const T v = T(A.state[(int64_t)p * A.n + ii]);
        L2[p] = (pair_a<D>(p) == pair_b<D>(p)) ? v : T(2) * v;
    }
}

// out row o of particle i: P_o [a~; s~] + W_o G~ / R.
template <int D, class T, class S>
__device__ __forceinline__ double out_row(const ApplyArgs<S>& A, int64_t i, int o, const T* acc, const T* Gt) {
    using Dm = Dims<D>;
    constexpr int nL = Dm::nL, nk = Dm::nk;
    const int64_t n = A.n;
    const S* P = A.state + (int64_t)(nL + o * nk) * n + i;
    const S* Wr = A.state + (int64_t)(nL + A.nrows * nk + o * D) * n + i;
    T v = T(0);
#pragma unroll
    for (int c = 0; c < nk; ++c) v += T(P[(int64_t)c * n]) * acc[c];
    T lin = T(0);
#pragma unroll
    for (int a = 0; a < D; ++a) lin += T(Wr[(int64_t)a * n]) * Gt[a];
    return (double)v + (double)lin * A.invR;
}

// What a launch does with the first-pass gradient G~: nothing, read it
// (FP64 form: the first pass is skipped) or write it.  Separate
// instantiations, so that a form without the gradient pays no registers for it.
// kLap is the matrix of the pressure system: one field, the Laplacian row
// alone (Dirichlet rows: the field), one number per particle.  The row's
// coefficients are staged in LDS with the window, in the place of the sums,
// and every lane contracts its own partial sums with them: one group sum
// instead of one per sum, and neither the barrier nor the wait for the state
// at the end of the work-group.  1,048,352 particles in 3-D (state of the
// Laplacian and PZ rows): 0.50 -> 0.46 ms, 524,288 in 2-D 0.053 -> 0.050 ms;
// bound by FP64 VALU issue (69%) and the latency of the staging.
enum { kGNone = 0, kGIn = 1, kGOut = 2, kLap = 3 };

// A chunk whose window exceeds the LDS capacity: the same two passes with
// every record read from the memory hierarchy.
template <int D, int KERNEL, class T, class S, int C, int GM>
__device__ __forceinline__ void apply_chunk_global(const ApplyArgs<S>& A, const WindowT<D>& w, int64_t p0,
                                                int64_t p1) {
    constexpr int nk = Dims<D>::nk, kLanes = ApplyCfg<T, C>::lanes, kH = kParts<T, kLanes>;
    const int64_t n = A.n;
    const int lane = threadIdx.x % kLanes;
    const int64_t i = p0 + threadIdx.x / kLanes;
    if (i >= p1) return;   // whole groups leave together
    const T invR = T(A.invR);
    const double ps = Scaled<T>::value ? A.invR : 1.0;   // position scale
    double xi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) xi[a] = a < D ? A.pos[a * n + i] * ps : 0.0;
    T L2[Dims<D>::nL];
    load_L<D, T, S>(A, i, L2);
    const int64_t rb = A.row_ptr[i], re = A.row_ptr[i + 1];
    for (int f = 0; f < A.nf; ++f) {
        const double* ph = A.phi + (int64_t)f * n;
        const double phi_i = ph[i];
        auto fetch = [&](int t, double4& q, T& v) {
            const int64_t j = window_global<D>(w, t);
            q = make_double4(A.pos[j] * ps, A.pos[n + j] * ps, D == 3 ? A.pos[2 * n + j] * ps : 0.0, ph[j]);
            v = T(A.vol[j]);
        };
        T a1[D][kH], Gt[D];
#pragma unroll
        for (int a = 0; a < D; ++a)
#pragma unroll
            for (int h = 0; h < kH; ++h) a1[a][h] = T(0);
        auto first = [&](int64_t e, int h) {
            double4 q;
            T vj, r[D], q2, vc, iq4;
            double dx[D];
            fetch(A.col16[e], q, vj);
            // (the short classes weigh as with the window in LDS: where a chunk's
            // records are read from does not show in the mixed form's results; the
            // FP64 form's first pass is in FP32 there and in FP64 here)
            if constexpr (C == kLongRows) pair_geom<D, KERNEL, T>(q, vj, xi, invR, dx, r, q2, vc);
            else pair_geom<D, KERNEL, T, Scaled<T>::value>(q, vj, xi, invR, dx, r, q2, vc, &iq4);
            const T wgt = vc * T(q.w - phi_i);
#pragma unroll
            for (int a = 0; a < D; ++a) a1[a][h] += wgt * r[a];
        };
        for (int64_t e = rb + lane; e < re; e += kH * kLanes)
#pragma unroll
            for (int h = 0; h < kH; ++h)
                if (e + h * kLanes < re) first(e + h * kLanes, h);
        group_gradient<D, T, kLanes>(L2, a1, Gt);
        if (GM == kGOut && lane == 0) {
#pragma unroll
            for (int a = 0; a < D; ++a) A.g_out[((int64_t)f * D + a) * n + i] = (float)Gt[a];
        }
        double Gp[D];
#pragma unroll
        for (int a = 0; a < D; ++a) Gp[a] = Scaled<T>::value ? (double)Gt[a] : (double)Gt[a] * A.invR;
        T part[nk][kH], acc[nk];
#pragma unroll
        for (int c = 0; c < nk; ++c)
#pragma unroll
            for (int h = 0; h < kH; ++h) part[c][h] = T(0);
        auto second = [&](int64_t e, int h) {
            double4 q;
            T vj, r[D], q2, vc;
            double dx[D];
            fetch(A.col16[e], q, vj);
            T iq4;
            pair_geom<D, KERNEL, T, true>(q, vj, xi, invR, dx, r, q2, vc, &iq4);
            double psi = q.w - phi_i;
#pragma unroll
            for (int a = 0; a < D; ++a) psi -= dx[a] * Gp[a];
            pair_sums<D, T, kH>(r, vc * iq4, vc, T(psi), L2, part, h);
        };
        for (int64_t e = rb + lane; e < re; e += kH * kLanes)
#pragma unroll
            for (int h = 0; h < kH; ++h)
                if (e + h * kLanes < re) second(e + h * kLanes, h);
#pragma unroll
        for (int c = 0; c < nk; ++c) acc[c] = group_total<kLanes>(part[c]);
        if constexpr (GM == kLap) {
            if (lane == 0)
                A.out[i] = A.dirichlet && A.dirichlet[i] ? phi_i : out_row<D, T, S>(A, i, A.lap_row, acc, Gt);
        } else {
            for (int o = lane; o < A.nrows; o += kLanes)
                A.out[((int64_t)f * n + i) * A.nrows + o] = out_row<D, T, S>(A, i, o, acc, Gt);
        }
    }
}

// GM (kGNone, kGIn, kGOut): what the launch does with G~; kLap: the system form.
template <int D, int KERNEL, class T, class S, int C, int GM>
__global__ __launch_bounds__((kChunk * ApplyCfg<T, C>::lanes), (ApplyCfg<T, C>::waves)) void k_apply(ApplyArgs<S> A) {
    constexpr bool GIN = GM == kGIn, GOUT = GM == kGOut, LAP = GM == kLap;
    static_assert(!GIN || !Scaled<T>::value, "only the FP64 form takes a given gradient");
    using Dm = Dims<D>;
    using Cfg = ApplyCfg<T, C>;
    constexpr int nk = Dm::nk, kS = Cfg::slots, kW = Cfg::win, kColCap = Cfg::cols;
    constexpr int kLanes = Cfg::lanes, kThreads = kChunk * kLanes;   // one chunk per work-group
    constexpr int kH = kParts<T, kLanes>;   // partial sums per lane
    static_assert(kS % kH == 0, "the entries past the slots start at part 0");
    constexpr int kColBlocks = kColCap ? (kColCap / 8 + kThreads - 1) / kThreads : 1;   // 16-byte blocks per thread
    __shared__ double4 sd[kW];
    __shared__ T sv[kW];
    __shared__ uint4 scol4[kColCap ? kColCap / 8 : 1];
    // the particles' sums and G~ for the epilogue (LAP: the Laplacian row's coefficients)
    __shared__ T sacc[LAP ? nk + D : kChunk][LAP ? kChunk : nk + D];
    __shared__ WindowT<D> w;
    uint32_t b;
    if (!chunk_of_block(A.nchunks, b)) return;   // uniform over the work-group
    const int64_t n = A.n;
    const int64_t p0 = A.cstart[b], p1 = A.cstart[b + 1];
    if (threadIdx.x < kWave) {
        if (A.cwin) window_load<D>(A.cwin, b, w);
        else chunk_window_wave<D>(A.g, A.cs, A.cinfo[b], w);
    }
    // per-particle data, requested while the window is formed
    const int lane = threadIdx.x % kLanes;
    const int pl = threadIdx.x / kLanes;
    const int64_t i = p0 + pl;
    const bool valid = i < p1;
    const int64_t ii = valid ? i : p0;
    const double ps = Scaled<T>::value ? A.invR : 1.0;   // position scale
    double xi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) xi[a] = a < D ? A.pos[a * n + ii] * ps : 0.0;
    T L2[Dm::nL];
    load_L<D, T, S>(A, ii, L2);
    const int64_t rb = valid ? A.row_ptr[ii] : 0, re = valid ? A.row_ptr[ii + 1] : 0;
    // the chunk's row entries [cb, ce), staged from the 16-byte aligned cb8
    const int64_t cb = A.row_ptr[p0], ce = A.row_ptr[p1], nnz = A.row_ptr[n];
    const int64_t cb8 = cb & ~int64_t(7);
    const bool col_lds = kColCap && ce - cb8 <= kColCap;
    __syncthreads();
    const int W = __builtin_amdgcn_readfirstlane(w.off[w.nr]);
    if (W > kW) {
        apply_chunk_global<D, KERNEL, T, S, C, GM>(A, w, p0, p1);
        return;
    }
    // stage the window records and the chunk's row entries, in batches of
    // loads that are all issued before the batch's first LDS store
    {
        constexpr int kRep = (kW + kThreads - 1) / kThreads;
        constexpr int kBatch = kRep < 4 ? kRep : 4;
        const double* ph = A.phi;
        if constexpr (LAP) {   // P_lap and W_lap: nk + D rows of the state
            constexpr int kPer = kThreads / kChunk, kRows = nk + D;
            const int q = threadIdx.x % kChunk;
            if (p0 + q < p1) {
#pragma unroll
                for (int k = 0; k < (kRows + kPer - 1) / kPer; ++k) {
                    const int c = threadIdx.x / kChunk + k * kPer;
                    if (c < kRows)
                        sacc[c][q] = T(A.state[(int64_t)(c < nk ? Dm::nL + A.lap_row * nk + c
                                                               : Dm::nL + A.nrows * nk + A.lap_row * D + c - nk) * n +
                                               p0 + q]);
                }
            }
        }
        uint4 cv[kColBlocks];
        if (col_lds) {
#pragma unroll
            for (int k = 0; k < kColBlocks; ++k) {
                const int blk = threadIdx.x + k * kThreads;
                const int64_t base = cb8 + 8 * (int64_t)blk;
                if (base < ce) {
                    if (base + 8 <= nnz) {
                        cv[k] = *reinterpret_cast<const uint4*>(A.col16 + base);
                    } else {   // the last block of the array: entry by entry
                        uint32_t h[4] = {0u, 0u, 0u, 0u};
                        for (int u = 0; u < 8 && base + u < nnz; ++u)
                            h[u / 2] |= (uint32_t)A.col16[base + u] << (16 * (u % 2));
                        cv[k] = make_uint4(h[0], h[1], h[2], h[3]);
                    }
                }
            }
        }
#pragma unroll
        for (int k0 = 0; k0 < kRep; k0 += kBatch) {
            double4 q[kBatch];
            T v[kBatch];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                const int t = threadIdx.x + (k0 + k) * kThreads;
                if (t < W) {   // lanes past the window load nothing (whole waves skip)
                    const int64_t j = window_global<D>(w, t);
                    q[k] = make_double4(A.pos[j] * ps, A.pos[n + j] * ps, D == 3 ? A.pos[2 * n + j] * ps : 0.0,
                                        ph[j]);
                    v[k] = T(A.vol[j]);
                }
            }
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                const int t = threadIdx.x + (k0 + k) * kThreads;
                if (t < W) {
                    sd[t] = q[k];
                    sv[t] = v[k];
                }
            }
        }
        if (col_lds) {
#pragma unroll
            for (int k = 0; k < kColBlocks; ++k) {
                const int blk = threadIdx.x + k * kThreads;
                if (cb8 + 8 * (int64_t)blk < ce) scol4[blk] = cv[k];
            }
        }
    }
    __syncthreads();
    // register slots: entry rb + lane + kLanes s; an empty slot repeats the
    // row's first entry (offset 0 for an empty row) and is masked out
    const uint16_t* scol = reinterpret_cast<const uint16_t*>(scol4);
    auto col_at = [&](int64_t e) -> int {
        return dcheck(col_lds ? (int)scol[e - cb8] : (int)A.col16[e], W, kChkWindow);
    };
    // (two 16-bit offsets per register)
    uint32_t cpk[(kS + 1) / 2];
    int nslot = 0;
    {
        const uint32_t first = re > rb ? (uint32_t)col_at(rb) : 0u;
        const int len = (int)(re - rb);   // 32-bit row-local indices: one LDS base, immediate offsets
        const uint16_t* srow = scol + (col_lds ? (int)(rb - cb8) : 0) + lane;
#pragma unroll
        for (int s = 0; s < kS; ++s) {
            const int idx = lane + kLanes * s;
            const bool in = idx < len;
            const uint32_t c = in ? (col_lds ? (uint32_t)srow[kLanes * s] : (uint32_t)A.col16[rb + idx]) : first;
            nslot += in ? 1 : 0;
            if (s % 2 == 0) cpk[s / 2] = c;
            else cpk[s / 2] |= c << 16;
        }
    }
    auto cols = [&](int s) -> int { return dcheck((int)((cpk[s / 2] >> (16 * (s % 2))) & 0xffffu), W, kChkWindow); };
    const int64_t tail = rb + (int64_t)kLanes * kS;
    const T invR = T(A.invR);
    for (int f = 0; f < A.nf; ++f) {
        const double* ph = A.phi + (int64_t)f * n;
        if (f > 0) {
            // every read of sd happened before the epilogue's barrier
            for (int t = threadIdx.x; t < W; t += kThreads) sd[t].w = ph[window_global<D>(w, t)];
            __syncthreads();
        }
        const double phi_i = ph[ii];
        // pass 1: first-order sums and G~ = L~ a~, in FP32 for both forms.  G
        // only sets the residual psi of pass 2; out = P [a; s](psi) + W G
        // holds for any G, so an FP32 G leaves the FP64 form's sums FP64 and
        // its result as accurate (psi keeps a linear part of relative size
        // 1e-7, which the operator reproduces exactly).
        float a1[D][kH];
        T Gt[D];
#pragma unroll
        for (int a = 0; a < D; ++a)
#pragma unroll
            for (int h = 0; h < kH; ++h) a1[a][h] = 0.0f;
        const float invRf = (float)A.invR;
        // The mixed form keeps each register slot's V_j c~ and V_j c~ / q^4
        // from pass 1, so pass 2 forms neither (the FP64 form needs its own
        // FP64 values).
        float vcs[kS], vqs[kS];
        auto term1 = [&](const double4& q, T vj, bool use, int h, float& vq) -> float {
            if constexpr (Scaled<T>::value) {
                double dx[D];
                T r[D], q2, vc, iq4;
                pair_geom<D, KERNEL, T, true>(q, vj, xi, invR, dx, r, q2, vc, &iq4, use);
                vq = vc * iq4;
                const T wgt = vc * T(q.w - phi_i);
#pragma unroll
                for (int a = 0; a < D; ++a) a1[a][h] += wgt * r[a];
                return vc;
            } else {
                float r[D], q2 = 0.0f;
                r[0] = (float)(q.x - xi[0]) * invRf;
                r[1] = (float)(q.y - xi[1]) * invRf;
                if (D == 3) r[D - 1] = (float)(q.z - xi[2]) * invRf;
#pragma unroll
                for (int a = 0; a < D; ++a) q2 += r[a] * r[a];
                q2 = use ? q2 : 4.0f;
                const float vc = (float)vj * kernel_shape<KERNEL>(vsqrt(q2));
                const float wgt = vc * (float)(q.w - phi_i);
#pragma unroll
                for (int a = 0; a < D; ++a) a1[a][h] += wgt * r[a];
                vq = 0.0f;
                return 0.0f;
            }
        };
        // The FP64 form given G~ (a mixed call's first pass on the same field
        // and geometry) skips its own: any G gives the same result up to the
        // rounding of psi.
        if constexpr (GIN) {
#pragma unroll
            for (int a = 0; a < D; ++a) Gt[a] = T(A.g_in[((int64_t)f * D + a) * n + ii]);
        } else {
            // software pipeline: the record of slot s + 1 is read while slot s
            // is summed (the scheduling barriers keep the compiler from
            // hoisting every slot's read, which would exhaust the registers)
            double4 qn = sd[cols(0)];
            T vn = sv[cols(0)];
#pragma unroll
            for (int s = 0; s < kS; ++s) {
                const double4 q = qn;
                const T vj = vn;
                if (s + 1 < kS) {
                    qn = sd[cols(s + 1)];
                    vn = sv[cols(s + 1)];
                }
                __builtin_amdgcn_sched_barrier(0);
                vcs[s] = term1(q, vj, s < nslot, s % kH, vqs[s]);
                __builtin_amdgcn_sched_barrier(0);
            }
            for (int64_t e0 = tail + lane; e0 < re; e0 += kH * kLanes) {
#pragma unroll
                for (int h = 0; h < kH; ++h) {
                    const int64_t e = e0 + h * kLanes;
                    if (e < re) {
                        const int t = col_at(e);
                        float vq_;
                        term1(sd[t], sv[t], true, h, vq_);
                    }
                }
            }
            group_gradient<D, T, kLanes>(L2, a1, Gt);
        }
        double Gp[D];
#pragma unroll
        for (int a = 0; a < D; ++a) Gp[a] = Scaled<T>::value ? (double)Gt[a] : (double)Gt[a] * A.invR;
        // G~ waits for the epilogue in LDS, not in registers
        if (!LAP && lane == 0) {
#pragma unroll
            for (int a = 0; a < D; ++a) sacc[pl][nk + a] = Gt[a];
        }
        // pass 2: sums of the residual psi_ij = phi_ij - (x_j - x_i) . G.
        // The empty asm makes the packed offsets opaque, so the record
        // addresses are recomputed here instead of being kept live from pass 1.
#pragma unroll
        for (int k = 0; k < (kS + 1) / 2; ++k) asm volatile("" : "+v"(cpk[k]));
        T part[nk][kH];
#pragma unroll
        for (int c = 0; c < nk; ++c)
#pragma unroll
            for (int h = 0; h < kH; ++h) part[c][h] = T(0);
        auto term2 = [&](const double4& q, T vj, bool use, int s, int h) {
            double dx[D];
            T r[D], q2, vc;
            T iq4;
            if (Scaled<T>::value && s >= 0) {   // V c~ and V c~ / q^4 from pass 1
#pragma unroll
                for (int a = 0; a < D; ++a) {
                    dx[a] = (a == 0 ? q.x : a == 1 ? q.y : q.z) - xi[a];
                    r[a] = T(dx[a]);
                }
                vc = vcs[s];
                double psi = q.w - phi_i;
#pragma unroll
                for (int a = 0; a < D; ++a) psi -= dx[a] * Gp[a];
                pair_sums<D, T, kH>(r, T(vqs[s]), vc, T(psi), L2, part, h);
                return;
            } else {
                pair_geom<D, KERNEL, T, true>(q, vj, xi, invR, dx, r, q2, vc, &iq4, use);
            }
            double psi = q.w - phi_i;
#pragma unroll
            for (int a = 0; a < D; ++a) psi -= dx[a] * Gp[a];
            pair_sums<D, T, kH>(r, vc * iq4, vc, T(psi), L2, part, h);
        };
        double4 qn = sd[cols(0)];
        T vn = sv[cols(0)];
#pragma unroll
        for (int s = 0; s < kS; ++s) {
            const double4 q = qn;
            const T vj = vn;
            if (s + 1 < kS) {
                qn = sd[cols(s + 1)];
                vn = sv[cols(s + 1)];
            }
            __builtin_amdgcn_sched_barrier(0);
            term2(q, vj, s < nslot, s, s % kH);
            __builtin_amdgcn_sched_barrier(0);
        }
        for (int64_t e0 = tail + lane; e0 < re; e0 += kH * kLanes) {
#pragma unroll
            for (int h = 0; h < kH; ++h) {
                const int64_t e = e0 + h * kLanes;
                if (e < re) {
                    const int t = col_at(e);
                    term2(sd[t], sv[t], true, -1, h);
                }
            }
        }
        if constexpr (LAP) {
            // the lane's sums against the Laplacian row, then one group sum
            T v = T(0);
#pragma unroll
            for (int c = 0; c < nk; ++c) v += sacc[c][pl] * part[c][0];
            v = group_sum(v, kLanes);
            if (lane == 0 && valid) {
                double lin = 0.0;
#pragma unroll
                for (int a = 0; a < D; ++a) lin += sacc[nk + a][pl] * Gp[a];
                A.out[i] = A.dirichlet && A.dirichlet[i] ? phi_i : (double)v + lin;
            }
            return;
        }
        // epilogue: the group's sums to LDS, then one thread per (row, particle)
        T acc[nk];
#pragma unroll
        for (int c = 0; c < nk; ++c) acc[c] = group_total<kLanes>(part[c]);
        if (lane == 0) {
#pragma unroll
            for (int c = 0; c < nk; ++c) sacc[pl][c] = acc[c];
        }
        __syncthreads();
        {
            const int q = threadIdx.x % kChunk;
            const int64_t iq = p0 + q;
            // the row index made opaque here, so that the state addresses are
            // formed now rather than kept in registers (or spilled) from the
            // start of the kernel
            int o0 = threadIdx.x / kChunk;
            asm volatile("" : "+v"(o0));
            if (iq < p1) {
                for (int o = o0; o < A.nrows; o += kThreads / kChunk)
                    A.out[((int64_t)f * n + iq) * A.nrows + o] =
                        out_row<D, T, S>(A, iq, o, &sacc[q][0], &sacc[q][nk]);
                if (GOUT && threadIdx.x < kChunk)
#pragma unroll
                    for (int a = 0; a < D; ++a) A.g_out[((int64_t)f * D + a) * n + iq] = (float)sacc[q][nk + a];
            }
        }
    }
}

template <int D, int KERNEL, class T, class S, int C>
static int launch_apply(const ApplyArgs<S>& a, int64_t cap, hipStream_t s) {
    const dim3 grid((unsigned)cap), block(kChunk * ApplyCfg<T, C>::lanes);
    const char* name = sizeof(T) == 4 ? "k_apply (mixed)" : "k_apply (fp64)";
    if constexpr (!Scaled<T>::value) {
        if (a.g_in) {
            VCT_LAUNCH("k_apply (fp64, given G)", (k_apply<D, KERNEL, T, S, C, kGIn>), grid, block, 0, s, a);
            VCT_LAUNCH_CHECK();
            return VCT_OK;
        }
    }
    if (a.g_out)
        VCT_LAUNCH(name, (k_apply<D, KERNEL, T, S, C, kGOut>), grid, block, 0, s, a);
    else
        VCT_LAUNCH(name, (k_apply<D, KERNEL, T, S, C, kGNone>), grid, block, 0, s, a);
    VCT_LAUNCH_CHECK();
    return VCT_OK;
}

// the system form (FP64, one field): out [n] = the Laplacian row, Dirichlet
// rows the field
template <int D, int KERNEL>
static int launch_lap(const ApplyArgs<double>& a, int64_t mean, int64_t cap, hipStream_t s) {
    constexpr int kShort = D == 2 ? kShort2 : kShort3;
    if (mean <= short_row<D>())
        VCT_LAUNCH("k_apply (fp64)", (k_apply<D, KERNEL, double, double, kShort, kLap>), dim3((unsigned)cap),
                   dim3(kChunk * ApplyCfg<double, kShort>::lanes), 0, s, a);
    else
        VCT_LAUNCH("k_apply (fp64)", (k_apply<D, KERNEL, double, double, kLongRows, kLap>), dim3((unsigned)cap),
                   dim3(kChunk * ApplyCfg<double, kLongRows>::lanes), 0, s, a);
    VCT_LAUNCH_CHECK();
    return VCT_OK;
}

template <int D, int KERNEL, class T, class S>
static int launch_class(const ApplyArgs<S>& a, int64_t mean, int64_t cap, hipStream_t s) {
    constexpr int kShort = D == 2 ? kShort2 : kShort3;
    if (mean <= short_row<D>()) return launch_apply<D, KERNEL, T, S, kShort>(a, cap, s);
    return launch_apply<D, KERNEL, T, S, kLongRows>(a, cap, s);
}

template <class T, class S>
static int dispatch(const vct_nlist* nl, int kernel, const ApplyArgs<S>& a, int64_t cap, hipStream_t s) {
    const int64_t mean = mean_row(nl);
    if (nl->dim == 2)
        return kernel == VCT_KERNEL_WENDLAND_C2 ? launch_class<2, VCT_KERNEL_WENDLAND_C2, T, S>(a, mean, cap, s)
                                                : launch_class<2, VCT_KERNEL_CUBIC_SPLINE, T, S>(a, mean, cap, s);
    return kernel == VCT_KERNEL_WENDLAND_C2 ? launch_class<3, VCT_KERNEL_WENDLAND_C2, T, S>(a, mean, cap, s)
                                            : launch_class<3, VCT_KERNEL_CUBIC_SPLINE, T, S>(a, mean, cap, s);
}

template <class S>
static ApplyArgs<S> make_args(const vct_nlist* nl, const Grid& g, int nf, const double* phi, const double* pos,
                              const double* vol, const S* state, uint32_t mask, double* out) {
    const int dim = nl->dim;
    const int64_t ncols = dim == 3 ? g.nc[0] * g.nc[1] : g.nc[0];
    ApplyArgs<S> a;
    a.n = nl->n;
    a.nf = nf;
    a.nrows = n_out_rows(dim, mask);
    a.invR = 1.0 / nl->R;
    a.g = g;
    a.phi = phi;
    a.pos = pos;
    a.vol = vol;
    a.row_ptr = nl->row_ptr;
    a.col16 = nl->col16;
    a.cs = nl->cell_start;
    a.cstart = nl->chunk_start;
    a.cinfo = reinterpret_cast<const int4*>(nl->chunk_info); a.cwin = nl->chunk_win;
    a.nchunks = nl->chunk_off + ncols;
    a.state = state;
    a.out = out;
    a.g_out = nullptr;
    a.g_in = nullptr;
    a.lap_row = 0;
    a.dirichlet = nullptr;
    return a;
}

// The pressure system's matrix times x (arguments checked by the solver).
int apply_lap(const vct_nlist* nl, const Grid& g, const double* x, const double* pos, const double* vol, int kernel,
              const double* state, uint32_t mask, const uint8_t* dirichlet, double* out, hipStream_t s) {
    auto a = make_args(nl, g, 1, x, pos, vol, state, mask, out);
    a.lap_row = group_row(nl->dim, mask, VCT_OUT_LAP);
    a.dirichlet = dirichlet;
    const int64_t ncols = nl->dim == 3 ? g.nc[0] * g.nc[1] : g.nc[0], cap = ncols + nl->n / kChunk + 1;
    const int64_t mean = mean_row(nl);
    if (nl->dim == 2)
        return kernel == VCT_KERNEL_WENDLAND_C2 ? launch_lap<2, VCT_KERNEL_WENDLAND_C2>(a, mean, cap, s)
                                                : launch_lap<2, VCT_KERNEL_CUBIC_SPLINE>(a, mean, cap, s);
    return kernel == VCT_KERNEL_WENDLAND_C2 ? launch_lap<3, VCT_KERNEL_WENDLAND_C2>(a, mean, cap, s)
                                            : launch_lap<3, VCT_KERNEL_CUBIC_SPLINE>(a, mean, cap, s);
}

VCT_CHECKS_TU(checks_apply)

}  // namespace vct

using namespace vct;

static int apply_ops(const vct_nlist* nl, int nf, const double* phi_sorted, const double* pos_sorted,
                     const double* vol_sorted, int kernel, const void* state, uint32_t out_mask, int precision,
                     double* out, float* g_out, const float* g_in, void* stream) {
    Grid g;
    int st = nlist_check(nl, g);
    if (st) return st;
    if (nf < 1 || !mask_valid(out_mask) ||
        (kernel != VCT_KERNEL_WENDLAND_C2 && kernel != VCT_KERNEL_CUBIC_SPLINE) ||
        (precision != VCT_FP64 && precision != VCT_MIXED && precision != VCT_MIXED_S64))
        return VCT_E_ARG;
    const int64_t n = nl->n;
    if (n == 0) return VCT_OK;
    if (!phi_sorted || !pos_sorted || !vol_sorted || !nl->col16 || !state || !out) return VCT_E_ARG;
    const int dim = nl->dim;
    const int64_t ncols = dim == 3 ? g.nc[0] * g.nc[1] : g.nc[0];
    const int64_t cap = ncols + n / kChunk + 1;   // upper bound of the chunk count
    hipStream_t s = as_stream(stream);
    switch (precision) {
    case VCT_FP64: {
        auto a = make_args(nl, g, nf, phi_sorted, pos_sorted, vol_sorted, static_cast<const double*>(state), out_mask,
                           out);
        a.g_out = g_out;
        a.g_in = g_in;
        return dispatch<double, double>(nl, kernel, a, cap, s);
    }
    case VCT_MIXED: {
        auto a = make_args(nl, g, nf, phi_sorted, pos_sorted, vol_sorted, static_cast<const float*>(state), out_mask,
                           out);
        a.g_out = g_out;
        return dispatch<float, float>(nl, kernel, a, cap, s);
    }
    default: {
        auto a = make_args(nl, g, nf, phi_sorted, pos_sorted, vol_sorted, static_cast<const double*>(state), out_mask,
                           out);
        a.g_out = g_out;
        return dispatch<float, double>(nl, kernel, a, cap, s);
    }
    }
}

extern "C" int vct_apply_ops(const vct_nlist* nl, int nf, const double* phi_sorted, const double* pos_sorted,
                             const double* vol_sorted, int kernel, const void* state, uint32_t out_mask,
                             int precision, double* out, void* stream) {
    VCT_API_RANGE("vct_apply_ops");
    return apply_ops(nl, nf, phi_sorted, pos_sorted, vol_sorted, kernel, state, out_mask, precision, out, nullptr,
                     nullptr, stream);
}

extern "C" int vct_apply_ops_ex(const vct_nlist* nl, int nf, const double* phi_sorted, const double* pos_sorted,
                                const double* vol_sorted, int kernel, const void* state, uint32_t out_mask,
                                int precision, double* out, float* g_out, const float* g_in, void* stream) {
    VCT_API_RANGE("vct_apply_ops_ex");
    if (g_out && g_in) return VCT_E_ARG;   // distinct roles: one call writes G~, a later one reads it
    return apply_ops(nl, nf, phi_sorted, pos_sorted, vol_sorted, kernel, state, out_mask, precision, out, g_out,
                     g_in, stream);
}
