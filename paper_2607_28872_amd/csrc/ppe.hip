// Pressure step of the projection method through the vertical coordinate
// transformation (paper Sec. 3.3, Eqs. VCT_ppe, VCT_ppe_w, VCT_predictor):
//   right-hand side  rhs_i = rho/dt div_i + gamma (rho jr_i - dens_i) / dt^2
//                    with div_i = sum_{I,K} J_IK <d v_I / d x^_K>^(1)_i (the
//                    physical divergence through the J-mapped first-order
//                    projected gradients, Eqs. div_1st and jacobi), dens_i the
//                    projected-space kernel-sum density and jr_i = Jbar_i / J_i;
//   pressure solve   c_trans . <D^ p>_i = rhs_i on ordinary rows, p_i = rhs_i on
//                    Dirichlet rows, by BiCGSTAB with the SPH(2) Laplacian of
//                    vct_apply_ops as the operator, its coefficients kept for the
//                    call where they fit;
//   corrector        v_i = v*_i - dt/rho J <grad^ p>^(1)_i (Eqs. gra_1st, grad_VCT).
#include <string.h>

#include "common.h"
#include "lapw.h"
#include "map_dev.h"
#include "tiles.h"

namespace vct {

int nlist_check(const vct_nlist* nl, Grid& g);
int apply_lap(const vct_nlist* nl, const Grid& g, const double* x, const double* pos, const double* vol, int kernel,
              const double* state, uint32_t mask, const uint8_t* dirichlet, double* out, hipStream_t s);

struct PpeArgs {
    int64_t n;
    double invR, R;
    Grid g;
    const double* pos;
    const double* vol;
    const double* state;
    int lap_row, nrows;
    const int64_t* row_ptr;
    const uint16_t* col16;
    const int64_t* cs;
    const int32_t* cstart;
    const int4* cinfo;
    const int32_t* cwin;
    const int64_t* nchunks;
    const double* f;          // [nc][n] fields (velocity components, or the pressure)
    const double* vstar;      // [dim][n] (corrector)
    const double* jr;         // [n] or NULL
    const uint8_t* dirichlet; // [n] or NULL
    const double* pbc;        // [n] or NULL
    double rho, dt, gamma;
    double* rhs;
    double* div;
    double* dens;
    double* vout;             // [dim][n] (corrector)
    double* dinv;             // [n] (Jacobi diagonal)
    double* wmat;             // [entries] the matrix's coefficients W_ij, or NULL: not kept
};

// Normalised kernel value w(q R) (unit integral): Wendland C2
// C (1 - q)^4 (1 + 4 q), C = 7 / (pi R^2) in 2-D and 21 / (2 pi R^3) in 3-D;
// cubic spline of Sec. 3.1 with l = R / 2, s = 2 q.
template <int D, int KERNEL>
__device__ __forceinline__ double kernel_value(double q, double R) {
    if (KERNEL == VCT_KERNEL_WENDLAND_C2) {
        const double C = D == 2 ? 7.0 / (M_PI * R * R) : 21.0 / (2.0 * M_PI * R * R * R);
        double t = 1.0 - q;
        t = t > 0.0 ? t : 0.0;
        const double t2 = t * t;
        return C * t2 * t2 * (1.0 + 4.0 * q);
    } else {
        const double l = 0.5 * R;
        const double ad = D == 2 ? 10.0 / (7.0 * M_PI * l * l) : 1.0 / (M_PI * l * l * l);
        const double s = 2.0 * q;
        double t = 2.0 - s;
        t = t > 0.0 ? t : 0.0;
        return s <= 1.0 ? ad * (1.0 - 1.5 * s * s + 0.75 * s * s * s) : ad * 0.25 * t * t * t;
    }
}

// One record of a first-order sweep: position and volume, and the fields.
template <int NC> struct FirstRec {
    double4 q;
    double f[NC];
};

// One chunk per work-group, RowShape<C>::lanes lanes per particle: the
// first-order sums a_c = sum_j V_j c~ f_c,ij r~_ij of nc fields (and, MODE 0,
// the kernel sum), then the particles' epilogue:
//   MODE 0: right-hand side (nc = dim velocity components);
//   MODE 1: corrector (nc = 1, the pressure).
// The sums go through LDS (in the place of the window) to the first wave, one
// particle per lane, which forms the gradients and the mapping; done by the
// first lane of every group it took every wave the instructions of a whole
// one.  1,048,352 particles in 3-D: right-hand side 0.97 -> 0.47 ms, corrector
// 0.54 -> 0.38 ms; 524,288 in 2-D 0.13 -> 0.050 and 0.13 -> 0.042 ms.
template <int D, int KERNEL, int MODE, int C>
__global__ __launch_bounds__((kChunk * RowShape<C>::lanes), RowShape<C>::waves) void k_ppe_first(PpeArgs A,
                                                                                                MapParams mp) {
    using Dm = Dims<D>;
    using Sh = RowShape<C>;
    constexpr int nL = Dm::nL, kLanes = Sh::lanes, kThreads = kChunk * kLanes, kWin = Sh::win;
    constexpr int NC = MODE == 0 ? D : 1;
    constexpr int kSums = NC * D + (MODE == 0 ? 1 : 0);
    // window records in LDS: position and volume, and the fields
    __shared__ double4 sd[kWin];
    __shared__ double sf[NC][kWin];
    __shared__ WindowT<D> w;
    static_assert(kSums * kChunk * 8 <= kWin * 32, "the sums fit the window buffer");
    uint32_t b;
    if (!chunk_of_block(A.nchunks, b)) return;   // uniform over the work-group
    const int64_t n = A.n;
    const int64_t p0 = A.cstart[b], p1 = A.cstart[b + 1];
    if (threadIdx.x < kWave) {
        if (A.cwin) window_load<D>(A.cwin, b, w);
        else chunk_window_wave<D>(A.g, A.cs, A.cinfo[b], w);
    }
    const int lane = threadIdx.x % kLanes, pl = threadIdx.x / kLanes;
    const int64_t i = p0 + pl;
    const bool valid = i < p1;
    const int64_t ii = valid ? i : p0;
    double xi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) xi[a] = a < D ? A.pos[a * n + ii] : 0.0;
    double fi[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) fi[c] = A.f[(int64_t)c * n + ii];
    const RowSlots<kLanes, Sh::slots> rs(A.col16, valid ? A.row_ptr[ii] : 0, valid ? A.row_ptr[ii + 1] : 0, lane);
    auto record = [&](int t) -> FirstRec<NC> {
        const int64_t j = window_global<D>(w, t);
        FirstRec<NC> z;
        z.q = make_double4(A.pos[j], A.pos[n + j], D == 3 ? A.pos[2 * n + j] : 0.0, A.vol[j]);
#pragma unroll
        for (int c = 0; c < NC; ++c) z.f[c] = A.f[(int64_t)c * n + j];
        return z;
    };
    __syncthreads();
    const int W = __builtin_amdgcn_readfirstlane(w.off[w.nr]);
    const bool in_lds = W <= kWin;
    if (in_lds)
        stage_window<kWin, kThreads>(W, record, [&](int t, const FirstRec<NC>& z) {
            sd[t] = z.q;
#pragma unroll
            for (int c = 0; c < NC; ++c) sf[c][t] = z.f[c];
        });
    __syncthreads();
    double acc[NC][D];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int a = 0; a < D; ++a) acc[c][a] = 0.0;
    double ksum = 0.0;
    sweep_row(rs, A.col16, W, in_lds,
        [&](int t) -> FirstRec<NC> {
            if (!in_lds) return record(t);
            FirstRec<NC> z;
            z.q = sd[t];
#pragma unroll
            for (int c = 0; c < NC; ++c) z.f[c] = sf[c][t];
            return z;
        },
        [&](const FirstRec<NC>& z) {
            const double4& q = z.q;
            double r[D];
            r[0] = (q.x - xi[0]) * A.invR;
            r[1] = (q.y - xi[1]) * A.invR;
            if (D == 3) r[D - 1] = (q.z - xi[2]) * A.invR;
            double q2 = r[0] * r[0];
#pragma unroll
            for (int a = 1; a < D; ++a) q2 = fma(r[a], r[a], q2);
            const double qn = vsqrt(q2);
            const double vc = q.w * kernel_shape<KERNEL>(qn);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const double fij = vc * (z.f[c] - fi[c]);
#pragma unroll
                for (int a = 0; a < D; ++a) acc[c][a] = fma(fij, r[a], acc[c][a]);
            }
            if (MODE == 0) ksum = fma(q.w, kernel_value<D, KERNEL>(qn, A.R), ksum);
        });
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int a = 0; a < D; ++a) acc[c][a] = group_sum(acc[c][a], kLanes);
    if (MODE == 0) ksum = group_sum(ksum, kLanes);
    __syncthreads();   // the window is no longer needed
    double* ssum = reinterpret_cast<double*>(sd);   // [kSums][kChunk]
    if (lane == 0) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int a = 0; a < D; ++a) ssum[(c * D + a) * kChunk + pl] = acc[c][a];
        if (MODE == 0) ssum[NC * D * kChunk + pl] = ksum;
    }
    __syncthreads();
    if (threadIdx.x >= kChunk || p0 + threadIdx.x >= p1) return;
    const int pq = threadIdx.x;
    const int64_t iq = p0 + pq;
    // first-order projected gradients G_c = L~ a_c / R
    double L2[nL];
    bool ok = true;
#pragma unroll
    for (int p = 0; p < nL; ++p) {
        L2[p] = A.state[(int64_t)p * n + iq];
        ok = ok && isfinite(L2[p]);
    }
    double G[NC][3];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        double g[D];
#pragma unroll
        for (int a = 0; a < D; ++a) {
            double t = 0.0;
#pragma unroll
            for (int bb = 0; bb < D; ++bb) t += L2[sym_index<D>(a, bb)] * ssum[(c * D + bb) * kChunk + pq];
            g[a] = t * A.invR;
        }
        // 3-D component order (2-D: x^, 0, z^)
        G[c][0] = g[0];
        G[c][1] = D == 3 ? g[1] : 0.0;
        G[c][2] = g[D - 1];
    }
    // the Jacobian column of z^ at the particle: J = [[1,0,gx],[0,1,gy],[0,0,alpha]]
    const MapCoef<double> mc =
        map_coef_at(mp, iq, A.pos[iq], D == 3 ? A.pos[n + iq] : 0.0, A.pos[(int64_t)(D - 1) * n + iq]);
    const double nanv = __builtin_nan("");
    if (MODE == 0) {
        // physical divergence: sum_I (J grad^ v_I)_I; component I along physical axis I
        const double gxy[2] = {mc.gx, mc.gy};
        double dv = 0.0;
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const int Ip = D == 3 ? c : (c == 0 ? 0 : 2);
            dv += Ip < 2 ? G[c][Ip] + gxy[Ip] * G[c][2] : mc.alpha * G[c][2];
        }
        double wself = kernel_value<D, KERNEL>(0.0, A.R);
        double ds = A.rho * fma(A.vol[iq], wself, ssum[NC * D * kChunk + pq]);
        if (!ok) dv = ds = nanv;
        if (A.div) A.div[iq] = dv;
        if (A.dens) A.dens[iq] = ds;
        const double jri = A.jr ? A.jr[iq] : 1.0;
        const bool dir = A.dirichlet && A.dirichlet[iq];
        A.rhs[iq] = dir ? (A.pbc ? A.pbc[iq] : 0.0)
                        : A.rho / A.dt * dv + A.gamma * (A.rho * jri - ds) / (A.dt * A.dt);
    } else {
        // physical pressure gradient J grad^ p
        const double gp[3] = {G[0][0] + mc.gx * G[0][2], G[0][1] + mc.gy * G[0][2], mc.alpha * G[0][2]};
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const int Ip = D == 3 ? c : (c == 0 ? 0 : 2);
            const double g = ok ? gp[Ip] : nanv;
            A.vout[(int64_t)c * n + iq] = A.vstar[(int64_t)c * n + iq] - A.dt / A.rho * g;
        }
    }
}

// Jacobi diagonal of the pressure system: the coefficient of p_i in row i,
// -sum_j W_ij on ordinary rows, 1 on Dirichlet rows; dinv = its inverse.  With
// wmat the coefficients W_ij are kept for k_ppe_matvec, in row order.  A row
// whose state is not finite (a flagged particle) has NaN for all of them and
// for dinv, so that a row without entries says so too.
// 1,048,352 particles in 3-D 0.42 -> 0.34 ms (0.52 with the coefficients),
// 524,288 in 2-D 0.058 -> 0.033 ms.
template <int D, int KERNEL, int C>
__global__ __launch_bounds__((kChunk * RowShape<C>::lanes), RowShape<C>::waves) void k_ppe_diag(PpeArgs A) {
    using Dm = Dims<D>;
    using Sh = RowShape<C>;
    constexpr int nL = Dm::nL, nk = Dm::nk, kLanes = Sh::lanes, kThreads = kChunk * kLanes, kWin = Sh::win;
    __shared__ double4 sd[kWin];
    __shared__ WindowT<D> w;
    uint32_t b;
    if (!chunk_of_block(A.nchunks, b)) return;   // uniform over the work-group
    const int64_t n = A.n;
    const int64_t p0 = A.cstart[b], p1 = A.cstart[b + 1];
    if (threadIdx.x < kWave) {
        if (A.cwin) window_load<D>(A.cwin, b, w);
        else chunk_window_wave<D>(A.g, A.cs, A.cinfo[b], w);
    }
    const int lane = threadIdx.x % kLanes;
    const int64_t i = p0 + threadIdx.x / kLanes;
    const bool valid = i < p1;
    const int64_t ii = valid ? i : p0;
    double xi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) xi[a] = a < D ? A.pos[a * n + ii] : 0.0;
    double L2[nL], Pl[nk];
#pragma unroll
    for (int p = 0; p < nL; ++p) L2[p] = (pair_a<D>(p) == pair_b<D>(p) ? 1.0 : 2.0) * A.state[(int64_t)p * n + ii];
#pragma unroll
    for (int c = 0; c < nk; ++c) Pl[c] = A.state[(int64_t)(nL + A.lap_row * nk + c) * n + ii];
    double bad = 0.0;   // 0, or NaN where the state (the response to a gradient included) is not finite
#pragma unroll
    for (int p = 0; p < nL; ++p) bad += 0.0 * L2[p];
#pragma unroll
    for (int c = 0; c < nk; ++c) bad += 0.0 * Pl[c];
#pragma unroll
    for (int a = 0; a < D; ++a) bad += 0.0 * A.state[(int64_t)(nL + A.nrows * nk + A.lap_row * D + a) * n + ii];
    L2[0] += bad;
    const RowSlots<kLanes, Sh::slots> rs(A.col16, valid ? A.row_ptr[ii] : 0, valid ? A.row_ptr[ii + 1] : 0, lane);
    auto record = [&](int t) -> double4 {
        const int64_t j = window_global<D>(w, t);
        return make_double4(A.pos[j], A.pos[n + j], D == 3 ? A.pos[2 * n + j] : 0.0, A.vol[j]);
    };
    __syncthreads();
    const int W = __builtin_amdgcn_readfirstlane(w.off[w.nr]);
    const bool in_lds = W <= kWin;
    if (in_lds) stage_window<kWin, kThreads>(W, record, [&](int t, const double4& q) { sd[t] = q; });
    __syncthreads();
    double s = 0.0;
    int64_t e = (valid ? A.row_ptr[ii] : 0) + lane;   // the lane's entries come in order
    sweep_row(rs, A.col16, W, in_lds, [&](int t) -> double4 { return in_lds ? sd[t] : record(t); },
              [&](const double4& q) {
                  const double wij = lap_weight<D, KERNEL>(q, xi, A.invR, L2, Pl);
                  s += wij;
                  if (A.wmat) {
                      A.wmat[e] = wij;
                      e += kLanes;
                  }
              });
    s = group_sum(s, kLanes);
    if (valid && lane == 0) {
        const bool dir = A.dirichlet && A.dirichlet[ii];
        A.dinv[ii] = dir ? 1.0 : 1.0 / (-(s + bad));
    }
}

// The product with the kept matrix: sum_j W_ij (x_j - x_i), on Dirichlet rows
// x_i.  A row without entries takes the NaN of its dinv where its state is not
// finite, as the product that forms the coefficients does.
// The coefficients are read once in row order, all of a lane's before the
// window's values are in LDS.  Bound by that read: 1,048,352 particles in 3-D
// (108M entries of 10 bytes), 0.228 ms, 4.8 TB/s, where forming the coefficients
// in each product takes 0.46 ms; cubic spline 0.143 against 0.316; 2-D, 524,288
// particles, 0.027 against 0.049.  (Non-temporal loads give up the part of the
// matrix that stays in the last-level cache: 0.297; eight waves per SIMD spill:
// 0.35.)
constexpr int kMatRow3 = 128, kMatRow2 = 40;       // entries per particle of the workspace (3-D, 2-D)
constexpr size_t kMatMax = (size_t)16 << 30;       // the largest kept matrix (bytes)
constexpr int kMatIters = 1;                       // iterations from which one is kept
template <int D, int C>
__global__ __launch_bounds__((kChunk * RowShape<C>::lanes), 4) void k_ppe_matvec(PpeArgs A,
                                                                                const double* __restrict__ x,
                                                                                double* __restrict__ out) {
    using Sh = RowShape<C>;
    constexpr int kLanes = Sh::lanes, kThreads = kChunk * kLanes, kSlots = Sh::slots, kWin = D == 3 ? 2048 : 1024;
    __shared__ double sx[kWin];
    __shared__ WindowT<D> w;
    uint32_t b;
    if (!chunk_of_block(A.nchunks, b)) return;   // uniform over the work-group
    const int64_t p0 = A.cstart[b], p1 = A.cstart[b + 1];
    if (threadIdx.x < kWave) {
        if (A.cwin) window_load<D>(A.cwin, b, w);
        else chunk_window_wave<D>(A.g, A.cs, A.cinfo[b], w);
    }
    const int lane = threadIdx.x % kLanes;
    const int64_t i = p0 + threadIdx.x / kLanes;
    const bool valid = i < p1;
    const int64_t ii = valid ? i : p0;
    const double xi = x[ii];
    const int64_t rb = valid ? A.row_ptr[ii] : 0, re = valid ? A.row_ptr[ii + 1] : 0;
    const RowSlots<kLanes, kSlots> rs(A.col16, rb, re, lane);
    const double* wr = A.wmat + rb + lane;
    double wij[kSlots];
#pragma unroll
    for (int s = 0; s < kSlots; ++s) wij[s] = s < rs.n ? wr[kLanes * s] : 0.0;
    __syncthreads();
    const int W = __builtin_amdgcn_readfirstlane(w.off[w.nr]);
    const bool in_lds = W <= kWin;
    auto value = [&](int t) { return x[window_global<D>(w, t)]; };
    if (in_lds) stage_window<kWin, kThreads>(W, value, [&](int t, double v) { sx[t] = v; });
    __syncthreads();
    double sum = 0.0;
    if (in_lds) {
#pragma unroll
        for (int s = 0; s < kSlots; ++s)
            if (s < rs.n) sum = fma(wij[s], sx[rs.at(s, W)] - xi, sum);
    }
    for (int64_t e = in_lds ? rs.tail : rb + lane; e < re; e += kLanes) {
        const int t = dcheck((int)A.col16[e], W, kChkWindow);
        sum = fma(A.wmat[e], (in_lds ? sx[t] : value(t)) - xi, sum);
    }
    sum = group_sum(sum, kLanes);
    if (valid && lane == 0) {
        if (rb == re && A.dinv[ii] != A.dinv[ii]) sum = __builtin_nan("");   // rare: no coefficient carries it
        out[ii] = A.dirichlet && A.dirichlet[ii] ? xi : sum;
    }
}

// ------------------------------------------------------------------ BiCGSTAB

// Vector kernels run a fixed grid (kVBlocks x kVThreads, grid-stride), so each
// dot product is the same fixed-order sum on every run: per thread in index
// order, per wave and work-group in lane and wave order, then the kVBlocks
// partials in order.  Scalars stay on the device.  The kernel that needs a
// scalar sums the partials itself, every work-group the same way, and its first
// work-group writes the state: a launch of its own for each sum, of one
// work-group, took 6 us, three times an iteration.  No kernel writes what it
// reads: the state goes round three copies (p writes the first, s the second, x
// the third), and v, t and x have partials of their own.  Twelve iterations of
// 72,000 particles in 3-D 0.995 -> 0.939 ms, of 27,000 in 2-D 0.580 -> 0.540,
// of 1,048,352 in 3-D 8.17 -> 8.09.
constexpr int kVThreads = 256;
constexpr int kVBlocks = 1024;
constexpr int kVSlots = 3;       // partial sums per launch
constexpr int kVParts = 5;       // of v and the first stage; t; x
constexpr int kPartT = 1, kPartX = 3;

// scalar slots
enum { S_RHO0, S_RHO1, S_ALPHA, S_OMEGA, S_BB, S_RR, S_DONE, S_ITERS, S_STATUS, S_RES, kNScalars };
// status values
enum { ST_RUNNING = 0, ST_CONVERGED = 1, ST_BREAKDOWN = 2, ST_MAXIT = 3 };
// copies of the state: after the sums of x (or the first stage), of v, of t
enum { C_NEXT, C_ALPHA, C_OMEGA, kNStates };

struct BicgVec {
    int64_t n;
    const double* b;
    double *x, *r, *rh, *p, *v, *s, *t, *ph, *sh, *dinv, *part, *sc;
    double tol2;
    int maxit;
};

__device__ __forceinline__ void block_partials(double (&v)[kVSlots], int ns, double* part) {
    __shared__ double red[kVSlots][kVThreads / kWave];
    const int wv = threadIdx.x / kWave, ln = threadIdx.x % kWave;
    for (int k = 0; k < ns; ++k) {
        const double s = group_sum(v[k], kWave);
        if (ln == 0) red[k][wv] = s;
    }
    __syncthreads();
    if ((int)threadIdx.x < ns) {
        double s = 0.0;
        for (int w2 = 0; w2 < kVThreads / kWave; ++w2) s += red[threadIdx.x][w2];
        part[threadIdx.x * kVBlocks + blockIdx.x] = s;
    }
}

// stage 0 (t = A x0): r = b - t, r^ = r, p = v = 0; partials (r^, r), (r, r), (b, b)
__global__ __launch_bounds__(kVThreads) void k_bicg_init(BicgVec V) {
    double acc[kVSlots] = {0.0, 0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * kVThreads + threadIdx.x; i < V.n; i += (int64_t)kVBlocks * kVThreads) {
        const double ri = V.b[i] - V.t[i];
        V.r[i] = ri;
        V.rh[i] = ri;
        V.p[i] = 0.0;
        V.v[i] = 0.0;
        acc[0] += ri * ri;
        acc[1] += ri * ri;
        acc[2] += V.b[i] * V.b[i];
    }
    block_partials(acc, 3, V.part);
}

// The sums of ns partials in the fixed order, for every thread of the
// work-group (THREADS of them).
template <int THREADS>
__device__ __forceinline__ void sum_partials(const double* __restrict__ part, int ns, double (&d)[kVSlots]) {
    constexpr int kGroups = kVBlocks / kWave, kPer = kGroups / (THREADS / kWave);
    __shared__ double red[kVSlots][kGroups];
    const int wv = threadIdx.x / kWave, ln = threadIdx.x % kWave;
    double v[kVSlots][kPer];
#pragma unroll
    for (int k = 0; k < kVSlots; ++k)
#pragma unroll
        for (int g = 0; g < kPer; ++g) v[k][g] = k < ns ? part[k * kVBlocks + (wv * kPer + g) * kWave + ln] : 0.0;
#pragma unroll
    for (int k = 0; k < kVSlots; ++k)
#pragma unroll
        for (int g = 0; g < kPer; ++g) {
            if (k >= ns) continue;   // uniform
            const double t = group_sum(v[k][g], kWave);
            if (ln == 0) red[k][wv * kPer + g] = t;
        }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kVSlots; ++k) {
        d[k] = 0.0;
        if (k < ns)
            for (int w2 = 0; w2 < kGroups; ++w2) d[k] += red[k][w2];
    }
}

// the scalar updates from the sums of a stage
enum { R_INIT, R_ALPHA, R_OMEGA, R_NEXT, R_RES };
__device__ __forceinline__ void bicg_update(int stage, const double (&d)[kVSlots], double tol2, int maxit,
                                            double (&sc)[kNScalars]) {
    switch (stage) {
    case R_INIT:
        sc[S_RHO1] = d[0];
        sc[S_RR] = d[1];
        sc[S_BB] = d[2];
        sc[S_RHO0] = sc[S_ALPHA] = sc[S_OMEGA] = 1.0;
        sc[S_ITERS] = 0.0;
        sc[S_STATUS] = ST_RUNNING;
        sc[S_DONE] = 0.0;
        if (d[1] <= tol2 * d[2]) { sc[S_DONE] = 1.0; sc[S_STATUS] = ST_CONVERGED; }
        if (maxit <= 0 && sc[S_DONE] == 0.0) { sc[S_DONE] = 1.0; sc[S_STATUS] = ST_MAXIT; }
        break;
    case R_ALPHA:
        if (d[0] == 0.0 || !isfinite(d[0])) { sc[S_DONE] = 1.0; sc[S_STATUS] = ST_BREAKDOWN; }
        else sc[S_ALPHA] = sc[S_RHO1] / d[0];
        break;
    case R_OMEGA:   // d[0] = (t, s), d[1] = (t, t)
        if (d[1] == 0.0 || !isfinite(d[1])) { sc[S_DONE] = 1.0; sc[S_STATUS] = ST_BREAKDOWN; }
        else sc[S_OMEGA] = d[0] / d[1];
        break;
    case R_NEXT:    // d[0] = (r^, r), d[1] = (r, r)
        sc[S_RHO0] = sc[S_RHO1];
        sc[S_RHO1] = d[0];
        sc[S_RR] = d[1];
        sc[S_ITERS] += 1.0;
        if (d[1] <= tol2 * sc[S_BB]) { sc[S_DONE] = 1.0; sc[S_STATUS] = ST_CONVERGED; }
        else if (!isfinite(d[1])) { sc[S_DONE] = 1.0; sc[S_STATUS] = ST_BREAKDOWN; }
        else if (sc[S_ITERS] >= maxit) { sc[S_DONE] = 1.0; sc[S_STATUS] = ST_MAXIT; }
        break;
    case R_RES:
        sc[S_RES] = d[0];
        break;
    }
}

// State `from` through a stage to state `to` (the same for a launch of one
// work-group), by every thread of the launch; a finished solve's state is
// passed on as it is.  The result is left in sc.
template <int THREADS>
__device__ __forceinline__ void bicg_stage(const BicgVec& V, int stage, int from, int to, const double* part, int ns,
                                           double (&sc)[kNScalars]) {
#pragma unroll
    for (int k = 0; k < kNScalars; ++k) sc[k] = stage == R_INIT ? 0.0 : V.sc[from * kNScalars + k];
    if (stage == R_INIT || stage == R_RES || sc[S_DONE] == 0.0) {   // uniform
        double d[kVSlots];
        sum_partials<THREADS>(part, ns, d);
        bicg_update(stage, d, V.tol2, V.maxit, sc);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < kNScalars; ++k) V.sc[to * kNScalars + k] = sc[k];
    }
}

// a stage by itself: the first, the last, and the end of a batch of iterations
__global__ __launch_bounds__(kVBlocks) void k_bicg_reduce(BicgVec V, int stage) {
    double sc[kNScalars];
    const int from = stage == R_NEXT ? C_OMEGA : C_NEXT;
    bicg_stage<kVBlocks>(V, stage, from, C_NEXT, V.part + (stage == R_NEXT ? kPartX * kVBlocks : 0),
                         stage == R_INIT ? 3 : stage == R_NEXT ? 2 : 1, sc);
}

// p = r + beta (p - omega v), p^ = dinv p; `next`: the sums of the x before it first
__global__ __launch_bounds__(kVThreads) void k_bicg_p(BicgVec V, int next) {
    double sc[kNScalars];
    if (next) {
        bicg_stage<kVThreads>(V, R_NEXT, C_OMEGA, C_NEXT, V.part + kPartX * kVBlocks, 2, sc);
    } else {
#pragma unroll
        for (int k = 0; k < kNScalars; ++k) sc[k] = V.sc[C_NEXT * kNScalars + k];
    }
    if (sc[S_DONE] != 0.0) return;
    const double beta = (sc[S_RHO1] / sc[S_RHO0]) * (sc[S_ALPHA] / sc[S_OMEGA]);
    const double om = sc[S_OMEGA];
    for (int64_t i = (int64_t)blockIdx.x * kVThreads + threadIdx.x; i < V.n; i += (int64_t)kVBlocks * kVThreads) {
        const double pi = V.r[i] + beta * (V.p[i] - om * V.v[i]);
        V.p[i] = pi;
        V.ph[i] = V.dinv[i] * pi;
    }
}

// v = A p^ (from the operator); partial (r^, v)
__global__ __launch_bounds__(kVThreads) void k_bicg_v(BicgVec V) {
    if (V.sc[C_NEXT * kNScalars + S_DONE] != 0.0) return;
    double acc[kVSlots] = {0.0, 0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * kVThreads + threadIdx.x; i < V.n; i += (int64_t)kVBlocks * kVThreads) {
        acc[0] += V.rh[i] * V.v[i];
    }
    block_partials(acc, 1, V.part);
}

// the sum of v; s = r - alpha v, s^ = dinv s
__global__ __launch_bounds__(kVThreads) void k_bicg_s(BicgVec V) {
    double sc[kNScalars];
    bicg_stage<kVThreads>(V, R_ALPHA, C_NEXT, C_ALPHA, V.part, 1, sc);
    if (sc[S_DONE] != 0.0) return;
    const double al = sc[S_ALPHA];
    for (int64_t i = (int64_t)blockIdx.x * kVThreads + threadIdx.x; i < V.n; i += (int64_t)kVBlocks * kVThreads) {
        const double si = V.r[i] - al * V.v[i];
        V.s[i] = si;
        V.sh[i] = V.dinv[i] * si;
    }
}

// t = A s^ (from the operator); partials (t, s), (t, t)
__global__ __launch_bounds__(kVThreads) void k_bicg_t(BicgVec V) {
    if (V.sc[C_ALPHA * kNScalars + S_DONE] != 0.0) return;
    double acc[kVSlots] = {0.0, 0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * kVThreads + threadIdx.x; i < V.n; i += (int64_t)kVBlocks * kVThreads) {
        const double ti = V.t[i];
        acc[0] += ti * V.s[i];
        acc[1] += ti * ti;
    }
    block_partials(acc, 2, V.part + kPartT * kVBlocks);
}

// the sums of t; x += alpha p^ + omega s^, r = s - omega t; partials (r^, r), (r, r)
__global__ __launch_bounds__(kVThreads) void k_bicg_x(BicgVec V) {
    double sc[kNScalars];
    bicg_stage<kVThreads>(V, R_OMEGA, C_ALPHA, C_OMEGA, V.part + kPartT * kVBlocks, 2, sc);
    if (sc[S_DONE] != 0.0) return;
    const double al = sc[S_ALPHA], om = sc[S_OMEGA];
    double acc[kVSlots] = {0.0, 0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * kVThreads + threadIdx.x; i < V.n; i += (int64_t)kVBlocks * kVThreads) {
        V.x[i] += al * V.ph[i] + om * V.sh[i];
        const double ri = V.s[i] - om * V.t[i];
        V.r[i] = ri;
        acc[0] += V.rh[i] * ri;
        acc[1] += ri * ri;
    }
    block_partials(acc, 2, V.part + kPartX * kVBlocks);
}

// true residual b - A x (t = A x); partial (res, res)
__global__ __launch_bounds__(kVThreads) void k_bicg_res(BicgVec V) {
    double acc[kVSlots] = {0.0, 0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * kVThreads + threadIdx.x; i < V.n; i += (int64_t)kVBlocks * kVThreads) {
        const double ri = V.b[i] - V.t[i];
        acc[0] += ri * ri;
    }
    block_partials(acc, 1, V.part);
}

static int ppe_common(const vct_nlist* nl, Grid& g, const double* pos_sorted, const double* vol_sorted, int kernel,
                      const double* state64, uint32_t out_mask, PpeArgs& a) {
    int st = nlist_check(nl, g);
    if (st) return st;
    if (!mask_valid(out_mask) || (kernel != VCT_KERNEL_WENDLAND_C2 && kernel != VCT_KERNEL_CUBIC_SPLINE))
        return VCT_E_ARG;
    const int dim = nl->dim;
    const int64_t n = nl->n;
    if (n > 0 && (!pos_sorted || !vol_sorted || !nl->col16 || !state64)) return VCT_E_ARG;
    const int64_t ncols = dim == 3 ? g.nc[0] * g.nc[1] : g.nc[0];
    memset(&a, 0, sizeof(a));
    a.n = n; a.R = nl->R; a.invR = 1.0 / nl->R; a.g = g; a.pos = pos_sorted; a.vol = vol_sorted; a.state = state64;
    a.lap_row = group_row(dim, out_mask, VCT_OUT_LAP);
    a.nrows = n_out_rows(dim, out_mask);
    a.row_ptr = nl->row_ptr; a.col16 = nl->col16; a.cs = nl->cell_start; a.cstart = nl->chunk_start;
    a.cinfo = reinterpret_cast<const int4*>(nl->chunk_info); a.cwin = nl->chunk_win;
    a.nchunks = nl->chunk_off + ncols;
    return VCT_OK;
}

static int64_t chunk_cap(const vct_nlist* nl, const Grid& g) {
    const int64_t ncols = nl->dim == 3 ? g.nc[0] * g.nc[1] : g.nc[0];
    return ncols + nl->n / kChunk + 1;
}

template <int MODE, int D, int KERNEL>
static int launch_first(const PpeArgs& a, const MapParams& mp, int64_t mean, int64_t cap, hipStream_t s) {
    const char* name = MODE == 0 ? "k_ppe_first (rhs)" : "k_ppe_first (correct)";
    constexpr int kShort = D == 2 ? kRowsShort2 : kRowsShort3;
    if (mean <= short_row<D>())
        VCT_LAUNCH(name, (k_ppe_first<D, KERNEL, MODE, kShort>), dim3((unsigned)cap),
                   dim3(kChunk * RowShape<kShort>::lanes), 0, s, a, mp);
    else
        VCT_LAUNCH(name, (k_ppe_first<D, KERNEL, MODE, kRowsLong>), dim3((unsigned)cap),
                   dim3(kChunk * RowShape<kRowsLong>::lanes), 0, s, a, mp);
    VCT_LAUNCH_CHECK();
    return VCT_OK;
}

template <int MODE>
static int launch_first(const vct_nlist* nl, int kernel, const PpeArgs& a, const MapParams& mp, int64_t cap,
                        hipStream_t s) {
    const int64_t mean = mean_row(nl);
    if (nl->dim == 2)
        return kernel == VCT_KERNEL_WENDLAND_C2 ? launch_first<MODE, 2, VCT_KERNEL_WENDLAND_C2>(a, mp, mean, cap, s)
                                                : launch_first<MODE, 2, VCT_KERNEL_CUBIC_SPLINE>(a, mp, mean, cap, s);
    return kernel == VCT_KERNEL_WENDLAND_C2 ? launch_first<MODE, 3, VCT_KERNEL_WENDLAND_C2>(a, mp, mean, cap, s)
                                            : launch_first<MODE, 3, VCT_KERNEL_CUBIC_SPLINE>(a, mp, mean, cap, s);
}

template <int D, int KERNEL>
static int launch_diag(const PpeArgs& a, int64_t mean, int64_t cap, hipStream_t s) {
    constexpr int kShort = D == 2 ? kRowsShort2 : kRowsShort3;
    if (mean <= short_row<D>())
        VCT_LAUNCH("k_ppe_diag", (k_ppe_diag<D, KERNEL, kShort>), dim3((unsigned)cap),
                   dim3(kChunk * RowShape<kShort>::lanes), 0, s, a);
    else
        VCT_LAUNCH("k_ppe_diag", (k_ppe_diag<D, KERNEL, kRowsLong>), dim3((unsigned)cap),
                   dim3(kChunk * RowShape<kRowsLong>::lanes), 0, s, a);
    VCT_LAUNCH_CHECK();
    return VCT_OK;
}

template <int D>
static int launch_matvec(const PpeArgs& a, int64_t mean, int64_t cap, const double* x, double* out, hipStream_t s) {
    constexpr int kShort = D == 2 ? kRowsShort2 : kRowsShort3;
    if (mean <= short_row<D>())
        VCT_LAUNCH("k_ppe_matvec", (k_ppe_matvec<D, kShort>), dim3((unsigned)cap),
                   dim3(kChunk * RowShape<kShort>::lanes), 0, s, a, x, out);
    else
        VCT_LAUNCH("k_ppe_matvec", (k_ppe_matvec<D, kRowsLong>), dim3((unsigned)cap),
                   dim3(kChunk * RowShape<kRowsLong>::lanes), 0, s, a, x, out);
    VCT_LAUNCH_CHECK();
    return VCT_OK;
}

// Workspace without the kept matrix (enough for the product that forms it), and
// the bytes of the matrix (0: too many particles for one).
static size_t ppe_ws_base(int64_t n) {
    return aligned_sum({(size_t)n * 9 * sizeof(double), (size_t)kVParts * kVBlocks * sizeof(double),
                        (size_t)kNStates * kNScalars * sizeof(double)});
}
static int64_t mat_entries(int dim, int64_t n) {
    const int64_t e = n * (dim == 3 ? kMatRow3 : kMatRow2);
    return (size_t)e * sizeof(double) <= kMatMax ? e : 0;
}

VCT_CHECKS_TU(checks_ppe)

}  // namespace vct

using namespace vct;

extern "C" int vct_ppe_rhs(const vct_nlist* nl, const double* pos_sorted, const double* vol_sorted, int kernel,
                           const double* state64, uint32_t out_mask, const vct_map* map, const double* vstar,
                           double rho, double dt, double gamma, const double* jr, const uint8_t* dirichlet,
                           const double* pbc, double* rhs, double* div, double* dens, void* stream) {
    VCT_API_RANGE("vct_ppe_rhs");
    Grid g;
    PpeArgs a;
    int st = ppe_common(nl, g, pos_sorted, vol_sorted, kernel, state64, out_mask, a);
    if (st) return st;
    if (!map || !(dt > 0.0) || !isfinite(rho) || !isfinite(gamma)) return VCT_E_ARG;
    MapParams mp;
    st = map_params_from(map, nl->dim, nl->n, mp);
    if (st) return st;
    if (nl->n == 0) return VCT_OK;
    if (!vstar || !rhs) return VCT_E_ARG;
    a.f = vstar; a.jr = jr; a.dirichlet = dirichlet; a.pbc = pbc; a.rho = rho; a.dt = dt; a.gamma = gamma;
    a.rhs = rhs; a.div = div; a.dens = dens;
    return launch_first<0>(nl, kernel, a, mp, chunk_cap(nl, g), as_stream(stream));
}

extern "C" int vct_ppe_correct(const vct_nlist* nl, const double* pos_sorted, const double* vol_sorted, int kernel,
                               const double* state64, uint32_t out_mask, const vct_map* map, const double* p,
                               const double* vstar, double rho, double dt, double* vout, void* stream) {
    VCT_API_RANGE("vct_ppe_correct");
    Grid g;
    PpeArgs a;
    int st = ppe_common(nl, g, pos_sorted, vol_sorted, kernel, state64, out_mask, a);
    if (st) return st;
    if (!map || !isfinite(dt) || !(rho != 0.0) || !isfinite(rho)) return VCT_E_ARG;
    MapParams mp;
    st = map_params_from(map, nl->dim, nl->n, mp);
    if (st) return st;
    if (nl->n == 0) return VCT_OK;
    if (!p || !vstar || !vout) return VCT_E_ARG;
    a.f = p; a.vstar = vstar; a.vout = vout; a.rho = rho; a.dt = dt;
    return launch_first<1>(nl, kernel, a, mp, chunk_cap(nl, g), as_stream(stream));
}

extern "C" size_t vct_ppe_workspace_size(int dim, int64_t n, uint32_t out_mask) {
    if ((dim != 2 && dim != 3) || n < 0 || !mask_valid(out_mask)) return 0;
    const int64_t nn = n > 0 ? n : 1;
    return aligned_sum({ppe_ws_base(nn), (size_t)mat_entries(dim, nn) * sizeof(double)});
}

extern "C" int vct_ppe_solve(const vct_nlist* nl, const double* pos_sorted, const double* vol_sorted, int kernel,
                             const double* state64, uint32_t out_mask, const uint8_t* dirichlet, const double* rhs,
                             double* p, double tol, int max_iter, int* iters, double* relres, void* ws,
                             size_t ws_bytes, void* stream) {
    VCT_API_RANGE("vct_ppe_solve");
    Grid g;
    PpeArgs a;
    int st = ppe_common(nl, g, pos_sorted, vol_sorted, kernel, state64, out_mask, a);
    if (st) return st;
    if (!(out_mask & VCT_OUT_LAP) || !(tol >= 0.0) || max_iter < 0) return VCT_E_ARG;
    const int dim = nl->dim;
    const int64_t n = nl->n;
    if (iters) *iters = 0;
    if (relres) *relres = 0.0;
    if (n == 0) return VCT_OK;
    if (!rhs || !p) return VCT_E_ARG;
    if (!ws || ws_bytes < ppe_ws_base(n)) return VCT_E_WORKSPACE;
    hipStream_t s = as_stream(stream);
    Carver cv(ws, ws_bytes);
    BicgVec V;
    V.n = n; V.b = rhs; V.x = p;
    double* vecs = cv.take<double>((size_t)n * 9);
    V.r = vecs; V.rh = vecs + n; V.p = vecs + 2 * n; V.v = vecs + 3 * n; V.s = vecs + 4 * n; V.t = vecs + 5 * n;
    V.ph = vecs + 6 * n; V.sh = vecs + 7 * n; V.dinv = vecs + 8 * n;
    V.part = cv.take<double>((size_t)kVParts * kVBlocks);
    V.sc = cv.take<double>(kNStates * kNScalars);
    V.tol2 = tol * tol;
    V.maxit = max_iter;
    const int64_t cap = chunk_cap(nl, g);
    a.dirichlet = dirichlet; a.dinv = V.dinv;
    const int64_t mean = mean_row(nl);
    // The matrix is kept where its entries fit the workspace and an iteration
    // may follow: storing it costs less than one product saves in 3-D (0.18
    // against 0.23 ms, 1,048,352 particles), three in 2-D (0.07 against 0.023,
    // 1,048,576), and an iteration takes two besides the two residuals.
    if (max_iter >= kMatIters && mat_entries(dim, n) > 0 && ws_bytes >= vct_ppe_workspace_size(dim, n, out_mask)) {
        int64_t nnz = 0;
        VCT_HIP_CHECK(hipMemcpyAsync(&nnz, nl->row_ptr + n, sizeof(nnz), hipMemcpyDeviceToHost, s));
        VCT_HIP_CHECK(hipStreamSynchronize(s));
        if (nnz <= mat_entries(dim, n)) a.wmat = cv.take<double>((size_t)mat_entries(dim, n));
    }
    if (dim == 2)
        st = kernel == VCT_KERNEL_WENDLAND_C2 ? launch_diag<2, VCT_KERNEL_WENDLAND_C2>(a, mean, cap, s)
                                              : launch_diag<2, VCT_KERNEL_CUBIC_SPLINE>(a, mean, cap, s);
    else
        st = kernel == VCT_KERNEL_WENDLAND_C2 ? launch_diag<3, VCT_KERNEL_WENDLAND_C2>(a, mean, cap, s)
                                              : launch_diag<3, VCT_KERNEL_CUBIC_SPLINE>(a, mean, cap, s);
    if (st) return st;
    auto matvec = [&](const double* xin, double* out) {
        if (a.wmat)
            return dim == 2 ? launch_matvec<2>(a, mean, cap, xin, out, s) : launch_matvec<3>(a, mean, cap, xin, out, s);
        return apply_lap(nl, g, xin, pos_sorted, vol_sorted, kernel, state64, out_mask, dirichlet, out, s);
    };
    const dim3 vg(kVBlocks), vb(kVThreads);
    if ((st = matvec(V.x, V.t)) < 0) return st;
    VCT_LAUNCH("k_bicg_init", k_bicg_init, vg, vb, 0, s, V);
    VCT_LAUNCH_CHECK();
    VCT_LAUNCH("k_bicg_reduce", k_bicg_reduce, dim3(1), dim3(kVBlocks), 0, s, V, (int)R_INIT);
    VCT_LAUNCH_CHECK();
    // iterations in batches; the host reads the scalars after each batch
    constexpr int kBatch = 8;
    double hs[kNScalars];
    int done_iters = 0;
    for (;;) {
        VCT_HIP_CHECK(hipMemcpyAsync(hs, V.sc, sizeof(hs), hipMemcpyDeviceToHost, s));
        VCT_HIP_CHECK(hipStreamSynchronize(s));
        if (hs[S_DONE] != 0.0 || done_iters >= max_iter) break;
        for (int k = 0; k < kBatch && done_iters < max_iter; ++k, ++done_iters) {
            VCT_LAUNCH("k_bicg_p", k_bicg_p, vg, vb, 0, s, V, (int)(k > 0));
            VCT_LAUNCH_CHECK();
            if ((st = matvec(V.ph, V.v)) < 0) return st;
            VCT_LAUNCH("k_bicg_v", k_bicg_v, vg, vb, 0, s, V);
            VCT_LAUNCH_CHECK();
            VCT_LAUNCH("k_bicg_s", k_bicg_s, vg, vb, 0, s, V);
            VCT_LAUNCH_CHECK();
            if ((st = matvec(V.sh, V.t)) < 0) return st;
            VCT_LAUNCH("k_bicg_t", k_bicg_t, vg, vb, 0, s, V);
            VCT_LAUNCH_CHECK();
            VCT_LAUNCH("k_bicg_x", k_bicg_x, vg, vb, 0, s, V);
            VCT_LAUNCH_CHECK();
        }
        VCT_LAUNCH("k_bicg_reduce", k_bicg_reduce, dim3(1), dim3(kVBlocks), 0, s, V, (int)R_NEXT);
        VCT_LAUNCH_CHECK();
    }
    // the true residual of the result
    if ((st = matvec(V.x, V.t)) < 0) return st;
    VCT_LAUNCH("k_bicg_res", k_bicg_res, vg, vb, 0, s, V);
    VCT_LAUNCH_CHECK();
    VCT_LAUNCH("k_bicg_reduce", k_bicg_reduce, dim3(1), dim3(kVBlocks), 0, s, V, (int)R_RES);
    VCT_LAUNCH_CHECK();
    VCT_HIP_CHECK(hipMemcpyAsync(hs, V.sc, sizeof(hs), hipMemcpyDeviceToHost, s));
    VCT_HIP_CHECK(hipStreamSynchronize(s));
    if (iters) *iters = (int)hs[S_ITERS];
    if (relres) *relres = hs[S_BB] > 0.0 ? sqrt(hs[S_RES] / hs[S_BB]) : sqrt(hs[S_RES]);
    return hs[S_STATUS] == ST_CONVERGED ? VCT_OK : VCT_W_NOCONV;
}
