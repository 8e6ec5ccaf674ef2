// Wavefront-per-reactor kernels.  One 64-lane wavefront owns one reactor:
//   - species phases run lane-per-species (lane l holds state component l,
//     i.e. T on lane 0 and Y_{l-1} on lane l; a second register slot holds
//     component l + 64 when N > 64);
//   - reaction phases run lane-per-reaction, scattering rates of progress
//     into per-species accumulators in LDS with FP64 LDS atomics;
//   - the Rosenbrock matrix (I/(gamma h) - J) lives in 16 x 16 register tiles
//     and is inverted by a blocked Gauss-Jordan elimination on the FP64 matrix
//     cores (wtile.h).
// This is the deep-vectorisation design of Section 4 applied to a 64-wide
// wavefront.  Integrators pull reactors from a device work queue (the
// paper's global atomic counter, Section 5.2) one reactor per wavefront, so
// reactors with different step counts never hold each other up (the waste of
// Eq. waste is zero by construction).  Every workgroup is one wavefront.
#include "ck_internal.h"
#include "kinetics.h"
#include "launch.h"
#include "reactions.h"
#include "wtile.h"

extern "C" __device__ unsigned long long __ockl_wfred_max_u64(unsigned long long);
extern "C" __device__ unsigned __ockl_wfred_max_u32(unsigned);
extern "C" __device__ double __ockl_wfred_add_f64(double);

namespace ck {
namespace {

__device__ __forceinline__ int lane_id() { return __lane_id(); }
// Value the compiler cannot see through: keeps cheap per-phase values (lane masks, pivot
// lanes) from being hoisted across phases, where they would only occupy and spill SGPRs.
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}
__device__ __forceinline__ int lane_fresh() { return opaque(__lane_id()); }
// The same for a wave-uniform value, kept in a scalar register.
__device__ __forceinline__ int opaque_s(int v) {
    asm volatile("" : "+s"(v));
    return v;
}
__device__ __forceinline__ double wsum(double v) { return __ockl_wfred_add_f64(v); }
__device__ __forceinline__ double bcast(double v, int src) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), src);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), src);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ bool wave_all(bool v) { return __ballot(!v) == 0ull; }

// ---------------------------------------------------------------------------------------
// LDS layout of one wavefront (doubles), ns1 = ns + 1 (a null species closes every array):
//   C G H WD [ns1]                                   every kernel
//   | scratch of the tiles                           kLdsTiles (ROS4 with another Jacobian)
//   | TB DWT HC [ns1] TROW[96] JC                    kLdsJac (ROS4): JC holds d wdot / dC for a window
//                                                    of columns, then the scratch of the tiles
// ---------------------------------------------------------------------------------------
enum LdsKind { kLdsRhs, kLdsTiles, kLdsJac };

// Constants of the species that a register slot of this lane holds (slot 0 of lane 0 is T), read once
// per kernel: an out-of-range slot takes a neighbour's values and `valid` masks what it stores.
struct SpeciesLane {
    double W, iW, Tmid;
    int k;
    bool valid;
};

struct Lds : RxArrays {
    SpeciesLane sl[2];
    double *TROW;   // temperature row of the matrix, by column, and 32 zeros
    double *park;   // this wavefront's slice of the workspace, or null
    int cv;         // 0: constant pressure (p = pressure); 1: constant volume (p = density)
};

// Column windows of the staged d wdot/dC for a padded size NP: matrix columns [32 w, 32 w + 32), the
// temperature column being matrix column 0, so that a window is whole tile columns.
template <int NP>
struct WaveShape {
    static constexpr int TR = WTile<NP>::TR;
    static constexpr int NWIN = TR > 2 ? 2 : 1;
    static constexpr int WIN = TR > 2 ? 32 : 16 * TR;
    static constexpr int LDJ = WIN | 1;
    static constexpr bool PARK = NWIN == 2;    // the first window's rate scalars wait for the second
};

// jc: doubles of the JC region (kLdsTiles, kLdsJac)
__host__ __device__ inline size_t lds_doubles(LdsKind kind, int ns, size_t jc) {
    size_t d = 4 * size_t(ns + 1);
    if (kind == kLdsTiles) d += jc;
    if (kind == kLdsJac) d += 3 * size_t(ns + 1) + 96 + jc;
    return d;
}

__device__ __forceinline__ Lds carve(double *b, LdsKind kind, int ns, int ldj) {
    Lds L;
    L.JC = L.TB = L.DWT = L.HC = L.TROW = nullptr;
    L.ldj = ldj;
    L.C = b; b += ns + 1;
    L.G = b; b += ns + 1;
    L.H = b; b += ns + 1;
    L.WD = b; b += ns + 1;
    if (kind == kLdsTiles) L.JC = b;
    if (kind == kLdsJac) {
        L.TB = b; b += ns + 1;
        L.DWT = b; b += ns + 1;
        L.HC = b; b += ns + 1;
        L.TROW = b; b += 96;
        L.JC = b;
    }
    L.park = nullptr;
    L.cv = 0;
    return L;
}

template <int RPL>
__device__ __forceinline__ void init_lds(const DevMech &M, Lds &L, LdsKind kind) {
    const int l = lane_id(), ns = M.nsp;
#pragma unroll
    for (int c = 0; c < RPL; c++) {
        const int i = l + 64 * c;
        SpeciesLane &s = L.sl[c];
        s.valid = i >= 1 && i <= ns;
        s.k = min(max(i - 1, 0), ns - 1);
        s.W = M.W()[s.k];
        s.iW = M.invW()[s.k];
        s.Tmid = M.Tmid()[s.k];
    }
    if (l == 0) {
        L.C[ns] = 1.0;
        L.G[ns] = 0.0;
        L.H[ns] = 0.0;
    }
    if (kind == kLdsJac)
        for (int e = l; e < 96; e += 64) L.TROW[e] = 0.0;
    __syncthreads();
}

template <int RPL>
struct Mix {
    TPow t;
    double rho, invrho, Wbar, Ctot, cpm;
    double cp[RPL], h[RPL], dcp[RPL];
};

// Mixture state and per-species thermodynamics (Section 3: ideal gas, Eq. tfits).  Every lane reads
// an in-range species, so the loads are issued together and only the stores are masked.
template <int RPL, bool JAC>
__device__ __forceinline__ void species_pass(const DevMech &M, const double (&y)[RPL], double P, const Lds &L, Mix<RPL> &x) {
    const double T = bcast(y[0], 0);
    double z[RPL];
    Nasa co[RPL];
    double sz = 0.0;
#pragma unroll
    for (int c = 0; c < RPL; c++) {
        co[c] = species_coef(M, L.sl[c].k, T < L.sl[c].Tmid);
        z[c] = L.sl[c].valid ? y[c] * L.sl[c].iW : 0.0;
        sz += z[c];
    }
    x.t = tpow(T);
    const double S = wsum(sz);          // sum_k Y_k / W_k
    x.Wbar = ck_rcp(S);
    if (L.cv) {   // constant volume: P holds the (fixed) density
        x.rho = P;
        x.Ctot = P * S;
    } else {
        x.Ctot = P * x.t.invT * M.invR;
        x.rho = x.Ctot * x.Wbar;
    }
    x.invrho = ck_rcp(x.rho);
    double cpp = 0.0;
#pragma unroll
    for (int c = 0; c < RPL; c++) {
        const Thermo th = species_thermo(M, co[c], x.t);
        x.cp[c] = th.cp;
        x.h[c] = th.h;
        if (JAC) x.dcp[c] = th.dcp;
        if (L.sl[c].valid) {
            const int k = L.sl[c].k;
            L.C[k] = x.rho * z[c];
            L.G[k] = th.g;
            L.WD[k] = 0.0;
            if (JAC) {
                L.H[k] = th.h - 1.0;
                L.TB[k] = 0.0;
                L.DWT[k] = 0.0;
                L.HC[k] = 0.0;
            }
        }
        cpp = fma(z[c], th.cp, cpp);
    }
    x.cpm = wsum(cpp) * M.R;
    __syncthreads();
}

__device__ __forceinline__ void zero_jc(const Lds &L, int ns) {
    const int tot = ns * L.ldj;
    for (int e = lane_fresh(); e < tot; e += 64) L.JC[e] = 0.0;
}

// Eqs. ydot and tdot from the accumulated production rates.  Constant volume: internal energies
// U_k = H_k - R T and c_v = c_p - R / Wbar in place of H_k and c_p.
template <int RPL>
__device__ __forceinline__ void finish_rhs(const DevMech &M, const Lds &L, const Mix<RPL> &x, double (&f)[RPL]) {
    const int lane = lane_fresh();
    const double shift = L.cv ? 1.0 : 0.0;
    double qp = 0.0;
#pragma unroll
    for (int c = 0; c < RPL; c++) {
        const double wd = L.sl[c].valid ? L.WD[L.sl[c].k] : 0.0;
        f[c] = L.sl[c].W * wd * x.invrho;
        qp = fma(x.h[c] - shift, wd, qp);
    }
    const double Q = wsum(qp) * (M.R * x.t.T);
    const double heat_cap = L.cv ? x.cpm - M.R * ck_rcp(x.Wbar) : x.cpm;
    const double fT = -Q * ck_rcp(x.rho * heat_cap);
    if (lane == 0) f[0] = fT;
}

template <int RPL, bool GEN = true>
__device__ __forceinline__ void rhs_wave(const DevMech &M, const Lds &L, const double (&y)[RPL], double P, double (&f)[RPL]) {
    Mix<RPL> x;
    const PairRec first = first_pair<64>(M, lane_fresh());
    species_pass<RPL, false>(M, y, P, L, x);
    reaction_pass<64, false, GEN>(M, L, x.t, x.Ctot, RxScale{0.0, 0.0, 0.0}, 0, 0, kRates, nullptr, lane_fresh(), first);
    __syncthreads();
    finish_rhs<RPL>(M, L, x, f);
    __syncthreads();
}

__device__ __forceinline__ RxScale rx_scale(const Lds &L, const Mix<1> &x) {
    return L.cv ? RxScale{0.0, 0.0, 0.0} : RxScale{x.t.invT, x.Wbar * x.invrho, 1.0};
}

// Chain rule for the lane's species row (lane k + 1) and its entry of the temperature row, in the
// specific mole numbers z = Y / W (J' of ChainIn): J'[k+1][0] = col0, J'[k+1][1+j] = JC[k][j] + beta,
// J'[0][1+k] = trow, J'[0][0] = J00.
struct Chain {
    double beta, col0, trow, J00;
};
__device__ __forceinline__ Chain chain_rule(const DevMech &M, const Lds &L, const Mix<1> &x, double y0, double fT) {
    const bool valid = L.sl[0].valid;
    const int k = L.sl[0].k;
    const double TBk = valid ? L.TB[k] : 0.0, WDk = valid ? L.WD[k] : 0.0, DWTk = valid ? L.DWT[k] : 0.0;
    const bool cv = L.cv != 0;
    ChainIn c;
    c.rho = x.rho;
    c.invrho = x.invrho;
    c.Wbar = x.Wbar;
    c.invT = x.t.invT;
    c.R = M.R;
    c.RT = M.R * x.t.T;
    c.cpm = x.cpm;
    c.fT = fT;
    const double e = cv ? 1.0 : 0.0;
    const double Hk = x.h[0] - e;                               // over R T
    c.sHB = c.RT * wsum(Hk * TBk);
    c.sHW = c.RT * wsum(Hk * WDk);
    c.dQT = M.R * wsum(fma(x.cp[0] - e, WDk, Hk * (x.t.T * DWTk - (cv ? 0.0 : WDk))));
    c.sdcp = M.R * wsum(valid ? y0 * x.dcp[0] * L.sl[0].iW : 0.0);
    Chain o;
    o.trow = valid ? chain_trow(c, cv, L.HC[k], x.cp[0]) : 0.0;
    o.J00 = chain_J00(c, cv);
    o.beta = TBk;
    o.col0 = DWTk * x.invrho;
    return o;
}

// f(y) and the tiles of M' = dg I - J' (J' the Jacobian in the specific mole numbers, similar to J by
// diag(1, W)) for N <= NP <= 64.  The first window's reaction pass also leaves every per-species sum
// of the chain rule, so each window's columns are final when they are read.  The second window takes
// the first one's rate constants from the park slice when they fit (else it evaluates them again).
// iw and w: 1/W and W of the lane's component (1 for T, 0 for padding).
template <int NP>
__device__ __forceinline__ void jac_tiles(const DevMech &M, const Lds &L, double y, double P, double dg,
                                          wd4 (&X)[WTile<NP>::TR][WTile<NP>::TR], double &f, double &iw, double &w) {
    using SH = WaveShape<NP>;
    constexpr int TR = SH::TR, NWIN = SH::NWIN, WIN = SH::WIN;
    Mix<1> x;
    const double yy[1] = {y};
    double ff[1];
    const int ns = M.nsp;
    const PairRec first = first_pair<64>(M, lane_fresh());
    zero_jc(L, ns);
    species_pass<1, true>(M, yy, P, L, x);
    const RxScale sc = rx_scale(L, x);
    const bool fits = NWIN == 2 && 3 * rx_blocks(M, 64) <= NP;
    reaction_pass<64, true>(M, L, x.t, x.Ctot, sc, -1, min(WIN, ns + 1), fits ? kRatesKeep : kRates,
                            L.park + lane_fresh(), lane_fresh(), first);
    __syncthreads();
    finish_rhs<1>(M, L, x, ff);
    f = ff[0];
    const Chain ch = chain_rule(M, L, x, y, bcast(f, 0));
    const int lane = lane_fresh();
    const int g = lane >> 4, c16 = lane & 15;
    if (L.sl[0].valid) {
        L.TROW[1 + L.sl[0].k] = ch.trow;
        L.JC[L.sl[0].k * SH::LDJ] = ch.col0;
    }
    if (lane == 0) L.TROW[0] = ch.J00;
    w = lane == 0 ? 1.0 : (L.sl[0].valid ? L.sl[0].W : 0.0);
    iw = lane == 0 ? 1.0 : (L.sl[0].valid ? L.sl[0].iW : 0.0);
    __syncthreads();
    double dgm[4];
#pragma unroll
    for (int v = 0; v < 4; v++) dgm[v] = c16 == g + 4 * v ? dg : 0.0;
    const int nsw = opaque_s(ns);
#pragma unroll
    for (int wnd = 0; wnd < NWIN; wnd++) {
        if (wnd > 0) {
            const PairRec again = first_pair<64>(M, lane_fresh());
            __syncthreads();
            zero_jc(L, ns);
            __syncthreads();
            reaction_pass<64, true>(M, L, x.t, x.Ctot, sc, WIN - 1, min(WIN, ns + 1 - WIN),
                                    fits ? kScatterKept : kScatter, L.park + lane_fresh(), lane_fresh(), again);
            __syncthreads();
        }
#pragma unroll
        for (int I = 0; I < TR; I++) {
            // matrix row 16 I + c: the temperature row, a species row or padding (zeros)
            const int r = 16 * I + c16;
            const bool sp = r >= 1 && r <= nsw;
            const double *row = sp ? &L.JC[(r - 1) * SH::LDJ] : (r == 0 ? L.TROW + WIN * wnd : L.TROW + 64);
            const double beta = sp ? L.TB[sp ? r - 1 : 0] : 0.0;
#pragma unroll
            for (int J = WIN / 16 * wnd; J < TR && J < WIN / 16 * (wnd + 1); J++)
#pragma unroll
                for (int v = 0; v < 4; v++) {
                    const int c0 = 16 * J + 4 * v;      // matrix columns c0 + g
                    if (c0 >= NP) {
                        X[J][I][v] = 0.0;
                        continue;
                    }
                    // beta on species columns: all but the temperature's and the padding's
                    const double b = c0 == 0 ? (g == 0 ? 0.0 : beta) : (c0 + 3 < NP - 8 || c0 + g <= nsw ? beta : 0.0);
                    X[J][I][v] = (I == J ? dgm[v] : 0.0) - (row[c0 - WIN * wnd + g] + b);
                }
        }
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------------------
// one steps
// ---------------------------------------------------------------------------------------
// Stages of a ROS4 step with the inverted matrix in tiles; iw scales a right-hand side, w a solution
// (the tiles are those of M in the variables z = y / w).
template <int NP>
__device__ __forceinline__ void ros4_stages(const DevMech &M, const Lds &L, double y, double P, double h,
                                            const wd4 (&X)[WTile<NP>::TR][WTile<NP>::TR], const WScratch &s, int ord,
                                            double f, double iw, double w, double &ynew, double &e) {
    const int lane = lane_fresh();
    auto solve = [&](double b) { return w * wt_solve<NP, double>(X, s, lane, ord, iw * b); };
    const double ih = 1.0 / h;
    const double u1 = solve(f);
    // the inverse stays in registers across the stage source terms
    double yt[1] = {y + Ros4::a21 * u1}, ft[1];
    rhs_wave<1>(M, L, yt, P, ft);
    const double u2 = solve(ft[0] + (Ros4::c21 * u1) * ih);
    yt[0] = y + Ros4::a31 * u1 + Ros4::a32 * u2;
    rhs_wave<1>(M, L, yt, P, ft);
    const double u3 = solve(ft[0] + (Ros4::c31 * u1 + Ros4::c32 * u2) * ih);
    const double u4 = solve(ft[0] + (Ros4::c41 * u1 + Ros4::c42 * u2 + Ros4::c43 * u3) * ih);
    ynew = y + Ros4::m1 * u1 + Ros4::m2 * u2 + Ros4::m3 * u3 + Ros4::m4 * u4;
    e = Ros4::e1 * u1 + Ros4::e2 * u2 + Ros4::e3 * u3 + Ros4::e4 * u4;
}

template <int NP>
struct Ros4Wave {
    __device__ static __forceinline__ bool step(const DevMech &M, const Lds &L, double y, double P, double h, double &ynew,
                                double &e) {
        wd4 X[WTile<NP>::TR][WTile<NP>::TR];
        double f, iw, w;
        jac_tiles<NP>(M, L, y, P, 1.0 / (Ros4::gamma * h), X, f, iw, w);
        const WScratch s = wt_scratch<NP>(L.JC);
        int ord;
        const bool ok = wt_invert<NP, double>(X, s, lane_fresh(), ord);
        ros4_stages<NP>(M, L, y, P, h, X, s, ord, f, iw, w, ynew, e);
        return ok;
    }
};

// ROS4 step with a forward-difference Jacobian (the paper's ROS4 set-up, Section 5): column j of
// J is (f(y + inc_j e_j) - f(y)) / inc_j, one source-term evaluation per column, with
//   inc_j = max(sqrt(eps) |y_j|, min_inc (rtol |y_j| + atol)),
//   min_inc = 1000 |h| eps N ||f(y)||_w (1 if that norm is 0), w_i = 1 / (rtol |y_i| + atol),
// as CVODE's dense difference quotient.  Columns are written to the parking slice (lane i holds
// row i), then loaded as tiles; f(y) doubles as the first stage's right-hand side.
template <int NP>
struct Ros4WaveFD {
    __device__ static __forceinline__ bool step(const DevMech &M, const Lds &L, double y, double P, double h,
                                                double &ynew, double &e, const IntOpts &o) {
        constexpr double eps = 2.220446049250313e-16;
        constexpr int TR = WTile<NP>::TR;
        const int N = M.N;
        const int lane = lane_fresh();
        const bool comp = lane < N;
        double yy[1] = {y}, f0[1];
        rhs_wave<1>(M, L, yy, P, f0);
        const double r = comp ? f0[0] / (o.rtol * fabs(y) + o.atol) : 0.0;
        const double fnorm = sqrt(wsum(r * r) / N);
        const double min_inc = fnorm != 0.0 ? 1000.0 * fabs(h) * eps * N * fnorm : 1.0;
        {
            double *pk = L.park + lane_fresh();
            for (int j = 0; j < N; j++) {
                const double yj = bcast(y, j);
                const double wj = 1.0 / (o.rtol * fabs(yj) + o.atol);
                const double inc = fmax(sqrt(eps) * fabs(yj), min_inc / wj);
                double yp[1] = {lane == j ? yj + inc : y}, fj[1];
                rhs_wave<1>(M, L, yp, P, fj);
                pk[j * 64] = comp ? (fj[0] - f0[0]) / inc : 0.0;   // J[lane][j]
            }
        }
        __syncthreads();      // lanes read each other's columns below
        const double dg = 1.0 / (Ros4::gamma * h);
        wd4 X[TR][TR];
        const int g = lane >> 4, c16 = lane & 15;
#pragma unroll
        for (int J = 0; J < TR; J++)
#pragma unroll
            for (int I = 0; I < TR; I++)
#pragma unroll
                for (int v = 0; v < 4; v++) {
                    const int row = 16 * I + c16, col = 16 * J + g + 4 * v;
                    const double d = (I == J && c16 == g + 4 * v && col < NP) ? dg : 0.0;
                    X[J][I][v] = d - (row < N && col < N ? L.park[col * 64 + row] : 0.0);
                }
        const WScratch s = wt_scratch<NP>(L.JC);
        int ord;
        const bool ok = wt_invert<NP, double>(X, s, lane_fresh(), ord);
        ros4_stages<NP>(M, L, y, P, h, X, s, ord, f0[0], 1.0, 1.0, ynew, e);
        return ok;
    }
};

// ---------------------------------------------------------------------------------------
// FP32 factorisation with FP64 residual refinement
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ double wmax_abs(double v) {
    return __longlong_as_double((long long)__ockl_wfred_max_u64((unsigned long long)__double_as_longlong(fabs(v))));
}

// ROS4 step whose linear solves use an FP32 inverse of M = I/(gamma h) - J (tiles, FP32 matrix cores),
// refined with FP64 residuals r = b - M x (M's FP64 tiles stay in registers beside it).  A solve is
// done once the correction is below 2^-48 of the solution (max norms over T and Y).  If a correction
// fails to halve the previous one, or the allowed sweeps run out first, the FP32 step is abandoned and
// the reactor-step is done again in FP64; `fb` counts such steps.  With zero sweeps the FP32 solutions
// are used as they are.
template <int NP>
struct Ros4Wave32 {
    __device__ static __forceinline__ bool step32(const DevMech &M, const Lds &L, double y, double P, double h,
                                                  double &ynew, double &e, int sweeps, bool &conv) {
        constexpr int TR = WTile<NP>::TR;
        wd4 X[TR][TR];
        wf4 F[TR][TR];
        double f, iw, w;
        jac_tiles<NP>(M, L, y, P, 1.0 / (Ros4::gamma * h), X, f, iw, w);
#pragma unroll
        for (int J = 0; J < TR; J++)
#pragma unroll
            for (int I = 0; I < TR; I++)
#pragma unroll
                for (int v = 0; v < 4; v++) F[J][I][v] = float(X[J][I][v]);
        const WScratch s = wt_scratch<NP>(L.JC);
        const int lane = lane_fresh();
        int ord;
        const bool ok = wt_invert<NP, float>(F, s, lane, ord);
        conv = true;
        auto solve = [&](double bb) -> double {
            const double b = iw * bb;
            double x = double(wt_solve<NP, float>(F, s, lane, ord, float(b)));
            if (sweeps <= 0) return w * x;
            double dprev = INFINITY;
            for (int k = 0; k < sweeps; k++) {
                const double mx = wt_times<NP>(X, s, lane, x);     // every lane takes part
                const double r = lane < NP ? b - mx : 0.0;
                const double d = double(wt_solve<NP, float>(F, s, lane, ord, float(r)));
                x += d;
                const double dmax = wmax_abs(w * d), xmax = wmax_abs(w * x);
                if (dmax <= 0x1p-48 * xmax) return w * x;
                if (!(dmax <= 0.5 * dprev)) break;      // stagnation (or not finite)
                dprev = dmax;
            }
            conv = false;
            return w * x;
        };
        const double ih = 1.0 / h;
        const double u1 = solve(f);
        if (!conv) return ok;
        double yt[1] = {y + Ros4::a21 * u1}, ft[1];
        rhs_wave<1>(M, L, yt, P, ft);
        const double u2 = solve(ft[0] + (Ros4::c21 * u1) * ih);
        if (!conv) return ok;
        yt[0] = y + Ros4::a31 * u1 + Ros4::a32 * u2;
        rhs_wave<1>(M, L, yt, P, ft);
        const double u3 = solve(ft[0] + (Ros4::c31 * u1 + Ros4::c32 * u2) * ih);
        if (!conv) return ok;
        const double u4 = solve(ft[0] + (Ros4::c41 * u1 + Ros4::c42 * u2 + Ros4::c43 * u3) * ih);
        if (!conv) return ok;
        ynew = y + Ros4::m1 * u1 + Ros4::m2 * u2 + Ros4::m3 * u3 + Ros4::m4 * u4;
        e = Ros4::e1 * u1 + Ros4::e2 * u2 + Ros4::e3 * u3 + Ros4::e4 * u4;
        return ok;
    }
    __device__ static __forceinline__ bool step(const DevMech &M, const Lds &L, double y, double P, double h, double &ynew,
                                double &e, int sweeps, int &fb) {
        bool conv = true;
        const bool ok = step32(M, L, y, P, h, ynew, e, sweeps, conv);
        if (conv) return ok;
        fb++;
        return Ros4Wave<NP>::step(M, L, y, P, h, ynew, e);
    }
};

template <int RPL>
struct Rkf45Wave {
    static constexpr double qinv = 0.2;
    __device__ static __forceinline__ void stage(const DevMech &M, const Lds &L, const double (&yt)[RPL], double P, double h,
                                 double (&k)[RPL]) {
        rhs_wave<RPL>(M, L, yt, P, k);
#pragma unroll
        for (int c = 0; c < RPL; c++) k[c] *= h;
    }
    __device__ static __forceinline__ bool step(const DevMech &M, const Lds &L, const double (&y)[RPL], double P, double h,
                                double (&ynew)[RPL], double (&e)[RPL]) {
        double k1[RPL], k2[RPL], k3[RPL], k4[RPL], k5[RPL], k6[RPL], yt[RPL];
        stage(M, L, y, P, h, k1);
#pragma unroll
        for (int c = 0; c < RPL; c++) yt[c] = y[c] + Rkf45::a21 * k1[c];
        stage(M, L, yt, P, h, k2);
#pragma unroll
        for (int c = 0; c < RPL; c++) yt[c] = y[c] + Rkf45::a31 * k1[c] + Rkf45::a32 * k2[c];
        stage(M, L, yt, P, h, k3);
#pragma unroll
        for (int c = 0; c < RPL; c++) yt[c] = y[c] + Rkf45::a41 * k1[c] + Rkf45::a42 * k2[c] + Rkf45::a43 * k3[c];
        stage(M, L, yt, P, h, k4);
#pragma unroll
        for (int c = 0; c < RPL; c++)
            yt[c] = y[c] + Rkf45::a51 * k1[c] + Rkf45::a52 * k2[c] + Rkf45::a53 * k3[c] + Rkf45::a54 * k4[c];
        stage(M, L, yt, P, h, k5);
#pragma unroll
        for (int c = 0; c < RPL; c++)
            yt[c] = y[c] + Rkf45::a61 * k1[c] + Rkf45::a62 * k2[c] + Rkf45::a63 * k3[c] + Rkf45::a64 * k4[c] +
                    Rkf45::a65 * k5[c];
        stage(M, L, yt, P, h, k6);
#pragma unroll
        for (int c = 0; c < RPL; c++) {
            ynew[c] = y[c] + Rkf45::b1 * k1[c] + Rkf45::b3 * k3[c] + Rkf45::b4 * k4[c] + Rkf45::b5 * k5[c];
            e[c] = Rkf45::d1 * k1[c] + Rkf45::d3 * k3[c] + Rkf45::d4 * k4[c] + Rkf45::d5 * k5[c] + Rkf45::d6 * k6[c];
        }
        return true;
    }
};

// ---------------------------------------------------------------------------------------
// per-reactor driver (Algorithm 1 on one wavefront)
// ---------------------------------------------------------------------------------------
template <int RPL>
__device__ __forceinline__ double wrms_wave(int N, const double (&e)[RPL], const double (&a)[RPL], const double (&b)[RPL],
                            double rtol, double atol) {
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < RPL; c++) {
        const int i = lane_id() + 64 * c;
        if (i < N) {
            const double sc = atol + rtol * fmax(fabs(a[c]), fabs(b[c]));
            const double r = e[c] / sc;
            s += r * r;
        }
    }
    return sqrt(wsum(s) / N);
}

template <int RPL>
__device__ __forceinline__ bool all_finite(int N, const double (&v)[RPL]) {
    bool ok = true;
#pragma unroll
    for (int c = 0; c < RPL; c++) ok = ok && (lane_id() + 64 * c >= N || isfinite(v[c]));
    return wave_all(ok);
}

// Step adapters with a common (array) interface.
template <int NP>
struct Ros4Adapter {
    static constexpr int RPL = 1;
    static constexpr int NSMAX = NP - 1;
    static constexpr LdsKind LDS = kLdsJac;
    static constexpr int LDJ = WaveShape<NP>::LDJ;
    static constexpr int kJc = NP * LDJ > WTile<NP>::kScratch ? NP * LDJ : WTile<NP>::kScratch;
    static constexpr bool PARK = WaveShape<NP>::PARK;
    static constexpr int PARK_ROWS = NP;
    static constexpr double qinv = 0.25;
    __device__ static __forceinline__ bool step(const DevMech &M, const Lds &L, const double (&y)[1], double P, double h,
                                double (&yn)[1], double (&e)[1], const IntOpts &, int &) {
        return Ros4Wave<NP>::step(M, L, y[0], P, h, yn[0], e[0]);
    }
};

template <int NP>
struct Ros4AdapterFD {
    static constexpr int RPL = 1;
    static constexpr int NSMAX = NP - 1;
    static constexpr LdsKind LDS = kLdsTiles;      // no d wdot/dC staging: only source-term evaluations
    static constexpr int LDJ = 0;
    static constexpr int kJc = WTile<NP>::kScratch;
    static constexpr bool PARK = true;
    static constexpr int PARK_ROWS = NP;
    static constexpr double qinv = 0.25;
    __device__ static __forceinline__ bool step(const DevMech &M, const Lds &L, const double (&y)[1], double P,
                                                double h, double (&yn)[1], double (&e)[1], const IntOpts &o, int &) {
        return Ros4WaveFD<NP>::step(M, L, y[0], P, h, yn[0], e[0], o);
    }
};

template <int NP>
struct Ros4Adapter32 : Ros4Adapter<NP> {
    __device__ static __forceinline__ bool step(const DevMech &M, const Lds &L, const double (&y)[1], double P, double h,
                                double (&yn)[1], double (&e)[1], const IntOpts &o, int &fb) {
        return Ros4Wave32<NP>::step(M, L, y[0], P, h, yn[0], e[0], o.refine_sweeps, fb);
    }
};

template <class S>
__device__ __forceinline__ void integrate_reactor(const DevMech &M, const Lds &L, int64_t r, double *y, int64_t ld, const double *p,
                                  const double *t_end, double *t_io, double *h_io, const IntOpts &o, int32_t *status,
                                  int32_t *nacc, int32_t *nrej) {
    constexpr int RPL = S::RPL;
    const int N = M.N;
    const int lane = lane_id();
    double yv[RPL];
#pragma unroll
    for (int c = 0; c < RPL; c++) {
        const int i = lane + 64 * c;
        yv[c] = i < N ? y[int64_t(i) * ld + r] : 0.0;
    }
    const double P = p[r];
    const double te = t_end[r];
    double t = t_io ? t_io[r] : 0.0;
    double h = h_io ? h_io[r] : 0.0;
    int st = CK_ST_OK;
    int na = 0, nj = 0, fb = 0;
    if (!all_finite<RPL>(N, yv)) {
        st = CK_ST_NONFINITE;
        h = 0.0;
    } else if (o.h_fixed > 0.0) {
        h = o.h_fixed;
    } else if (!(h > 0.0)) {
        if (o.h0 > 0.0) {
            h = o.h0;
        } else if (t < te) {
            // EstimateH0 (Hairer, Norsett & Wanner II.4, order 4)
            double f0[RPL], f1[RPL], yt[RPL];
            rhs_wave<RPL>(M, L, yv, P, f0);
            if (!all_finite<RPL>(N, f0)) {
                st = CK_ST_NONFINITE;
                h = 0.0;
            } else {
                double s0 = 0.0, s1 = 0.0;
#pragma unroll
                for (int c = 0; c < RPL; c++) {
                    if (lane + 64 * c < N) {
                        const double sc = o.atol + o.rtol * fabs(yv[c]);
                        s0 += (yv[c] / sc) * (yv[c] / sc);
                        s1 += (f0[c] / sc) * (f0[c] / sc);
                    }
                }
                const double d0 = sqrt(wsum(s0) / N), d1 = sqrt(wsum(s1) / N);
                const double span = te - t;
                double h0 = (d0 < 1e-5 || d1 < 1e-5) ? 1e-6 : 0.01 * d0 / d1;
                h0 = fmin(h0, span);
#pragma unroll
                for (int c = 0; c < RPL; c++) yt[c] = yv[c] + h0 * f0[c];
                rhs_wave<RPL>(M, L, yt, P, f1);
                double s2 = 0.0;
#pragma unroll
                for (int c = 0; c < RPL; c++) {
                    if (lane + 64 * c < N) {
                        const double sc = o.atol + o.rtol * fabs(yv[c]);
                        const double v = (f1[c] - f0[c]) / sc;
                        s2 += v * v;
                    }
                }
                const double d2 = sqrt(wsum(s2) / N) / h0;
                const double dm = fmax(d1, d2);
                const double h1 = dm <= 1e-15 ? fmax(1e-6, h0 * 1e-3) : pow(0.01 / dm, 0.2);
                h = fmin(fmin(100.0 * h0, h1), span);
            }
        }
    }
    if (st == CK_ST_OK) {
        while (t < te) {
            if (int64_t(na) + nj >= o.max_steps) {
                st = CK_ST_MAX_STEPS;
                break;
            }
            const bool clipped = (t + h >= te);
            const double hs = clipped ? te - t : h;
            double yn[RPL], e[RPL];
            const bool ok = S::step(M, L, yv, P, hs, yn, e, o, fb);
            double err;
            if (o.h_fixed > 0.0)
                err = 0.0;
            else if (!ok)
                err = INFINITY;
            else {
                err = wrms_wave<RPL>(N, e, yv, yn, o.rtol, o.atol);
                if (!all_finite<RPL>(N, yn)) err = INFINITY;
            }
            const bool acc = err < 1.0;
            if (acc) {
#pragma unroll
                for (int c = 0; c < RPL; c++) yv[c] = yn[c];
                t = clipped ? te : t + hs;
                na++;
            } else {
                nj++;
            }
            const double fac = o.h_fixed > 0.0 ? 1.0 : step_factor(err, S::qinv, acc);
            h = hs * fac;
            if (t < te && h < h_floor(t)) {
                st = CK_ST_H_UNDERFLOW;
                break;
            }
        }
    }
#pragma unroll
    for (int c = 0; c < RPL; c++) {
        const int i = lane + 64 * c;
        if (i < N) y[int64_t(i) * ld + r] = yv[c];
    }
    if (lane == 0) {
        if (t_io) t_io[r] = t;
        if (h_io) h_io[r] = h;
        status[r] = st;
        nacc[r] = na;
        nrej[r] = nj;
        if (o.n_fallback) o.n_fallback[r] = fb;
    }
}

template <int R>
struct Rkf45S {
    static constexpr int RPL = R;
    static constexpr int NSMAX = 64 * R - 1;
    static constexpr LdsKind LDS = kLdsRhs;
    static constexpr int LDJ = 0;
    static constexpr int kJc = 0;
    static constexpr bool PARK = false;
    static constexpr int PARK_ROWS = 0;
    static constexpr double qinv = 0.2;
    __device__ static __forceinline__ bool step(const DevMech &M, const Lds &L, const double (&y)[R], double P, double h,
                                double (&yn)[R], double (&e)[R], const IntOpts &, int &) {
        return Rkf45Wave<R>::step(M, L, y, P, h, yn, e);
    }
};

// Consecutive workgroups are dispatched round-robin over the 8 XCDs; map them so that
// the reactors handled on one XCD are contiguous (their state shares L2 lines).  The grid
// is a multiple of 8 workgroups, which makes the map a permutation of [0, nb).
__device__ __forceinline__ int64_t xcd_reactor(int64_t b, int64_t nb) {
    const int64_t per = nb / 8;
    const int64_t x = b % 8, i = b / 8;
    return x * per + i;
}

}  // namespace

// ---------------------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------------------
template <int RPL, bool GEN>
__global__ void __launch_bounds__(64) rhs_wave_kernel(DevMech M, int64_t n, const double *y, int64_t ld,
                                                      const double *p, double *dydt, int cv) {
    // laid out for the largest species count of the instantiation, so every offset is a constant
    __shared__ double lds_raw[4 * 64 * RPL];
    Lds L = carve(lds_raw, kLdsRhs, 64 * RPL - 1, 0);
    L.cv = cv;
    init_lds<RPL>(M, L, kLdsRhs);
    const int N = M.N, lane = lane_id();
    const int64_t nb = int64_t(gridDim.x);
    const int64_t r = xcd_reactor(blockIdx.x, nb);
    if (r >= n) return;
    double yv[RPL], f[RPL];
#pragma unroll
    for (int c = 0; c < RPL; c++) {
        const int i = lane + 64 * c;
        yv[c] = i < N ? y[int64_t(i) * ld + r] : 0.0;
    }
    rhs_wave<RPL, GEN>(M, L, yv, p[r], f);
#pragma unroll
    for (int c = 0; c < RPL; c++) {
        const int i = lane + 64 * c;
        if (i < N) dydt[int64_t(i) * ld + r] = f[c];
    }
}

// Standalone Jacobian for N <= 64: workgroups of eight wavefronts, one reactor each, d wdot/dC staged
// in windows of WIN matrix columns (the temperature column is column 0).  Bound by the stores: an entry
// of a reactor is eight bytes of a line that it shares with fifteen neighbours, so the eight staged
// windows are written out together, eight neighbouring reactors by one store (64 bytes), instead of
// one reactor at a time (a line per lane).  Rates are evaluated again for a later window.
template <int NSMAX, int WIN>
struct JacShape {
    static constexpr int R = 8;                     // reactors of a workgroup
    static constexpr int LDJ = WIN | 1;
    static constexpr int NWIN = (NSMAX + 1 + WIN - 1) / WIN;
    static constexpr int kSlab0 = 8 * (NSMAX + 1) + (NSMAX + 1) * LDJ;
    // slab stride 8 modulo 32 doubles: the eight reactors of a store read different banks
    static constexpr int kSlab = kSlab0 + (8 - kSlab0 % 32 + 32) % 32;
    static constexpr size_t kLds = size_t(R) * kSlab + 2 * (NSMAX + 1);
};
template <int NSMAX, int WIN>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 4))) jac_wave_kernel(DevMech M, int64_t n, const double *y,
                                                       int64_t ld, const double *p, double *jac, int cv) {
    using SH = JacShape<NSMAX, WIN>;
    extern __shared__ double lds_raw[];
    const int N = M.N, ns = M.nsp, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    const int64_t r0 = xcd_reactor(blockIdx.x, int64_t(gridDim.x)) * SH::R;
    if (r0 >= n) return;
    double *W = lds_raw + SH::R * SH::kSlab, *IW = W + NSMAX + 1;
    // null species, W by matrix row (1 for the temperature row) and 1/W by matrix column
    Lds L;
    double *b = lds_raw + wave * SH::kSlab;
    double *const fields[7] = {b, b + (NSMAX + 1), b + 2 * (NSMAX + 1), b + 3 * (NSMAX + 1), b + 4 * (NSMAX + 1),
                               b + 5 * (NSMAX + 1), b + 6 * (NSMAX + 1)};
    L.C = fields[0];
    L.G = fields[1];
    L.H = fields[2];
    L.WD = fields[3];
    L.TB = fields[4];
    L.DWT = fields[5];
    L.HC = fields[6];
    L.TROW = b + 7 * (NSMAX + 1);
    L.JC = b + 8 * (NSMAX + 1);
    L.ldj = SH::LDJ;
    L.cv = cv;
    init_lds<1>(M, L, kLdsRhs);
    for (int e = int(threadIdx.x); e < N; e += 512) {
        W[e] = e == 0 ? 1.0 : M.W()[e - 1];
        IW[e] = e == 0 ? 1.0 : M.invW()[e - 1];
    }
    const int64_t r = min(r0 + wave, n - 1);         // the last workgroup's idle wavefronts repeat a reactor
    const double yl = lane < N ? y[int64_t(lane) * ld + r] : 0.0;
    const double yy[1] = {yl};
    double ff[1];
    Mix<1> x;
    const PairRec first = first_pair<64>(M, lane);
    zero_jc(L, ns);
    species_pass<1, true>(M, yy, p[r], L, x);
    const RxScale sc = rx_scale(L, x);
    reaction_pass<64, true>(M, L, x.t, x.Ctot, sc, -1, min(WIN, N), kRates, nullptr, lane, first);
    __syncthreads();
    finish_rhs<1>(M, L, x, ff);
    const Chain c = chain_rule(M, L, x, yl, bcast(ff[0], 0));
    __syncthreads();
    // per-row scalars in place of the sums: W beta in TB, W col0 in DWT, by species; the temperature row
    if (L.sl[0].valid) {
        const int k = L.sl[0].k;
        L.TB[k] = L.sl[0].W * c.beta;
        L.DWT[k] = L.sl[0].W * c.col0;
        L.TROW[1 + k] = c.trow;
    }
    if (lane == 0) L.TROW[0] = c.J00;
    for (int w = 0; w < SH::NWIN; w++) {
        if (w > 0) {
            if (w * WIN >= N) break;
            zero_jc(L, ns);
            __syncthreads();
            const PairRec again = first_pair<64>(M, lane);
            reaction_pass<64, true>(M, L, x.t, x.Ctot, sc, w * WIN - 1, min(WIN, N - w * WIN), kScatter, nullptr, lane,
                                    again);
        }
        __syncthreads();
        const int s = int(threadIdx.x) & 7;
        const double *slab = lds_raw + s * SH::kSlab;
        const int cols = min(WIN, N - w * WIN);
        if (r0 + s < n)
            for (int e = int(threadIdx.x) >> 3; e < N * WIN; e += 64) {
                const int i = e / WIN, jj = e % WIN, j = w * WIN + jj;
                if (jj >= cols) continue;
                double v;
                if (i == 0) v = IW[j] * slab[7 * (NSMAX + 1) + j];
                else if (j == 0) v = slab[5 * (NSMAX + 1) + i - 1];
                else v = IW[j] * fma(W[i], slab[8 * (NSMAX + 1) + (i - 1) * SH::LDJ + jj], slab[4 * (NSMAX + 1) + i - 1]);
                jac[(int64_t(i) * N + j) * ld + r0 + s] = v;
            }
        __syncthreads();
    }
}

template <class S>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) integrate_wave_kernel(DevMech M, int64_t n, double *y, int64_t ld,
                                                            const double *p, const double *t_end, double *t_io,
                                                            double *h_io, IntOpts o, unsigned *queue,
                                                            double *park, int32_t *status, int32_t *nacc,
                                                            int32_t *nrej) {
    // LDS laid out for the largest species count of the instantiation: every offset is a
    // compile-time constant, so LDS addresses need no scalar registers
    extern __shared__ double lds_raw[];
    Lds L = carve(lds_raw, S::LDS, S::NSMAX, S::LDJ);
    L.cv = o.reactor;
    if (S::PARK) L.park = park + size_t(blockIdx.x) * (size_t(S::PARK_ROWS) * 64);
    init_lds<S::RPL>(M, L, S::LDS);
    for (;;) {
        unsigned v = 0;
        if (lane_id() == 0) v = atomicAdd(queue, 1u);
        const int64_t r = int64_t(unsigned(__builtin_amdgcn_readfirstlane(int(v))));
        if (r >= n) break;
        integrate_reactor<S>(M, L, r, y, ld, p, t_end, t_io, h_io, o, status, nacc, nrej);
        __syncthreads();
    }
}

__global__ void zero_u32_kernel(unsigned *q) { *q = 0u; }

// ---------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------
namespace {
int pad_np(int N) { return ((N + 7) / 8) * 8; }

// Resident wavefronts per CU are capped so that parked LU rows fit the workspace.
constexpr int kWaveMaxPerCu = 8;

template <class S>
int launch_int(const DevMech &M, int64_t n, double *y, int64_t ld, const double *p, const double *t_end, double *t,
               double *h, const IntOpts &o, unsigned *queue, int32_t *status, int32_t *nacc, int32_t *nrej,
               hipStream_t s) {
    if (M.nsp > S::NSMAX) return CK_EUNSUPPORTED;
    const size_t lds = lds_doubles(S::LDS, S::NSMAX, S::kJc) * sizeof(double);
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess) return CK_EHIP;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return CK_EHIP;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, integrate_wave_kernel<S>, 64, lds) != hipSuccess || per < 1)
        return CK_EHIP;
    if (o.blocks_per_cu > 0 && o.blocks_per_cu < per) per = o.blocks_per_cu;
    if (per > kWaveMaxPerCu) per = kWaveMaxPerCu;
    int64_t grid = int64_t(cus) * per;
    if (grid > n) grid = n;
    double *park = S::PARK ? reinterpret_cast<double *>(reinterpret_cast<char *>(queue) + 256) : nullptr;
    zero_u32_kernel<<<1, 1, 0, s>>>(queue);
    integrate_wave_kernel<S><<<dim3(unsigned(grid)), dim3(64), lds, s>>>(M, n, y, ld, p, t_end, t, h, o, queue,
                                                                          park, status, nacc, nrej);
    return hipGetLastError() == hipSuccess ? CK_OK : CK_EHIP;
}
}  // namespace

namespace {
template <int NSMAX, int WIN>
int launch_jac(const DevMech &M, int64_t n, const double *y, int64_t ld, const double *p, double *jac, int cv,
               hipStream_t s) {
    using SH = JacShape<NSMAX, WIN>;
    if (M.nsp > NSMAX) return CK_EUNSUPPORTED;
    const size_t lds = SH::kLds * sizeof(double);
    auto kern = jac_wave_kernel<NSMAX, WIN>;
    if (lds > 64 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)) != hipSuccess)
        return CK_EHIP;
    const int64_t groups = (n + SH::R - 1) / SH::R;
    kern<<<dim3(unsigned((groups + 7) / 8 * 8)), dim3(512), lds, s>>>(M, n, y, ld, p, jac, cv);
    return hipGetLastError() == hipSuccess ? CK_OK : CK_EHIP;
}
}  // namespace

bool wave_supported(const DevMech &M, int method, int precision) {
    if (method == 0) return M.N <= 64;
    return precision == CK_PREC_FP64 && M.N <= 128;
}

size_t wave_ws_bytes(const DevMech &M, int cus) {
    // parked FP64 rows of every resident wavefront (FP64 ROS4 with NP > 32, or any NP <= 64 with
    // the forward-difference Jacobian)
    const int np = pad_np(M.N);
    if (np > 64) return 256;
    return 256 + size_t(cus) * kWaveMaxPerCu * size_t(np) * 64 * sizeof(double);
}

int launch_rhs_wave(const DevMech &M, int64_t n, const double *y, int64_t ld, const double *p, double *dydt,
                    int cv, hipStream_t s) {
    const unsigned grid = unsigned((n + 7) / 8 * 8);
    // the general-form code needs 20 more registers than the rest: a kernel of its own
    auto kern = M.N <= 64 ? (M.n_gen > 0 ? rhs_wave_kernel<1, true> : rhs_wave_kernel<1, false>)
                          : (M.n_gen > 0 ? rhs_wave_kernel<2, true> : rhs_wave_kernel<2, false>);
    kern<<<dim3(grid), dim3(64), 0, s>>>(M, n, y, ld, p, dydt, cv);
    return hipGetLastError() == hipSuccess ? CK_OK : CK_EHIP;
}

int launch_jac_wave(const DevMech &M, int64_t n, const double *y, int64_t ld, const double *p, double *jac,
                    int cv, hipStream_t s) {
    if (M.N > 64) return cv ? CK_EUNSUPPORTED : launch_jac_coop(M, n, y, ld, p, jac, s);
    if (M.N <= 16) return launch_jac<15, 16>(M, n, y, ld, p, jac, cv, s);
    if (M.N <= 32) return launch_jac<31, 32>(M, n, y, ld, p, jac, cv, s);
    if (M.N <= 56) return launch_jac<55, 32>(M, n, y, ld, p, jac, cv, s);
    return launch_jac<63, 24>(M, n, y, ld, p, jac, cv, s);      // eight windows of 32 columns exceed the LDS
}

int launch_integrate_wave(int method, const DevMech &M, int64_t n, double *y, int64_t ld, const double *p,
                          const double *t_end, double *t, double *h, const IntOpts &o, void *ws, int32_t *status,
                          int32_t *nacc, int32_t *nrej, hipStream_t s) {
    unsigned *q = static_cast<unsigned *>(ws);
    if (method == 1) {
        if (M.N <= 64) return launch_int<Rkf45S<1>>(M, n, y, ld, p, t_end, t, h, o, q, status, nacc, nrej, s);
        return launch_int<Rkf45S<2>>(M, n, y, ld, p, t_end, t, h, o, q, status, nacc, nrej, s);
    }
    if (o.jacobian == CK_JAC_FD) {
        if (o.precision != CK_PREC_FP64) return CK_EUNSUPPORTED;
        switch (pad_np(M.N)) {
#define CK_CASEFD(NPV) \
    case NPV: return launch_int<Ros4AdapterFD<NPV>>(M, n, y, ld, p, t_end, t, h, o, q, status, nacc, nrej, s);
            CK_CASEFD(8) CK_CASEFD(16) CK_CASEFD(24) CK_CASEFD(32) CK_CASEFD(40) CK_CASEFD(48) CK_CASEFD(56)
            CK_CASEFD(64)
#undef CK_CASEFD
            default: return CK_EUNSUPPORTED;
        }
    }
    if (o.precision == CK_PREC_FP32_REFINE) {
        switch (pad_np(M.N)) {
#define CK_CASE32(NPV) \
    case NPV: return launch_int<Ros4Adapter32<NPV>>(M, n, y, ld, p, t_end, t, h, o, q, status, nacc, nrej, s);
            CK_CASE32(8) CK_CASE32(16) CK_CASE32(24) CK_CASE32(32) CK_CASE32(40) CK_CASE32(48) CK_CASE32(56)
            CK_CASE32(64)
#undef CK_CASE32
            default: return CK_EUNSUPPORTED;
        }
    }
    switch (pad_np(M.N)) {
        case 8: return launch_int<Ros4Adapter<8>>(M, n, y, ld, p, t_end, t, h, o, q, status, nacc, nrej, s);
        case 16: return launch_int<Ros4Adapter<16>>(M, n, y, ld, p, t_end, t, h, o, q, status, nacc, nrej, s);
        case 24: return launch_int<Ros4Adapter<24>>(M, n, y, ld, p, t_end, t, h, o, q, status, nacc, nrej, s);
        case 32: return launch_int<Ros4Adapter<32>>(M, n, y, ld, p, t_end, t, h, o, q, status, nacc, nrej, s);
        case 40: return launch_int<Ros4Adapter<40>>(M, n, y, ld, p, t_end, t, h, o, q, status, nacc, nrej, s);
        case 48: return launch_int<Ros4Adapter<48>>(M, n, y, ld, p, t_end, t, h, o, q, status, nacc, nrej, s);
        case 56: return launch_int<Ros4Adapter<56>>(M, n, y, ld, p, t_end, t, h, o, q, status, nacc, nrej, s);
        case 64: return launch_int<Ros4Adapter<64>>(M, n, y, ld, p, t_end, t, h, o, q, status, nacc, nrej, s);
        default: return CK_EUNSUPPORTED;
    }
}

}  // namespace ck
