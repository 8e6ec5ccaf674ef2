// Wavefront-per-reactor device code.  One 64-lane wavefront owns one reactor:
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
#pragma once

#include "ck_internal.h"
#include "kinetics.h"
#include "launch.h"
#include "reactions.h"
#include "wtile.h"

extern "C" __device__ unsigned long long __ockl_wfred_max_u64(unsigned long long);

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
__device__ __forceinline__ double bcast(double v, int src) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), src);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), src);
    return __hiloint2double(hi, lo);
}
// Sums over the wavefront, up to four at a time: the first two steps fold different values into the
// lane halves and rows, so four sums take seven additions and the latency of one (RKF45 M53 x 8191
// 26.3 -> 25.0 ms, ROS4 M53 x 5 41.7 -> 41.2 ms).
template <int CTRL>
__device__ __forceinline__ double row_add(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row_sum(double v) {        // row_ror 1, 2, 4, 8
    return row_add<0x128>(row_add<0x124>(row_add<0x122>(row_add<0x121>(v))));
}
__device__ __forceinline__ double wsum(double v) {
    const double h = wt_fold32(v, v);
    return bcast(row_sum(wt_fold16(h, h)), 0);
}
__device__ __forceinline__ void wsum(double &a, double &b) {
    const double h = wt_fold32(a, b), r = row_sum(wt_fold16(h, h));
    a = bcast(r, 0);
    b = bcast(r, 32);
}
__device__ __forceinline__ void wsum(double &a, double &b, double &c, double &d) {
    const double r = row_sum(wt_fold16(wt_fold32(a, b), wt_fold32(c, d)));
    a = bcast(r, 0);
    b = bcast(r, 32);
    c = bcast(r, 16);
    d = bcast(r, 48);
}
__device__ __forceinline__ bool wave_all(bool v) { return __ballot(!v) == 0ull; }

// ---------------------------------------------------------------------------------------
// LDS layout of one wavefront (doubles), ns1 = ns + 1 (a null species closes every array):
//   C G H WD [ns1]                                   every kernel
//   | scratch of the tiles                           kLdsTiles (ROS4 with another Jacobian)
//   | TB DWT HC [ns1] TROW JC                        kLdsJac (ROS4): JC holds d wdot / dC for a window
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
    static constexpr int TR = WTile<NP>::TR, RPL = WTile<NP>::ROWS;
    static constexpr int NWIN = (TR + 1) / 2;
    static constexpr int WIN = TR > 1 ? 32 : 16;
    static constexpr int LDJ = WIN | 1;
    static constexpr int ZERO = 16 * TR;       // offset of the zeros in TROW
    static constexpr bool PARK = NWIN > 1;     // the first window's rate scalars wait for the others
    static constexpr int kJc = NP * LDJ > WTile<NP>::kScratch ? NP * LDJ : WTile<NP>::kScratch;
};
__host__ __device__ inline int trow_doubles(int ns) { return (ns + 16) / 16 * 16 + 32; }

// jc: doubles of the JC region (kLdsTiles, kLdsJac)
__host__ __device__ inline size_t lds_doubles(LdsKind kind, int ns, size_t jc) {
    size_t d = 4 * size_t(ns + 1);
    if (kind == kLdsTiles) d += jc;
    if (kind == kLdsJac) d += 3 * size_t(ns + 1) + trow_doubles(ns) + jc;
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
        L.TROW = b; b += trow_doubles(ns);
        L.JC = b;
    }
    L.park = nullptr;
    L.cv = 0;
    return L;
}

template <int RPL>
__device__ __forceinline__ void init_lds(const DevMech &M, Lds &L, LdsKind kind, int nsmax = 0) {
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
        for (int e = l; e < trow_doubles(nsmax); e += 64) L.TROW[e] = 0.0;
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
    Thermo th[RPL];
    x.t = tpow(T);
    double S = 0.0, cpm = 0.0;          // sum_k Y_k / W_k, mixture c_p / R
#pragma unroll
    for (int c = 0; c < RPL; c++) {
        co[c] = species_coef(M, L.sl[c].k, T < L.sl[c].Tmid);
        z[c] = L.sl[c].valid ? y[c] * L.sl[c].iW : 0.0;
        th[c] = species_thermo(M, co[c], x.t);
        S += z[c];
        cpm = fma(z[c], th[c].cp, cpm);
    }
    wsum(S, cpm);
    x.cpm = cpm * M.R;
    x.Wbar = ck_rcp(S);
    if (L.cv) {   // constant volume: P holds the (fixed) density
        x.rho = P;
        x.Ctot = P * S;
    } else {
        x.Ctot = P * x.t.invT * M.invR;
        x.rho = x.Ctot * x.Wbar;
    }
    x.invrho = ck_rcp(x.rho);
#pragma unroll
    for (int c = 0; c < RPL; c++) {
        x.cp[c] = th[c].cp;
        x.h[c] = th[c].h;
        if (JAC) x.dcp[c] = th[c].dcp;
        if (L.sl[c].valid) {
            const int k = L.sl[c].k;
            L.C[k] = x.rho * z[c];
            L.G[k] = th[c].g;
            L.WD[k] = 0.0;
            if (JAC) {
                L.H[k] = th[c].h - 1.0;
                L.TB[k] = 0.0;
                L.DWT[k] = 0.0;
                L.HC[k] = 0.0;
            }
        }
    }
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

template <int RPL>
__device__ __forceinline__ RxScale rx_scale(const Lds &L, const Mix<RPL> &x) {
    return L.cv ? RxScale{0.0, 0.0, 0.0} : RxScale{x.t.invT, x.Wbar * x.invrho, 1.0};
}

// Chain rule for the lane's species rows k and their entries of the temperature row, in the specific
// mole numbers z = Y / W (J' of ChainIn): J'[k+1][0] = col0, J'[k+1][1+j] = JC[k][j] + beta,
// J'[0][1+k] = trow, J'[0][0] = J00.
template <int RPL>
struct Chain {
    double beta[RPL], col0[RPL], trow[RPL], J00;
};
template <int RPL>
__device__ __forceinline__ Chain<RPL> chain_rule(const DevMech &M, const Lds &L, const Mix<RPL> &x,
                                                 const double (&y)[RPL], double fT) {
    const bool cv = L.cv != 0;
    const double e = cv ? 1.0 : 0.0;
    Chain<RPL> o;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll
    for (int c = 0; c < RPL; c++) {
        const bool valid = L.sl[c].valid;
        const int k = L.sl[c].k;
        const double TBk = valid ? L.TB[k] : 0.0, WDk = valid ? L.WD[k] : 0.0, DWTk = valid ? L.DWT[k] : 0.0;
        const double Hk = x.h[c] - e;                               // over R T
        s0 = fma(Hk, TBk, s0);
        s1 = fma(Hk, WDk, s1);
        s2 += fma(x.cp[c] - e, WDk, Hk * (x.t.T * DWTk - (cv ? 0.0 : WDk)));
        s3 += valid ? y[c] * x.dcp[c] * L.sl[c].iW : 0.0;
        o.beta[c] = TBk;
        o.col0[c] = DWTk * x.invrho;
    }
    ChainIn c;
    c.rho = x.rho;
    c.Wbar = x.Wbar;
    c.invT = x.t.invT;
    c.R = M.R;
    c.RT = M.R * x.t.T;
    c.cpm = x.cpm;
    c.fT = fT;
    wsum(s0, s1, s2, s3);
    c.sHB = c.RT * s0;
    c.sHW = c.RT * s1;
    c.dQT = M.R * s2;
    c.sdcp = M.R * s3;
#pragma unroll
    for (int q = 0; q < RPL; q++) o.trow[q] = L.sl[q].valid ? chain_trow(c, cv, L.HC[L.sl[q].k], x.cp[q]) : 0.0;
    o.J00 = chain_J00(c, cv);
    return o;
}

// f(y) and the tiles of M' = dg I - J' (J' the Jacobian in the specific mole numbers, similar to J by
// diag(1, W)) for N <= NP <= 112.  The first window's reaction pass also leaves every per-species sum
// of the chain rule, so each window's columns are final when they are read.  The other windows take
// the first one's rate constants from the park slice when they fit (else they evaluate them again).
// iw and w: 1/W and W of the lane's components (1 for T, 0 for padding).
template <int NP>
__device__ __forceinline__ void jac_tiles(const DevMech &M, const Lds &L, const double (&y)[WaveShape<NP>::RPL],
                                          double P, double dg, wd4 (&X)[WTile<NP>::TR][WTile<NP>::TR],
                                          double (&f)[WaveShape<NP>::RPL], double (&iw)[WaveShape<NP>::RPL],
                                          double (&w)[WaveShape<NP>::RPL]) {
    using SH = WaveShape<NP>;
    constexpr int TR = SH::TR, NWIN = SH::NWIN, WIN = SH::WIN, RPL = SH::RPL;
    Mix<RPL> x;
    const int ns = M.nsp;
    const PairRec first = first_pair<64>(M, lane_fresh());
    zero_jc(L, ns);
    species_pass<RPL, true>(M, y, P, L, x);
    const RxScale sc = rx_scale<RPL>(L, x);
    const bool fits = NWIN > 1 && 3 * rx_blocks(M, 64) <= NP;
    reaction_pass<64, true>(M, L, x.t, x.Ctot, sc, -1, min(WIN, ns + 1), fits ? kRatesKeep : kRates,
                            L.park + lane_fresh(), lane_fresh(), first);
    __syncthreads();
    finish_rhs<RPL>(M, L, x, f);
    const Chain<RPL> ch = chain_rule<RPL>(M, L, x, y, bcast(f[0], 0));
    const int lane = lane_fresh();
    const int g = lane >> 4, c16 = lane & 15;
#pragma unroll
    for (int c = 0; c < RPL; c++) {
        const SpeciesLane &sl = L.sl[c];
        if (sl.valid) {
            L.TROW[1 + sl.k] = ch.trow[c];
            L.JC[sl.k * SH::LDJ] = ch.col0[c];
        }
        w[c] = lane + 64 * c == 0 ? 1.0 : (sl.valid ? sl.W : 0.0);
        iw[c] = lane + 64 * c == 0 ? 1.0 : (sl.valid ? sl.iW : 0.0);
    }
    if (lane == 0) L.TROW[0] = ch.J00;
    __syncthreads();
    double dgm[4];
#pragma unroll
    for (int v = 0; v < 4; v++) dgm[v] = c16 == g + 4 * v ? dg : 0.0;
    const int nsw = opaque_s(ns);
    auto next_window = [&](int wnd) {
        const PairRec again = first_pair<64>(M, lane_fresh());
        __syncthreads();
        zero_jc(L, ns);
        __syncthreads();
        reaction_pass<64, true>(M, L, x.t, x.Ctot, sc, WIN * wnd - 1, min(WIN, ns + 1 - WIN * wnd),
                                fits ? kScatterKept : kScatter, L.park + lane_fresh(), lane_fresh(), again);
        __syncthreads();
    };
    auto tiles = [&](auto wi) {
        constexpr int wnd = decltype(wi)::value;
#pragma unroll
        for (int I = 0; I < TR; I++) {
            // matrix row 16 I + c: the temperature row, a species row or padding (zeros)
            const int r = 16 * I + c16;
            const bool sp = r >= 1 && r <= nsw;
            const double *row = sp ? &L.JC[(r - 1) * SH::LDJ] : (r == 0 ? L.TROW + WIN * wnd : L.TROW + SH::ZERO);
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
                    constexpr int pad = NP > 64 ? 16 : 8;
                    const double b = c0 == 0 ? (g == 0 ? 0.0 : beta) : (c0 + 3 < NP - pad || c0 + g <= nsw ? beta : 0.0);
                    X[J][I][v] = ((I == J ? dgm[v] : 0.0) - b) - row[c0 - WIN * wnd + g];
                }
        }
    };
    tiles(std::integral_constant<int, 0>{});
    if constexpr (NWIN == 2) {
        next_window(1);
        tiles(std::integral_constant<int, 1>{});
    } else if constexpr (NWIN > 2) {
        // one copy of the reaction pass for the later windows
#pragma unroll 1
        for (int wnd = 1; wnd < NWIN; wnd++) {
            next_window(wnd);
            wt_for<1, NWIN>([&](auto wi) {
                if (wnd == decltype(wi)::value) tiles(wi);
            });
        }
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------------------
// one steps
// ---------------------------------------------------------------------------------------
// Stages of a ROS4 step: solve(b, u) returns u = M^-1 b.
template <int RPL, class Solve>
__device__ __forceinline__ void ros4_stages(const DevMech &M, const Lds &L, const double (&y)[RPL], double P, double h,
                                            const double (&f)[RPL], const Solve &solve, double (&ynew)[RPL],
                                            double (&e)[RPL]) {
    const double ih = 1.0 / h;
    double u1[RPL], u2[RPL], u3[RPL], u4[RPL], yt[RPL], ft[RPL], b[RPL];
    if (!solve(f, u1)) return;
    // the inverse stays in registers across the stage source terms
#pragma unroll
    for (int c = 0; c < RPL; c++) yt[c] = y[c] + Ros4::a21 * u1[c];
    rhs_wave<RPL>(M, L, yt, P, ft);
#pragma unroll
    for (int c = 0; c < RPL; c++) b[c] = ft[c] + (Ros4::c21 * u1[c]) * ih;
    if (!solve(b, u2)) return;
#pragma unroll
    for (int c = 0; c < RPL; c++) yt[c] = y[c] + Ros4::a31 * u1[c] + Ros4::a32 * u2[c];
    rhs_wave<RPL>(M, L, yt, P, ft);
#pragma unroll
    for (int c = 0; c < RPL; c++) b[c] = ft[c] + (Ros4::c31 * u1[c] + Ros4::c32 * u2[c]) * ih;
    if (!solve(b, u3)) return;
#pragma unroll
    for (int c = 0; c < RPL; c++) b[c] = ft[c] + (Ros4::c41 * u1[c] + Ros4::c42 * u2[c] + Ros4::c43 * u3[c]) * ih;
    if (!solve(b, u4)) return;
#pragma unroll
    for (int c = 0; c < RPL; c++) {
        ynew[c] = y[c] + Ros4::m1 * u1[c] + Ros4::m2 * u2[c] + Ros4::m3 * u3[c] + Ros4::m4 * u4[c];
        e[c] = Ros4::e1 * u1[c] + Ros4::e2 * u2[c] + Ros4::e3 * u3[c] + Ros4::e4 * u4[c];
    }
}

// Solve with the inverted tiles of M in the variables z = y / w: iw scales a right-hand side, w a solution.
template <int NP, int PJ = 0>
__device__ __forceinline__ bool tile_solve(const wd4 (&X)[WTile<NP>::TR][WTile<NP>::TR], const WScratch &s,
                                           const int (&ord)[WTile<NP>::ROWS], const double (&iw)[WTile<NP>::ROWS],
                                           const double (&w)[WTile<NP>::ROWS], const double (&b)[WTile<NP>::ROWS],
                                           double (&u)[WTile<NP>::ROWS], const double *park = nullptr) {
    double bz[WTile<NP>::ROWS], z[WTile<NP>::ROWS];
#pragma unroll
    for (int c = 0; c < WTile<NP>::ROWS; c++) bz[c] = iw[c] * b[c];
    wt_solve<NP, double, PJ>(X, s, lane_fresh(), ord, bz, z, park);
#pragma unroll
    for (int c = 0; c < WTile<NP>::ROWS; c++) u[c] = w[c] * z[c];
    return true;
}

template <int NP>
struct Ros4Wave {
    static constexpr int RPL = WaveShape<NP>::RPL;
    __device__ static __forceinline__ bool step(const DevMech &M, const Lds &L, const double (&y)[RPL], double P, double h,
                                                double (&ynew)[RPL], double (&e)[RPL]) {
        wd4 X[WTile<NP>::TR][WTile<NP>::TR];
        double f[RPL], iw[RPL], w[RPL];
        jac_tiles<NP>(M, L, y, P, 1.0 / (Ros4::gamma * h), X, f, iw, w);
        const WScratch s = wt_scratch<NP>(L.JC);
        int ord[RPL];
        const bool ok = wt_invert<NP, double>(X, s, lane_fresh(), ord, M.N);
        constexpr int PJ = WTile<NP>::PJ;
        if constexpr (PJ > 0) {
            // the solves' vectors move to the Jacobian's per-species sums, the tiles to the staging area
            static_assert(WTile<NP>::kPark <= WaveShape<NP>::kJc && 2 * 64 * RPL <= 3 * NP);
            __syncthreads();
            wt_park<NP>(X, L.JC, lane_fresh());
            WScratch sv = s;
            sv.BS = L.TB;
            sv.XS = L.TB + 64 * RPL;
            ros4_stages<RPL>(M, L, y, P, h, f,
                             [&](const double (&b)[RPL], double (&u)[RPL]) {
                                 return tile_solve<NP, PJ>(X, sv, ord, iw, w, b, u, L.JC);
                             },
                             ynew, e);
        } else {
            ros4_stages<RPL>(M, L, y, P, h, f,
                             [&](const double (&b)[RPL], double (&u)[RPL]) {
                                 return tile_solve<NP>(X, s, ord, iw, w, b, u);
                             },
                             ynew, e);
        }
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
    __device__ static __forceinline__ bool step(const DevMech &M, const Lds &L, const double (&yy)[1], double P,
                                                double h, double (&ynew)[1], double (&e)[1], const IntOpts &o) {
        const double y = yy[0];
        constexpr double eps = 2.220446049250313e-16;
        constexpr int TR = WTile<NP>::TR;
        const int N = M.N;
        const int lane = lane_fresh();
        const bool comp = lane < N;
        double f0[1];
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
        int ord[1];
        const bool ok = wt_invert<NP, double>(X, s, lane_fresh(), ord, M.N);
        const double one[1] = {1.0};
        ros4_stages<1>(M, L, yy, P, h, f0,
                       [&](const double (&b)[1], double (&u)[1]) { return tile_solve<NP>(X, s, ord, one, one, b, u); },
                       ynew, e);
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
    __device__ static __forceinline__ bool step32(const DevMech &M, const Lds &L, const double (&y)[1], double P, double h,
                                                  double (&ynew)[1], double (&e)[1], int sweeps, bool &conv) {
        constexpr int TR = WTile<NP>::TR;
        wd4 X[TR][TR];
        wf4 F[TR][TR];
        double f[1], iw[1], w[1];
        jac_tiles<NP>(M, L, y, P, 1.0 / (Ros4::gamma * h), X, f, iw, w);
#pragma unroll
        for (int J = 0; J < TR; J++)
#pragma unroll
            for (int I = 0; I < TR; I++)
#pragma unroll
                for (int v = 0; v < 4; v++) F[J][I][v] = float(X[J][I][v]);
        const WScratch s = wt_scratch<NP>(L.JC);
        const int lane = lane_fresh();
        int ord[1];
        const bool ok = wt_invert<NP, float>(F, s, lane, ord, M.N);
        conv = true;
        auto inverse = [&](double b) {
            const float bf[1] = {float(b)};
            float xf[1];
            wt_solve<NP, float>(F, s, lane, ord, bf, xf);
            return double(xf[0]);
        };
        auto solve = [&](const double (&bb)[1], double (&u)[1]) -> bool {
            const double b = iw[0] * bb[0];
            double x[1] = {inverse(b)};
            if (sweeps > 0) {
                conv = false;
                double dprev = INFINITY;
                for (int k = 0; k < sweeps; k++) {
                    double mx[1];
                    wt_times<NP>(X, s, lane, x, mx);                // every lane takes part
                    const double d = inverse(lane < NP ? b - mx[0] : 0.0);
                    x[0] += d;
                    const double dmax = wmax_abs(w[0] * d), xmax = wmax_abs(w[0] * x[0]);
                    if (dmax <= 0x1p-48 * xmax) {
                        conv = true;
                        break;
                    }
                    if (!(dmax <= 0.5 * dprev)) break;      // stagnation (or not finite)
                    dprev = dmax;
                }
            }
            u[0] = w[0] * x[0];
            return conv;
        };
        ros4_stages<1>(M, L, y, P, h, f, solve, ynew, e);
        return ok;
    }
    __device__ static __forceinline__ bool step(const DevMech &M, const Lds &L, const double (&y)[1], double P, double h,
                                                double (&ynew)[1], double (&e)[1], int sweeps, int &fb) {
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
    static constexpr int RPL = WaveShape<NP>::RPL;
    static constexpr int NSMAX = NP - 1;
    static constexpr LdsKind LDS = kLdsJac;
    static constexpr int LDJ = WaveShape<NP>::LDJ;
    static constexpr int kJc = WaveShape<NP>::kJc;
    static constexpr bool PARK = WaveShape<NP>::PARK;
    static constexpr int PARK_ROWS = NP;
    // resident wavefronts per SIMD: two share its registers up to 64 rows; the 392 tile registers of 112
    // rows leave room for one
    static constexpr int WPE = NP > 64 ? 1 : 2;
    static constexpr double qinv = 0.25;
    __device__ static __forceinline__ bool step(const DevMech &M, const Lds &L, const double (&y)[RPL], double P, double h,
                                double (&yn)[RPL], double (&e)[RPL], const IntOpts &, int &) {
        return Ros4Wave<NP>::step(M, L, y, P, h, yn, e);
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
    static constexpr int WPE = 2;
    static constexpr double qinv = 0.25;
    __device__ static __forceinline__ bool step(const DevMech &M, const Lds &L, const double (&y)[1], double P,
                                                double h, double (&yn)[1], double (&e)[1], const IntOpts &o, int &) {
        return Ros4WaveFD<NP>::step(M, L, y, P, h, yn, e, o);
    }
};

template <int NP>
struct Ros4Adapter32 : Ros4Adapter<NP> {
    __device__ static __forceinline__ bool step(const DevMech &M, const Lds &L, const double (&y)[1], double P, double h,
                                double (&yn)[1], double (&e)[1], const IntOpts &o, int &fb) {
        return Ros4Wave32<NP>::step(M, L, y, P, h, yn, e, o.refine_sweeps, fb);
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
    static constexpr int WPE = 2;
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

template <class S>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(S::WPE, S::WPE))) integrate_wave_kernel(DevMech M, int64_t n, double *y, int64_t ld,
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
    init_lds<S::RPL>(M, L, S::LDS, S::NSMAX);
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

// Resident wavefronts per CU of the N <= 64 kernels are capped so that park slices fit the workspace.
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
    if (per > 4 * S::WPE) per = 4 * S::WPE;      // park slices in the workspace: kWaveMaxPerCu at two per SIMD
    int64_t grid = int64_t(cus) * per;
    if (grid > n) grid = n;
    double *park = S::PARK ? reinterpret_cast<double *>(reinterpret_cast<char *>(queue) + 256) : nullptr;
    zero_u32_kernel<<<1, 1, 0, s>>>(queue);
    integrate_wave_kernel<S><<<dim3(unsigned(grid)), dim3(64), lds, s>>>(M, n, y, ld, p, t_end, t, h, o, queue,
                                                                          park, status, nacc, nrej);
    return hipGetLastError() == hipSuccess ? CK_OK : CK_EHIP;
}
}  // namespace
}  // namespace ck
