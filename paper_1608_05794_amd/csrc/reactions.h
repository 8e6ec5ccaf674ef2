// Reaction pass of the deep-vectorised kernels: the threads of one reactor's wavefront (or
// workgroup) take one reaction each, read the species arrays of the reactor from LDS and add
// their contributions to per-species accumulators in LDS (Eqs. wdot, kfor, krev, kc and their
// derivatives).  Shared by the wavefront and the workgroup kernels.
#pragma once

#include "kinetics.h"

namespace ck {

// Species arrays and accumulators of one reactor (LDS).  C, G and H hold nsp + 1 entries: the
// extra one is a null species (C = 1, G = H = 0) that fills the unused slots of pair-form
// reactions; the accumulators have an entry for it too, which nothing reads.
struct RxArrays {
    double *C;      // concentrations
    double *G;      // g_k = H_k/(RT) - S_k/R - ln(p0/(RT)): sums of nu_k g_k are -ln Kc
    double *H;      // H_k/(RT) - 1
    double *WD;     // production rates
    // Jacobian only.  JC: d wdot_k / dC_j at fixed T (mass action and third-body efficiencies),
    // nsp + 1 rows of a column window.  TB and DWT hold what the chain rule through C(T, Y) needs
    // per species, with the weights of RxScale: with r_i = q_i - sum_j C_j dq_i/dC_j (the part of
    // the rate that is not first order in the concentrations),
    //   TB_k  = sum_i nu_ki (R_i dc_i/d[M] + sB r_i),   DWT_k = sum_i nu_ki (dq_i/dT + sT r_i).
    // HC_j = sum_k h_k JC[k][j] (h: enthalpies or internal energies over RT) comes reaction by
    // reaction as dq_i/dC_j sum_k nu_ki h_k, so no column of JC is read for it.
    double *JC, *TB, *DWT, *HC;
    int ldj;
};

// Weights of the chain rule: constant pressure sT = 1/T, sB = Wbar/rho, dh = 1 (h = H + 1);
// constant volume (C does not depend on T and the density is fixed) 0, 0, 0.
struct RxScale {
    double sT, sB, dh;
};

__device__ __forceinline__ double lds_at(const double *p, int byte_off) {
    return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(p) + byte_off);
}
__device__ __forceinline__ void lds_add(double *p, int byte_off, double v) {
    atomicAdd(reinterpret_cast<double *>(reinterpret_cast<char *>(p) + byte_off), v);
}

// What a pass evaluates.  kRates: rate constants, production rates and every accumulator, plus
// the JC columns of the window; kRatesKeep: the same, and the scalars that a later column window
// needs go to `keep` (entry (3 b + v) * T of the thread's b-th reaction); kScatterKept: JC columns
// of the window from those scalars; kScatter: JC columns of the window, rate constants evaluated
// again.
enum RxMode { kRates = 0, kRatesKeep = 1, kScatterKept = 2, kScatter = 3 };

// Blocks of T reactions in a pass (rows of kept scalars: three per block).
__host__ __device__ inline int rx_blocks(const DevMech &M, int T) {
    return (M.n_gen + T - 1) / T + (M.nrxn - M.n_gen + T - 1) / T;
}

// One pair-form reaction in registers.
struct PairRec {
    double lnA, beta, EaR;
    int4 off;
};
__device__ __forceinline__ PairRec pair_rec(const DevMech &M, int i) {
    const PairBlock &b = M.pair[i >> 6];
    const int l = i & 63;
    return PairRec{b.lnA[l], b.beta[l], b.EaR[l], b.off[l]};
}
// The first reaction of thread tid: requested ahead of the species pass, whose result it waits for.
template <int T>
__device__ __forceinline__ PairRec first_pair(const DevMech &M, int tid) {
    if (T != 64) return PairRec{};
    return pair_rec(M, min(tid, max(M.nrxn - M.n_gen - 1, 0)));
}

// Third-body efficiencies of pair-form reaction i < n_fall: the first three in registers.
struct Effs {
    int4 e;             // species offsets; type | number << 2
    double am1[3];
    int begin;
};
__device__ __forceinline__ Effs pair_effs(const DevMech &M, int i) {
    const FactorBlock &fb = M.factor[i >> 6];
    const int l = i & 63;
    return Effs{fb.eff[l], {fb.am1[0][l], fb.am1[1][l], fb.am1[2][l]}, fb.eff_begin[l]};
}
// f(byte offset of the species, alpha - 1) for each of them.
template <class F>
__device__ __forceinline__ void for_efficiencies(const DevMech &M, const Effs &x, F &&f) {
    const int n = x.e.w >> 2;
    if (n > 0) f(x.e.x, x.am1[0]);
    if (n > 1) f(x.e.y, x.am1[1]);
    if (n > 2) f(x.e.z, x.am1[2]);
    for (int j = 3; j < n; j++) f(8 * M.eff[x.begin + j].sp, M.eff[x.begin + j].am1);
}

// d wdot/dC of one pair-form reaction for the columns [c0, c0 + win): the four slots' columns, then
// those of the third-body efficiencies.  Rows of the null species go to a row that is never read.
__device__ __forceinline__ void pair_columns(const DevMech &M, const RxArrays &A, const int4 &o, double cA, double cB,
                                             double cC, double cD, double ckf, double ckr, double rdm, const Effs &ef,
                                             int c0, int win) {
    const int rA = o.x * A.ldj, rB = o.y * A.ldj, rC = o.z * A.ldj, rD = o.w * A.ldj;
    auto column = [&](int off, double dq) {
        const int col = off - 8 * c0;
        if (unsigned(col) < unsigned(8 * win)) {
            lds_add(A.JC, rA + col, -dq);
            lds_add(A.JC, rB + col, -dq);
            lds_add(A.JC, rC + col, dq);
            lds_add(A.JC, rD + col, dq);
        }
    };
    column(o.x, ckf * cB);
    column(o.y, ckf * cA);
    column(o.z, -ckr * cD);
    column(o.w, -ckr * cC);
    if (rdm != 0.0) for_efficiencies(M, ef, [&](int off, double am1) { column(off, rdm * am1); });
}

// A later column window from the first window's scalars.  The pass is a chain of loads and LDS adds, so
// the next block's offsets and scalars are requested while this one is scattered (windows 2..4 of M111:
// 90 -> 74 k cycles a step; M53, one window more: 16.3 -> 15.2 k).
template <int T>
__device__ __forceinline__ void pair_scatter(const DevMech &M, const RxArrays &A, int c0, int win, const double *keep,
                                             int tid) {
    const int nf = M.nrxn - M.n_gen;
    if (tid >= nf) return;
    struct Kept {
        int4 off;
        double ckf, ckr, rdm;
        Effs ef;
    };
    auto load = [&](int i, Kept &k) {
        k.off = M.pair[i >> 6].off[i & 63];
        k.ckf = keep[0];
        k.ckr = keep[T];
        k.rdm = 0.0;
        if (i < M.n_fall) {
            k.rdm = keep[2 * T];
            k.ef = pair_effs(M, i);
        }
        keep += 3 * T;
    };
    Kept next;
    load(tid, next);
    for (int i = tid; i < nf; i += T) {
        const Kept k = next;
        if (i + T < nf) load(i + T, next);
        const int4 o = k.off;
        pair_columns(M, A, o, lds_at(A.C, o.x), lds_at(A.C, o.y), lds_at(A.C, o.z), lds_at(A.C, o.w), k.ckf, k.ckr, k.rdm,
                     k.ef, c0, win);
    }
}

// Pair-form reactions (at most two reactant and two product units, 2 A counting as A + A, and
// reversible): straight-line code with four slots of coefficient one, no stoichiometric powers and
// no sign selects.  Slots 1 and 3 may be the null species.
template <int T, bool JAC>
__device__ __forceinline__ void pair_reactions(const DevMech &M, const RxArrays &A, const TPow &t, double Ctot,
                                               const RxScale &sc, int c0, int win, RxMode mode, double *keep,
                                               int tid, PairRec next) {
    const int nf = M.nrxn - M.n_gen;
    const int null_off = 8 * M.nsp;
    for (int i = tid; i < nf; i += T) {
        // One wavefront per reactor: the next block's records are requested while this one is evaluated
        // (M53: RHS stage 10.7 -> 9.5 k cycles).  The workgroup kernels have four wavefronts to cover the
        // load and no registers for it (M111 ROS4: 406 ms without, 431 ms with).
        const PairRec R = T == 64 ? next : pair_rec(M, i);
        if (T == 64 && i + T < nf) next = pair_rec(M, i + T);
        const int4 o = R.off;
        const double cA = lds_at(A.C, o.x), cB = lds_at(A.C, o.y), cC = lds_at(A.C, o.z), cD = lds_at(A.C, o.w);
        const bool has1 = o.y != null_off, has3 = o.w != null_off;
        const bool factor = i < M.n_fall;        // third-body or fall-off (the leading reactions)
        Effs ef;
        if (factor) ef = pair_effs(M, i);
        const double lnkf = fma(-R.EaR, t.invT, fma(R.beta, t.lnT, R.lnA));
        const double sg = (lds_at(A.G, o.z) + lds_at(A.G, o.w)) - (lds_at(A.G, o.x) + lds_at(A.G, o.y));
        double ckf = ck_exp(lnkf);
        double ckr = ck_exp(lnkf + sg);             // kr = kf / Kc, ln Kc = -sum_k nu_k g_k
        const double pf = cA * cB, pr = cC * cD;
        double dlnkf = 0.0, rdm = 0.0, rdT = 0.0, rdMc = 0.0;
        if (JAC) dlnkf = fma(R.EaR, t.invT, R.beta) * t.invT;
        if (factor) {
            const FactorBlock &fb = M.factor[i >> 6];
            const int l = i & 63;
            const FactorIn in{ef.e.w & 3,  fb.lnA0[l],  fb.beta0[l], fb.Ea0R[l],
                              fb.a[l],     fb.invT3[l], fb.invT1[l], fb.T2[l]};
            double Mc = Ctot;
            Mc = fma(ef.am1[0], lds_at(A.C, ef.e.x), Mc);
            Mc = fma(ef.am1[1], lds_at(A.C, ef.e.y), Mc);
            Mc = fma(ef.am1[2], lds_at(A.C, ef.e.z), Mc);
            for (int j = 3; j < ef.e.w >> 2; j++) {
                const EffRec E = M.eff[ef.begin + j];
                Mc = fma(E.am1, A.C[E.sp], Mc);
            }
            Factor c;
            rate_factor<JAC>(in, t, Mc, lnkf, dlnkf, c);
            const double Rn = ckf * pf - ckr * pr;
            ckf *= c.c;
            ckr *= c.c;
            if (JAC) {
                rdm = Rn * c.dcdM;
                rdT = Rn * c.dcdT;
                rdMc = rdm * c.Mc;
            }
        }
        const double qf = ckf * pf, qr = ckr * pr, q = qf - qr;
        if (!JAC || mode != kScatter) {
            double vT = 0.0, vB = 0.0, shx = 0.0;
            if (JAC) {
                const double sh = (lds_at(A.H, o.z) + lds_at(A.H, o.w)) - (lds_at(A.H, o.x) + lds_at(A.H, o.y));
                const double d1 = has1 ? 1.0 : 0.0, d3 = has3 ? 1.0 : 0.0;
                const double r = fma(d3, qr, -fma(d1, qf, rdMc));
                vT = fma(sc.sT, r, fma(q, dlnkf, fma(qr * sh, t.invT, rdT)));
                vB = fma(sc.sB, r, rdm);
                shx = fma(sc.dh, d3 - d1, sh);
            }
            lds_add(A.WD, o.x, -q);
            lds_add(A.WD, o.z, q);
            if (JAC) {
                lds_add(A.DWT, o.x, -vT);
                lds_add(A.DWT, o.z, vT);
                lds_add(A.TB, o.x, -vB);
                lds_add(A.TB, o.z, vB);
                lds_add(A.HC, o.x, ckf * cB * shx);
                lds_add(A.HC, o.z, -ckr * cD * shx);
            }
            if (has1) {
                lds_add(A.WD, o.y, -q);
                if (JAC) {
                    lds_add(A.DWT, o.y, -vT);
                    lds_add(A.TB, o.y, -vB);
                    lds_add(A.HC, o.y, ckf * cA * shx);
                }
            }
            if (has3) {
                lds_add(A.WD, o.w, q);
                if (JAC) {
                    lds_add(A.DWT, o.w, vT);
                    lds_add(A.TB, o.w, vB);
                    lds_add(A.HC, o.w, -ckr * cC * shx);
                }
            }
            if (JAC && factor && rdm != 0.0)
                for_efficiencies(M, ef, [&](int off, double am1) { lds_add(A.HC, off, rdm * am1 * shx); });
        }
        if (JAC && mode == kRatesKeep) {
            keep[0] = ckf;
            keep[T] = ckr;
            if (factor) keep[2 * T] = rdm;
            keep += 3 * T;
        }
        if (JAC) pair_columns(M, A, o, cA, cB, cC, cD, ckf, ckr, rdm, ef, c0, win);
    }
}

// Reactions of any form: up to three species per side with coefficients 1..3, irreversible ones.
// BOUND: slots that no reaction of the wavefront's block uses are skipped by scalar branches, which
// takes 22 registers off a Jacobian pass and lets another wavefront reside (N = 32, 155 reactions, a
// third of them general, 30000 Jacobians: 351 us with, 426 us without).  The source term is better off
// without the branches (N = 32 as above: 98 us with, 93 us without).
// POWERS: derivatives by dprod_powers, for kernels with the registers for it (Jacobian of N = 64, 315 general
// reactions, one reactor: 52 -> 43 us; the ROS4 kernels of pair-form mechanisms would lose 1 to 2 %).
template <int T, bool JAC, bool BOUND, bool POWERS>
__device__ __forceinline__ void general_reactions(const DevMech &M, const RxArrays &A, const TPow &t, double Ctot,
                                                  const RxScale &sc, int c0, int win, RxMode mode, double *keep,
                                                  int tid) {
    auto Cg = [&](int k) { return A.C[k]; };
    auto Gg = [&](int k) { return A.G[k]; };
    auto Hg = [&](int k) { return A.H[k]; };
    for (int i = tid; i < M.n_gen; i += T) {
        const RxnRec R = M.rx[i];
        const int nmax = BOUND ? __builtin_amdgcn_readfirstlane(R.blk_slots) : kMaxSlots;
        Slots S;
        load_slots(R, Cg, S, nmax);
        SlotPowers w;
        if (JAC && POWERS) slot_powers(S, nmax, w);
        auto dprod = [&](int s) { return POWERS ? dprod_powers(S, w, s, nmax) : dprod_slot(S, s, nmax); };
        double ckf, ckr, rdm;
        if (JAC && mode == kScatterKept) {
            ckf = keep[0];
            ckr = keep[T];
            rdm = keep[2 * T];
        } else {
            Rate q;
            reaction_rate<JAC>(M, R, S, nmax, t, Ctot, Cg, Gg, Hg, q);
            const double Rn = q.kf * q.pf - q.kr * q.pr;
            ckf = q.c * q.kf;
            ckr = q.c * q.kr;
            rdm = JAC ? Rn * q.dcdM : 0.0;
            if (!JAC || mode != kScatter) {
                const double qi = q.c * Rn;
                double vT = 0.0, vB = 0.0, shx = 0.0;
                if (JAC) {
                    double of = 0.0, orr = 0.0;
#pragma unroll
                    for (int s = 0; s < kMaxSlots; s++) {
                        if (s >= nmax) break;
                        of += S.sgn[s] < 0 ? double(S.nu[s]) : 0.0;
                        orr += S.sgn[s] > 0 ? double(S.nu[s]) : 0.0;
                        shx += S.sgn[s] != 0 ? (S.sgn[s] * S.nu[s]) * (Hg(S.sp[s]) + sc.dh) : 0.0;
                    }
                    const double qf = ckf * q.pf, qr = ckr * q.pr;
                    const double r = (1.0 - of) * qf - (1.0 - orr) * qr - rdm * q.Mc;
                    vT = q.c * (q.kf * q.dlnkf * q.pf - q.kr * q.dlnkr * q.pr) + Rn * q.dcdT + sc.sT * r;
                    vB = rdm + sc.sB * r;
                }
#pragma unroll
                for (int s = 0; s < kMaxSlots; s++) {
                    if (s >= nmax) break;
                    if (S.sgn[s] == 0) continue;
                    const double v = S.sgn[s] * S.nu[s];
                    atomicAdd(&A.WD[S.sp[s]], v * qi);
                    if (JAC) {
                        atomicAdd(&A.DWT[S.sp[s]], v * vT);
                        atomicAdd(&A.TB[S.sp[s]], v * vB);
                        const double d = dprod(s);
                        atomicAdd(&A.HC[S.sp[s]], (S.sgn[s] < 0 ? ckf * d : -ckr * d) * shx);
                    }
                }
                if (JAC && rdm != 0.0) {
                    const int eb = R.eff_begin, ec = rx_neff(R.meta);
                    for (int e = 0; e < ec; e++) atomicAdd(&A.HC[M.eff[eb + e].sp], rdm * M.eff[eb + e].am1 * shx);
                }
            }
            if (JAC && mode == kRatesKeep) {
                keep[0] = ckf;
                keep[T] = ckr;
                keep[2 * T] = rdm;
            }
        }
        if (JAC) {
            auto column = [&](int sp, double dq) {
                const int col = sp - c0;
                if (unsigned(col) >= unsigned(win)) return;
#pragma unroll
                for (int a = 0; a < kMaxSlots; a++) {
                    if (a >= nmax) break;
                    if (S.sgn[a] != 0) atomicAdd(&A.JC[S.sp[a] * A.ldj + col], (S.sgn[a] * S.nu[a]) * dq);
                }
            };
#pragma unroll
            for (int b = 0; b < kMaxSlots; b++) {
                if (b >= nmax) break;
                if (S.sgn[b] == 0) continue;
                const double d = dprod(b);
                column(S.sp[b], S.sgn[b] < 0 ? ckf * d : -ckr * d);
            }
            if (rdm != 0.0) {
                const int eb = R.eff_begin, ec = rx_neff(R.meta);
                for (int e = 0; e < ec; e++) column(M.eff[eb + e].sp, rdm * M.eff[eb + e].am1);
            }
            if (mode == kRatesKeep || mode == kScatterKept) keep += 3 * T;
        }
    }
}

// Every reaction of the mechanism.  Window: columns [c0, c0 + win) of JC, win already cut to the
// species count.  first: first_pair(M, tid).  The caller synchronises before and after.  GEN = false
// leaves the general form out (the caller knows that the mechanism has none); BOUND, POWERS:
// general_reactions.
template <int T, bool JAC, bool GEN = true, bool BOUND = (T > 64), bool POWERS = false>
__device__ __forceinline__ void reaction_pass(const DevMech &M, const RxArrays &A, const TPow &t, double Ctot,
                                              const RxScale &sc, int c0, int win, RxMode mode, double *keep,
                                              int tid, const PairRec &first) {
    if (GEN && M.n_gen > 0) {
        general_reactions<T, JAC, BOUND, POWERS>(M, A, t, Ctot, sc, c0, win, mode, keep, tid);
        if (JAC && (mode == kRatesKeep || mode == kScatterKept)) keep += 3 * T * ((M.n_gen + T - 1) / T);
    }
    if (JAC && mode == kScatterKept) pair_scatter<T>(M, A, c0, win, keep, tid);
    else pair_reactions<T, JAC>(M, A, t, Ctot, sc, c0, win, mode, keep, tid, first);
}

// Chain rule from the accumulators to J = df/dy for the lane's species k, shared by the kernels.
// The matrix is formed for the specific mole numbers z_k = Y_k / W_k instead of the mass fractions
// (a similarity transform with diag(1, W)): J'[k][j] = JC[k][j] + beta, so that no entry has to be
// scaled by its row's and column's molar mass; rows and columns of J follow with factors W_k and
// 1/W_j.  With sums over the reactor's species (callers reduce them):
//   sHB = sum H TB, sHW = sum H wdot, dQT = sum [R cp wdot + H (DWT - wdot / T)]   (H: J/mol)
// at constant pressure, and U = H - RT, c_v, no wdot/T term at constant volume.
struct ChainIn {
    double rho, Wbar, invT, RT, R, cpm, fT, sHB, sHW, dQT, sdcp;
};
__device__ __forceinline__ double chain_trow(const ChainIn &c, bool cv, double HC, double cp) {
    // dQ / dz_j - (dT/dt) d(rho c)/dz_j over rho c (per mole: times W_j against Y_j)
    if (!cv) {
        const double D = c.rho * c.cpm;
        const double dQ = c.rho * (c.RT * HC + c.sHB) - c.Wbar * c.sHW;
        const double dD = c.rho * (c.R * cp - c.cpm * c.Wbar);
        return -(dQ + c.fT * dD) / D;
    }
    const double D = c.rho * (c.cpm - c.R / c.Wbar);
    const double dQ = c.rho * (c.RT * HC + c.sHB);
    const double dD = c.rho * c.R * (cp - 1.0);
    return -(dQ + c.fT * dD) / D;
}
__device__ __forceinline__ double chain_J00(const ChainIn &c, bool cv) {
    const double D = c.rho * (cv ? c.cpm - c.R / c.Wbar : c.cpm);
    const double dD = c.rho * (cv ? c.sdcp : c.sdcp - c.cpm * c.invT);
    return -(c.dQT + c.fT * dD) / D;
}

}  // namespace ck
