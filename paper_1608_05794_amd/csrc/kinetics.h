// Device-side kinetics: NASA-7 thermodynamics (Eq. tfits, standard form),
// modified Arrhenius rates (Eq. kfor), equilibrium constants and reverse
// rates (Eqs. krev, kc), third-body and fall-off factors, and their
// temperature / concentration derivatives.  Shared by the lane-per-reactor
// and the wavefront-per-reactor kernels; species data are read through small
// accessor objects so each kernel keeps its own memory layout.
#pragma once

#include "ck_internal.h"

namespace ck {

// exp(x) = 2^n (1 + r + r^2 P(r)), n = round(x / ln 2), |r| <= ln 2 / 2: P is the degree-9 Chebyshev
// interpolant of (e^r - 1 - r) / r^2 (relative error 1.6e-17, below the rounding of the last step).
// 17 operations and no branch (measured over the range: 2.2e-16 relative); 0 and inf beyond the exponent
// range as long as |x| < 1e15, where the conversion to int saturates (the loader bounds the activation
// temperatures, exponents and Troe temperatures so that no rate leaves that range between 1 K and 1e11 K).
// NaN for an infinite x.
__device__ __forceinline__ double ck_exp(double x) {
    const double n = __builtin_rint(x * 1.4426950408889634);
    double r = fma(n, -0.6931471805598903, x);
    r = fma(n, -5.497923018708371e-14, r);
    double p = 2.5100397137931663e-08;
    p = fma(p, r, 2.762010358488696e-07);
    p = fma(p, r, 2.755726843551756e-06);
    p = fma(p, r, 2.4801521264122017e-05);
    p = fma(p, r, 0.00019841269863069374);
    p = fma(p, r, 0.0013888888917234206);
    p = fma(p, r, 0.008333333333330058);
    p = fma(p, r, 0.04166666666662409);
    p = fma(p, r, 0.16666666666666669);
    p = fma(p, r, 0.5000000000000001);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return __builtin_amdgcn_ldexp(p, int(n));
}

// 1 / x: hardware estimate and two Newton-Raphson steps (within an ulp for normal x; NaN for 0 and infinite x,
// where the kernels would go on to an infinite or undefined rate anyhow: T, rho, the mean molar mass).
__device__ __forceinline__ double ck_rcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

// ln x for finite x > 0, NaN otherwise: x = 2^e m with m in [sqrt(1/2), sqrt(2)), f = m - 1, s = f / (2 + f),
// ln m = 2 atanh(s) = f - s (f - z P(z)), z = s^2, P the degree-6 Chebyshev interpolant of
// (2 atanh(s) / s - 2) / z (relative error 5e-18 of the result).
__device__ __forceinline__ double ck_log(double x) {
    double m = __builtin_amdgcn_frexp_mant(x);
    int e = __builtin_amdgcn_frexp_exp(x);
    const bool low = m < 0.7071067811865476;
    m = low ? m + m : m;
    e = low ? e - 1 : e;
    const double f = m - 1.0, d = 2.0 + f;
    double s = f * ck_rcp(d);
    s = fma(fma(-d, s, f), ck_rcp(d), s);
    const double z = s * s;
    double p = 0.146171283998073;
    p = fma(p, z, 0.15331666676597175);
    p = fma(p, z, 0.1818289077802613);
    p = fma(p, z, 0.22222211112104948);
    p = fma(p, z, 0.2857142862611452);
    p = fma(p, z, 0.399999999998992);
    p = fma(p, z, 0.666666666666667);
    const double de = double(e);
    const double v = fma(de, 0.6931471805598903, f - fma(s, fma(-z, p, f), de * -5.497923018708371e-14));
    return x > 0.0 ? v : __builtin_nan("");
}

struct Thermo {
    double cp, h, g, dcp;   // cp/R, H/(RT), H/(RT) - S/R - ln(p0/(RT)), d(cp/R)/dT
};

// Powers of T and the multiples that the NASA-7 forms need.
struct TPow {
    double T, invT, lnT, T2, T3, T4;
};

__device__ __forceinline__ TPow tpow(double T) {
    TPow p;
    p.T = T;
    p.invT = ck_rcp(T);
    p.lnT = ck_log(T);
    p.T2 = T * T;
    p.T3 = p.T2 * T;
    p.T4 = p.T3 * T;
    return p;
}

// NASA-7 coefficients of species k: the low range (T < Tmid) or the high one (per-lane select).
struct Nasa {
    double a1, a2, a3, a4, a5, a6, a7;
};
__device__ __forceinline__ Nasa species_coef(const DevMech &M, int k, bool low) {
    const int ns = M.nsp;
    const double *c = M.thermo() + (low ? 0 : 7) * ns + k;
    return Nasa{c[0], c[ns], c[2 * ns], c[3 * ns], c[4 * ns], c[5 * ns], c[6 * ns]};
}

// The 1/k factors of the integrated polynomials go to the powers of T, which every species shares,
// so a species costs seven coefficient loads and 16 multiply-adds.  g is formed as one polynomial:
// a1 (1 - ln T) - a2 T/2 - a3 T^2/6 - a4 T^3/12 - a5 T^4/20 + a6/T - a7, plus ln T - ln(p0/R).
__device__ __forceinline__ Thermo species_thermo(const DevMech &M, const Nasa &a, const TPow &t) {
    const double h2 = t.T * (1.0 / 2.0), h3 = t.T2 * (1.0 / 3.0), h4 = t.T3 * (1.0 / 4.0), h5 = t.T4 * (1.0 / 5.0);
    const double g3 = t.T2 * (-1.0 / 6.0), g4 = t.T3 * (-1.0 / 12.0), g5 = t.T4 * (-1.0 / 20.0);
    Thermo o;
    o.cp = fma(a.a5, t.T4, fma(a.a4, t.T3, fma(a.a3, t.T2, fma(a.a2, t.T, a.a1))));
    o.h = fma(a.a6, t.invT, fma(a.a5, h5, fma(a.a4, h4, fma(a.a3, h3, fma(a.a2, h2, a.a1)))));
    o.g = fma(a.a6, t.invT, fma(a.a5, g5, fma(a.a4, g4, fma(a.a3, g3, fma(a.a2, -h2, a.a1 * (1.0 - t.lnT)))))) +
          ((t.lnT - M.ln_p0_R) - a.a7);
    o.dcp = fma(4.0 * a.a5, t.T3, fma(3.0 * a.a4, t.T2, fma(2.0 * a.a3, t.T, a.a2)));
    return o;
}
__device__ __forceinline__ Thermo species_thermo(const DevMech &M, int k, const TPow &t) {
    return species_thermo(M, species_coef(M, k, t.T < M.Tmid()[k]), t);
}

// x^n for n in 0..3
__device__ __forceinline__ double ipow(double x, int n) {
    const double x2 = x * x;
    return n == 0 ? 1.0 : (n == 1 ? x : (n == 2 ? x2 : x2 * x));
}

// The species slots of one reaction with their concentrations, in registers.
struct Slots {
    double c[kMaxSlots];
    int sp[kMaxSlots];
    int nu[kMaxSlots];     // 0 for unused slots
    int sgn[kMaxSlots];    // -1 reactant, +1 product, 0 unused
    int n, nre;
};

// nmax: a wave-uniform bound on the slot count (slots beyond it are skipped by scalar branches).
template <class Cget>
__device__ __forceinline__ void load_slots(const RxnRec &R, const Cget &C, Slots &S, int nmax) {
    S.n = rx_nslot(R.meta);
    S.nre = rx_nreac(R.meta);
#pragma unroll
    for (int s = 0; s < kMaxSlots; s++) {
        if (s >= nmax) {
            S.sp[s] = 0;
            S.nu[s] = 0;
            S.sgn[s] = 0;
            S.c[s] = 1.0;
            continue;
        }
        const bool used = s < S.n;
        S.sp[s] = rx_sp(R, s);
        S.nu[s] = used ? rx_nu(R, s) : 0;
        S.sgn[s] = used ? (s < S.nre ? -1 : 1) : 0;
        S.c[s] = C(used ? S.sp[s] : 0);
    }
}

// Third-body / fall-off factor c of a reaction, [M], and the derivatives of c.
struct Factor {
    double c, Mc, dcdM, dcdT;
};

// Parameters of a factor: type, low-pressure limit and Troe data.
struct FactorIn {
    int type;
    double lnA0, beta0, Ea0R, a, invT3, invT1, T2;
};

// Factor at [M] = Mc of a reaction whose (high-pressure) rate constant is exp(lnkf).
template <bool DERIV>
__device__ __forceinline__ void rate_factor(const FactorIn &F, const TPow &t, double Mc, double lnkf, double dlnkf,
                                            Factor &o) {
    const int ty = F.type;
    o.Mc = Mc;
    o.c = Mc;
    if (DERIV) {
        o.dcdM = 1.0;
        o.dcdT = 0.0;
    }
    if (ty == kThirdBody) return;
    // fall-off: Pr = k0 [M] / k_inf, c = Pr / (1 + Pr) F
    const double lnk0 = fma(-F.Ea0R, t.invT, fma(F.beta0, t.lnT, F.lnA0));
    const double ratio = ck_exp(lnk0 - lnkf);
    const double Pr = ratio * Mc;
    double Fb = 1.0, g = 0.0, dlogF_dL = 0.0, dFc_over_Fc = 0.0;
    if (ty == kTroe) {
        constexpr double kLog10e = 0.4342944819032518, kLn10 = 2.302585092994046;
        const double a = F.a;
        const double e3 = ck_exp(-t.T * F.invT3);
        const double e1 = ck_exp(-t.T * F.invT1);
        const double e2 = ck_exp(-F.T2 * t.invT);
        const double Fc = (1.0 - a) * e3 + a * e1 + e2;
        const double L = kLog10e * ck_log(fmax(Fc, 1e-300));
        const double cc = -0.4 - 0.67 * L;
        const double nn = 0.75 - 1.27 * L;
        const double x = fma(kLog10e, ck_log(fmax(Pr, 1e-300)), cc);
        const double d = nn - 0.14 * x;
        // d = 0: f1 beyond any bound and F = 1; any other d is unchanged (a select instead: Jacobian M53 x 8192
        // 142.3 us, 139.7 with the addition)
        const double id = ck_rcp(d + 0x1p-500);
        const double f1 = x * id;
        const double iu = ck_rcp(fma(f1, f1, 1.0));
        Fb = ck_exp(kLn10 * L * iu);
        if (DERIV) {
            const double iu2 = iu * iu;
            const double id2 = id * id;
            g = L * (-2.0 * f1 * iu2) * (nn * id2);
            dlogF_dL = iu - L * 2.0 * f1 * iu2 * ((-0.67 * nn + 1.27 * x) * id2);
            const double dFc = -(1.0 - a) * F.invT3 * e3 - a * F.invT1 * e1 + F.T2 * t.invT * t.invT * e2;
            dFc_over_Fc = dFc / Fc;
        }
    }
    const double ionep = 1.0 / (1.0 + Pr);
    o.c = Pr * ionep * Fb;
    if (DERIV) {
        const double dc_dPr = Fb * ionep * (ionep + g);
        const double dlnPr_dT = (F.beta0 + F.Ea0R * t.invT) * t.invT - dlnkf;
        o.dcdM = dc_dPr * ratio;
        o.dcdT = dc_dPr * Pr * dlnPr_dT;
        if (ty == kTroe) o.dcdT += o.c * dlogF_dL * dFc_over_Fc;
    }
}

// Everything one reaction contributes at (T, C).
struct Rate {
    double kf, kr;        // multiply the mass-action products; k_inf for fall-off
    double pf, pr;        // prod C^nu' and prod C^nu''
    double c, Mc;         // third-body / fall-off factor and its [M] (0 for elementary reactions)
    double dlnkf, dlnkr;  // d ln k / dT            (DERIV only)
    double dcdM, dcdT;    // d c / d[M], d c / dT   (DERIV only)
};

// Rate constants and factors of reaction R (Eqs. kfor, krev, kc; third-body and
// fall-off factor c).  Gget(k) returns H_k/(RT) - S_k/R - ln(p0/(RT)), Hget(k) H_k/(RT) - 1, so that
// ln Kc = -sum_j nu_j g_j and d ln Kc / dT = sum_j nu_j h_j / T without the net mole change.
template <bool DERIV, class Cget, class Gget, class Hget>
__device__ __forceinline__ void reaction_rate(const DevMech &M, const RxnRec &R, const Slots &S, int nmax,
                                              const TPow &t, double Ctot, const Cget &C, const Gget &G,
                                              const Hget &H, Rate &o) {
    const double lnkf = fma(-R.EaR, t.invT, fma(R.beta, t.lnT, R.lnA));
    o.kf = ck_exp(lnkf);
    if (DERIV) o.dlnkf = (R.beta + R.EaR * t.invT) * t.invT;
    o.pf = 1.0;
    o.pr = 1.0;
    double sg = 0.0, sh = 0.0;
#pragma unroll
    for (int s = 0; s < kMaxSlots; s++) {
        if (s >= nmax) break;
        const double p = ipow(S.c[s], S.nu[s]);
        if (S.sgn[s] < 0) o.pf *= p;
        else o.pr *= p;
        const int sp = S.sgn[s] != 0 ? S.sp[s] : 0;
        const double w = double(S.sgn[s] * S.nu[s]);
        sg += w * G(sp);
        if (DERIV) sh += w * H(sp);
    }
    const int meta = R.meta;
    if (rx_rev(meta)) {
        o.kr = ck_exp(lnkf + sg);      // kr = kf / Kc
        if (DERIV) o.dlnkr = o.dlnkf - sh * t.invT;
    } else {
        o.kr = 0.0;
        if (DERIV) o.dlnkr = 0.0;
    }
    o.c = 1.0;
    o.Mc = 0.0;
    if (DERIV) {
        o.dcdM = 0.0;
        o.dcdT = 0.0;
    }
    if (rx_type(meta) == kElementary) return;
    double Mc = Ctot;
    const int eb = R.eff_begin, ec = rx_neff(meta);
    for (int e = 0; e < ec; e++) {
        const EffRec E = M.eff[eb + e];
        Mc += E.am1 * C(E.sp);
    }
    FactorIn in{rx_type(meta), 0, 0, 0, 0, 0, 0, 0};
    if (in.type != kThirdBody) {
        const FallRec F = M.fall[R.fall];
        in = FactorIn{in.type, F.lnA0, F.beta0, F.Ea0R, F.a, F.invT3, F.invT1, F.T2};
    }
    Factor f;
    rate_factor<DERIV>(in, t, Mc, lnkf, o.dlnkf, f);
    o.c = f.c;
    o.Mc = f.Mc;
    if (DERIV) {
        o.dcdM = f.dcdM;
        o.dcdT = f.dcdT;
    }
}

// d(prod over the side of slot s)/dC of slot s: nu_s C_s^(nu_s-1) times the side's other factors.
__device__ __forceinline__ double dprod_slot(const Slots &S, int s, int nmax) {
    double p = 1.0;
#pragma unroll
    for (int t = 0; t < kMaxSlots; t++) {
        if (t >= nmax) break;
        if (S.sgn[t] != S.sgn[s]) continue;
        const double ct = S.c[t];
        if (t == s)
            p *= S.nu[t] == 1 ? 1.0 : (S.nu[t] == 2 ? 2.0 * ct : 3.0 * ct * ct);
        else
            p *= ipow(ct, S.nu[t]);
    }
    return p;
}

// The same from the powers of every slot, with a factor of 1 for the other side's slots where dprod_slot
// skips them: the lanes' reactions differ in all of it, and the selects take a third of the branches'
// instructions off a general reaction's Jacobian, for twelve more registers.
struct SlotPowers {
    double pw[kMaxSlots], dv[kMaxSlots];     // C^nu and nu C^(nu-1)
};
__device__ __forceinline__ void slot_powers(const Slots &S, int nmax, SlotPowers &o) {
#pragma unroll
    for (int t = 0; t < kMaxSlots; t++) {
        if (t >= nmax) break;
        const double ct = S.c[t];
        o.pw[t] = ipow(ct, S.nu[t]);
        o.dv[t] = S.nu[t] == 1 ? 1.0 : (S.nu[t] == 2 ? 2.0 * ct : 3.0 * ct * ct);
    }
}
__device__ __forceinline__ double dprod_powers(const Slots &S, const SlotPowers &w, int s, int nmax) {
    double p = 1.0;
#pragma unroll
    for (int t = 0; t < kMaxSlots; t++) {
        if (t >= nmax) break;
        p *= S.sgn[t] == S.sgn[s] ? (t == s ? w.dv[t] : w.pw[t]) : 1.0;
    }
    return p;
}

// ROS4 coefficients (Appendix C; gamma as tabulated).
struct Ros4 {
    static constexpr double gamma = 0.57282;
    static constexpr double a21 = 2.0;
    static constexpr double a31 = 1.867943637803922, a32 = 0.2344449711399156;
    static constexpr double c21 = -7.137615036412310;
    static constexpr double c31 = 2.580708087951457, c32 = 0.6515950076447975;
    static constexpr double c41 = -2.137148994382534, c42 = -0.3214669691237626, c43 = -0.6949742501781779;
    static constexpr double m1 = 2.255570073418735, m2 = 0.2870493262186792, m3 = 0.4353179431840180,
                            m4 = 1.093502252409163;
    static constexpr double e1 = -0.2815431932141155, e2 = -0.07276199124938920, e3 = -0.1082196201495311,
                            e4 = -1.093502252409163;
};

// Runge--Kutta--Fehlberg 4(5) (Appendix B).
struct Rkf45 {
    static constexpr double a21 = 1.0 / 4.0;
    static constexpr double a31 = 3.0 / 32.0, a32 = 9.0 / 32.0;
    static constexpr double a41 = 1932.0 / 2197.0, a42 = -7200.0 / 2197.0, a43 = 7296.0 / 2197.0;
    static constexpr double a51 = 439.0 / 216.0, a52 = -8.0, a53 = 3680.0 / 513.0, a54 = -845.0 / 4104.0;
    static constexpr double a61 = -8.0 / 27.0, a62 = 2.0, a63 = -3544.0 / 2565.0, a64 = 1859.0 / 4104.0,
                            a65 = -11.0 / 40.0;
    static constexpr double b1 = 25.0 / 216.0, b3 = 1408.0 / 2565.0, b4 = 2197.0 / 4104.0, b5 = -1.0 / 5.0;
    static constexpr double d1 = 16.0 / 135.0 - 25.0 / 216.0, d3 = 6656.0 / 12825.0 - 1408.0 / 2565.0,
                            d4 = 28561.0 / 56430.0 - 2197.0 / 4104.0, d5 = -9.0 / 50.0 + 1.0 / 5.0,
                            d6 = 2.0 / 55.0;
};

// Step-size control shared by every integrator kernel (the paper leaves
// EstimateH0 and AdjustStepSize unspecified; this is the library's fixed
// specification: safety 0.9, factor in [0.2, 5], error exponent 1/q).
__device__ __forceinline__ double step_factor(double err, double q_inv, bool accepted) {
    if (accepted) return err == 0.0 ? 5.0 : fmin(5.0, fmax(0.2, 0.9 * pow(err, -q_inv)));
    return isfinite(err) ? fmax(0.2, 0.9 * pow(err, -q_inv)) : 0.2;
}

__device__ __forceinline__ double h_floor(double t) { return fmax(1e-30, 16.0 * 2.220446049250313e-16 * fabs(t)); }

}  // namespace ck
