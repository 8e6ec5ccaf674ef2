// Wavefront-per-reactor kernels for N <= 64 (source term and RKF45: N <= 128); the device code is in
// wave.h.
#include "wave.h"

namespace ck {

// ---------------------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------------------
// Source term.  Bound by vector issue: 905 instructions a reactor at M53 (2291 before the pair form), 92 %
// of the issue slots busy with four wavefronts per SIMD, LDS 54 %: M53 x 131072 466 -> 247 us,
// M111 x 30011 205 -> 107 us.  One workgroup per reactor: workgroups that stride through the batch,
// with the next state requested ahead, were a tenth slower (254 against 230 us of the kernel alone); a
// line of memory per lane costs 2 % against contiguous states.
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

// Standalone Jacobian for N <= 64: workgroups of one or eight wavefronts, one reactor each, d wdot/dC
// staged in windows of WIN matrix columns (the temperature column is column 0).
//
// Eight: bound by the stores: an entry of a reactor is eight bytes of a line that it shares with fifteen
// neighbours, so the eight staged windows are written out together, eight neighbouring reactors by one
// store (64 bytes), instead of one reactor at a time (a line per lane): M53 x 8192 141 us, 233 us with one.  The
// windows of eight reactors fill a CU's LDS, so rates are evaluated again for a later window.
//
// One: the whole matrix in one window.  A call on few reactors is a latency: here every reactor has a
// SIMD to itself and its rates are evaluated once (M53 x 64 45 us with eight, 25 us with one; N = 64
// 56 and 26 us).  launch_jac_wave has the rule.
template <int NSMAX, int WIN, int RW>
struct JacShape {
    static constexpr int R = RW;                    // reactors of a workgroup
    static constexpr int LDJ = WIN | 1;
    static constexpr int NWIN = (NSMAX + 1 + WIN - 1) / WIN;
    static constexpr int kSlab0 = 8 * (NSMAX + 1) + (NSMAX + 1) * LDJ;
    // slab stride 8 modulo 32 doubles: the eight reactors of a store read different banks
    static constexpr int kSlab = R == 1 ? kSlab0 : kSlab0 + (8 - kSlab0 % 32 + 32) % 32;
    static constexpr size_t kLds = size_t(R) * kSlab + 2 * (NSMAX + 1);
    // general reactions: where more wavefronts than two a SIMD fit the LDS, registers limit them
    static constexpr bool BOUND = R == 1 && NSMAX < 36, POWERS = R == 1 && NSMAX > 16;
};
// WPE: resident wavefronts per SIMD that the registers have to allow
template <int NSMAX, int WIN, int RW, int WPE>
__global__ void __launch_bounds__(64 * RW) __attribute__((amdgpu_waves_per_eu(WPE, 4)))
jac_wave_kernel(DevMech M, int64_t n, const double *y, int64_t ld, const double *p, double *jac, int cv) {
    using SH = JacShape<NSMAX, WIN, RW>;
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
    for (int e = int(threadIdx.x); e < N; e += 64 * SH::R) {
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
    const RxScale sc = rx_scale<1>(L, x);
    reaction_pass<64, true, true, SH::BOUND, SH::POWERS>(M, L, x.t, x.Ctot, sc, -1, min(WIN, N), kRates, nullptr,
                                                         lane, first);
    __syncthreads();
    finish_rhs<1>(M, L, x, ff);
    const Chain<1> c = chain_rule<1>(M, L, x, yy, bcast(ff[0], 0));
    __syncthreads();
    // per-row scalars in place of the sums: W beta in TB, W col0 in DWT, by species; the temperature row
    if (L.sl[0].valid) {
        const int k = L.sl[0].k;
        L.TB[k] = L.sl[0].W * c.beta[0];
        L.DWT[k] = L.sl[0].W * c.col0[0];
        L.TROW[1 + k] = c.trow[0];
    }
    if (lane == 0) L.TROW[0] = c.J00;
    for (int w = 0; w < SH::NWIN; w++) {
        if (w > 0) {
            if (w * WIN >= N) break;
            zero_jc(L, ns);
            __syncthreads();
            const PairRec again = first_pair<64>(M, lane);
            reaction_pass<64, true, true, SH::BOUND, SH::POWERS>(M, L, x.t, x.Ctot, sc, w * WIN - 1,
                                                                 min(WIN, N - w * WIN), kScatter, nullptr, lane, again);
        }
        __syncthreads();
        if constexpr (SH::R == 1 && NSMAX >= 32) {
            // one window, a matrix column per lane: no divisions, and the rows' loads go out together, eight at
            // a time (M53 x 1 30 us with the loop below, 24 so)
            if (lane < N) {
                const bool t = lane == 0;      // the temperature column is staged whole: 1 x - 0
                const double iw = IW[lane];
                const double *a = t ? L.DWT : L.JC + lane;
                double *out = jac + int64_t(lane) * ld + r0;
                out[0] = iw * L.TROW[lane];
#pragma unroll 8
                for (int i = 1; i < N; i++)
                    out[int64_t(i) * N * ld] =
                        iw * fma(t ? 1.0 : W[i], a[(i - 1) * (t ? 1 : SH::LDJ)], t ? -0.0 : L.TB[i - 1]);
            }
            break;
        }
        const int s = int(threadIdx.x) % SH::R;
        const double *slab = lds_raw + s * SH::kSlab;
        const int cols = min(WIN, N - w * WIN);
        if (r0 + s < n)
            for (int e = int(threadIdx.x) / SH::R; e < N * WIN; e += 64) {
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

// ---------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------
namespace {
int pad_np(int N) { return ((N + 7) / 8) * 8; }
}  // namespace

namespace {
template <int NSMAX, int WIN, int RW, int WPE>
int launch_jac(const DevMech &M, int64_t n, const double *y, int64_t ld, const double *p, double *jac, int cv,
               hipStream_t s) {
    using SH = JacShape<NSMAX, WIN, RW>;
    if (M.nsp > NSMAX) return CK_EUNSUPPORTED;
    const size_t lds = SH::kLds * sizeof(double);
    auto kern = jac_wave_kernel<NSMAX, WIN, RW, WPE>;
    if (lds > 64 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)) != hipSuccess)
        return CK_EHIP;
    const int64_t groups = (n + SH::R - 1) / SH::R;
    kern<<<dim3(unsigned((groups + 7) / 8 * 8)), dim3(64 * RW), lds, s>>>(M, n, y, ld, p, jac, cv);
    return hipGetLastError() == hipSuccess ? CK_OK : CK_EHIP;
}
}  // namespace

bool wave_supported(const DevMech &M, int method, int precision) {
    if (method == 0) return M.N <= 64;
    return precision == CK_PREC_FP64 && M.N <= 128;
}

size_t wave_ws_bytes(const DevMech &M, int cus) {
    // a slice of NP rows of 64 doubles for every resident wavefront: the first Jacobian window's rate
    // scalars (analytic ROS4, NP > 32), or the matrix (forward differences)
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
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return CK_EHIP;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return CK_EHIP;
    // Workgroups of eight: one a CU at a time (LDS), so they take rounds of 8 CUs reactors, and an idle part
    // of the last round costs as much as a full one.  One reactor a workgroup takes a time in proportion to n,
    // is a SIMD's alone in a small batch and has the better occupancy at small N; its stores are narrow, which
    // costs most where ld is a multiple of 4 KiB and a reactor's entries share their channels.  So: one by one
    // where the rounds of eight are poorly filled (M53 x 1200 46 us, eight 49; x 2100 67, 84; x 8192 270, 157),
    // and general reactions, which keep eight reactors from overlapping, more often (N = 64, all 315 general:
    // x 2100 137 us, eight 207; x 16384, ld a multiple of 4 KiB, N = 54: 675 us, eight 460).
    const bool general = M.n_gen > 0;
    const int64_t round = 8 * int64_t(cus), rounds = (n + round - 1) / round;
    auto filled_to = [&](int eighths) { return n <= eighths * rounds * cus; };
    if (M.N <= 16) {
        // the general pass takes spills for a fourth wavefront once three do not hold the batch (N = 14,
        // all 65 reactions general: x 2048 41 us, 37 with three; x 30000 235 us, 256)
        if (general && n > 12 * int64_t(cus)) return launch_jac<15, 16, 1, 4>(M, n, y, ld, p, jac, cv, s);
        return launch_jac<15, 16, 1, 3>(M, n, y, ld, p, jac, cv, s);
    }
    if (M.N <= 32) {
        // N = 32, pair form: x 2048 33 us, eight 29; x 2100 36, 43; x 16384 133, 138.  N = 18 is better off one by
        // one at every n (x 30000 129 us, eight 190), N = 25 too (151, 213).
        if (M.N > 24 && !filled_to(7) && rounds <= (general ? 2 : 4))
            return launch_jac<31, 32, 8, 2>(M, n, y, ld, p, jac, cv, s);
        return launch_jac<31, 32, 1, 3>(M, n, y, ld, p, jac, cv, s);
    }
    // three wavefronts a SIMD (N = 34, all 165 reactions general: x 30000 381 us, eight 708)
    if (M.N <= 36) return launch_jac<35, 36, 1, 3>(M, n, y, ld, p, jac, cv, s);
    bool one;
    if (general)
        // N = 40: one by one always (x 8192 177 us, eight 253).  Full rounds of eight pay from N = 45 on (N = 54,
        // irreversible, x 8192 237 us, one by one 315) while they are few or ld is that multiple.
        one = M.N <= 40 || filled_to(M.N <= 48 || rounds > 1 ? 7 : 5) ||
              (rounds > 1 && (M.N <= 44 || (rounds >= 5 && ld % 512 != 0)));
    else
        one = filled_to(M.N <= 48 ? 6 : 5);
    // the fewer columns staged, the more workgroups a CU holds: ten, seven, five and four
    if (one && M.N <= 40) return launch_jac<39, 40, 1, 1>(M, n, y, ld, p, jac, cv, s);
    if (one && M.N <= 48) return launch_jac<47, 48, 1, 1>(M, n, y, ld, p, jac, cv, s);
    if (one && M.N <= 56) return launch_jac<55, 56, 1, 1>(M, n, y, ld, p, jac, cv, s);
    if (one) return launch_jac<63, 64, 1, 1>(M, n, y, ld, p, jac, cv, s);
    if (M.N <= 56) return launch_jac<55, 32, 8, 2>(M, n, y, ld, p, jac, cv, s);
    return launch_jac<63, 24, 8, 2>(M, n, y, ld, p, jac, cv, s);      // eight windows of 32 columns exceed the LDS
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
