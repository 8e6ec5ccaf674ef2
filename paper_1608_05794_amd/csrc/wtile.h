// Dense linear algebra of one wavefront (N <= 112): the iteration matrix in 16 x 16 register tiles and
// its inverse by blocked Gauss-Jordan elimination with partial pivoting, rank-16 updates on the FP64
// matrix cores; stage solves are matrix-vector products.
//
// Layout.  Lane l = 16 g + c.  Tile X[J][I] holds the TRANSPOSE of the matrix block (I, J) in the
// accumulator layout of the 16x16x4 instruction: register v of lane (g, c) is
//     A[16 I + c][16 J + g + 4 v]     (FP64 instruction: rows of the accumulator interleave over g).
// Transposed, an update A[:, J] += T U[:, J] is X[J][I] += U^T T^T, whose B operand (lane (g, c) holds
// T[16 I + c][4 s + g]) is register s of the eliminated panel's own tile, so the panel is not loaded a
// second time; the A operand is the panel's pivot rows, read from LDS.  A matrix-vector product is
// 16 TR multiply-adds per lane and row block and a sum over the four lane groups that leaves row
// 16 g + c on lane (g, c), i.e. one component per lane (rows from 64 on in a second register).
//
// Why this form (measured at N = 54, M53, 16384 reactors to 1e-13 s): the register LU with one row per
// lane spent about 6300 vector instructions on the factorisation (two lane reads and a hazard wait per
// multiply-add, in a serial chain per column) and 900 on each of the four substitutions, of 17.2 k a
// step.  Here a panel costs one pivot search and 15 broadcast columns per pivot, the other columns go
// to the matrix cores, and a solve is about 80 instructions.
#pragma once

#include <type_traits>

#include "kinetics.h"

namespace ck {

typedef double wd4 __attribute__((ext_vector_type(4)));
typedef float wf4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double wt_readlane(double v, int src) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), src);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), src);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ float wt_readlane(float v, int src) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src));
}

// Element types of the tiles.  The FP32 instruction keeps its accumulator rows contiguous (row 4 g + v
// on lane group g, register v) where the FP64 one interleaves them (g + 4 v); feeding its A operand
// the columns in the order ucol(c) gives both the same tile layout.
template <class T> struct WtType;
template <> struct WtType<double> {
    using V = wd4;
    __device__ static __forceinline__ V mfma(double a, double b, V c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    __device__ static __forceinline__ int ucol(int c) { return c; }
    __device__ static __forceinline__ unsigned key(double v) { return unsigned(__double2hiint(fabs(v))); }
    __device__ static __forceinline__ double rcp(double v) { return __builtin_amdgcn_rcp(v); }
};
template <> struct WtType<float> {
    using V = wf4;
    __device__ static __forceinline__ V mfma(float a, float b, V c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    __device__ static __forceinline__ int ucol(int c) { return (c >> 2) + 4 * (c & 3); }
    __device__ static __forceinline__ unsigned key(float v) { return __float_as_uint(fabsf(v)); }
    __device__ static __forceinline__ float rcp(float v) { return __builtin_amdgcn_rcpf(v); }
};

// f(integral_constant<i>) for i in [B, E).
template <int B, int E, class F>
__device__ __forceinline__ void wt_for(F &&f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        wt_for<B + 1, E>(static_cast<F &&>(f));
    }
}

// Search for the next pivot and its reciprocal, cut into short stages of one dependency chain.  The
// pivot is the row with the largest |a| (FP64: by the high word, which is ordered like |a|; values
// within a relative 2^-20 of the largest may tie, and then the first lane is taken); key is 0 for rows
// already used.  With two rows per lane (lane and lane + 64) sel tells which one it is.
// Stages 0..5: largest key (rows of 16 lanes, then each row's last lane into the next row and row 1's
// into the upper half); 6, 7: lane; 8, 9: 1 / pivot estimate; 10..13: two Newton-Raphson steps.
template <class E, int ROWS>
struct PivotSearch {
    unsigned key[ROWS], m;
    int src;
    bool any, sel;
    E piv, rp, t;
    __device__ __forceinline__ void start(const E (&R)[ROWS][16], const bool (&done)[ROWS]) {
#pragma unroll
        for (int r = 0; r < ROWS; r++) key[r] = done[r] ? 0u : WtType<E>::key(R[r][0]);
        m = ROWS == 2 ? max(key[0], key[ROWS - 1]) : key[0];
    }
    template <int CTRL, int LANES>
    __device__ __forceinline__ void fold() {
        m = max(m, unsigned(__builtin_amdgcn_update_dpp(0, int(m), CTRL, LANES, 0xf, true)));
    }
    template <int S>
    __device__ __forceinline__ void stage(const E (&R)[ROWS][16]) {
        if constexpr (S == 0) fold<0x111, 0xf>();      // row_shr 1
        if constexpr (S == 1) fold<0x112, 0xf>();      // row_shr 2
        if constexpr (S == 2) fold<0x114, 0xf>();      // row_shr 4
        if constexpr (S == 3) fold<0x118, 0xf>();      // row_shr 8
        if constexpr (S == 4) fold<0x142, 0xa>();      // row_bcast 15
        if constexpr (S == 5) fold<0x143, 0xc>();      // row_bcast 31
        if constexpr (S == 6) {
            m = unsigned(__builtin_amdgcn_readlane(int(m), 63));
            any = m != 0u;
        }
        if constexpr (S == 7) {
            if constexpr (ROWS == 1) {
                src = __builtin_ctzll(__builtin_amdgcn_ballot_w64(key[0] == m));
                sel = false;
            } else {
                const unsigned long long b0 = __builtin_amdgcn_ballot_w64(key[0] == m);
                sel = b0 == 0ull;
                src = __builtin_ctzll(sel ? __builtin_amdgcn_ballot_w64(key[ROWS - 1] == m) : b0);
            }
        }
        if constexpr (S == 8) {
            piv = wt_readlane(R[0][0], src);
            if constexpr (ROWS == 2) {
                const E p1 = wt_readlane(R[ROWS - 1][0], src);
                piv = sel ? p1 : piv;
            }
        }
        if constexpr (S == 9) rp = WtType<E>::rcp(piv);
        if constexpr (S == 10 || S == 12) t = fma(-piv, rp, E(1));
        if constexpr (S == 11 || S == 13) rp = fma(t, rp, rp);
    }
};

// Halves of two registers exchanged between the lane halves (32) or between even and odd rows of 16
// lanes (16), then added: lanes of the lower half (even rows) get the sum of a over the pair, the
// others that of b.
__device__ __forceinline__ double wt_fold32(double a, double b) {
    auto lo = __builtin_amdgcn_permlane32_swap(unsigned(__double2loint(a)), unsigned(__double2loint(b)), false, false);
    auto hi = __builtin_amdgcn_permlane32_swap(unsigned(__double2hiint(a)), unsigned(__double2hiint(b)), false, false);
    return __hiloint2double(int(hi[0]), int(lo[0])) + __hiloint2double(int(hi[1]), int(lo[1]));
}
__device__ __forceinline__ float wt_fold32(float a, float b) {
    auto v = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(v[0]) + __uint_as_float(v[1]);
}
__device__ __forceinline__ float wt_fold16(float a, float b) {
    auto v = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(v[0]) + __uint_as_float(v[1]);
}
__device__ __forceinline__ double wt_fold16(double a, double b) {
    auto lo = __builtin_amdgcn_permlane16_swap(unsigned(__double2loint(a)), unsigned(__double2loint(b)), false, false);
    auto hi = __builtin_amdgcn_permlane16_swap(unsigned(__double2hiint(a)), unsigned(__double2hiint(b)), false, false);
    return __hiloint2double(int(hi[0]), int(lo[0])) + __hiloint2double(int(hi[1]), int(lo[1]));
}

template <int NP>
struct WTile {
    static_assert(NP % 8 == 0 && (NP <= 64 || (NP % 16 == 0 && NP <= 112)), "up to 112 rows, 392 tile registers");
    static constexpr int TR = (NP + 15) / 16;     // tiles per side
    static constexpr int ROWS = NP > 64 ? 2 : 1;  // matrix rows per lane where rows lie one per lane
    // column stride of the panel buffer and row stride of the pivot rows (doubles): 4 over a multiple
    // of 16, so the four lane groups of an access start in different banks
    static constexpr int PLD = 16 * TR + 4;
    static constexpr int kScratch = 16 * PLD + 3 * 64 * ROWS;   // panel / pivot rows, vectors, pivot orders
    // Tile columns of the inverse that wait in LDS while the stages run (kPark doubles).  At 112 rows
    // the tiles leave 120 registers where a source term takes about 130; left to itself the compiler
    // spills tiles and reloads them one by one inside the solves (M111: a solve 15 k cycles; ROS4 x 4099 302 -> 291 ms).
    static constexpr int PJ = TR == 7 ? 2 : 0;
    static constexpr int kPark = PJ * TR * 4 * 64;
    using Mat = wd4[TR][TR];
};

// Scratch in LDS (WTile::kScratch doubles): PNL and the pivot rows UB share one buffer.
struct WScratch {
    double *PNL, *BS, *XS;
    int *ORD;
};
template <int NP>
__device__ __forceinline__ WScratch wt_scratch(double *b) {
    WScratch s;
    s.PNL = b;
    s.BS = b + 16 * WTile<NP>::PLD;
    s.XS = s.BS + 64 * WTile<NP>::ROWS;
    s.ORD = reinterpret_cast<int *>(s.XS + 64 * WTile<NP>::ROWS);
    return s;
}

// Lane group G's value on every lane group (permlane swaps of a register with itself).
template <int G>
__device__ __forceinline__ unsigned wt_group(unsigned u) {
    auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    auto q = __builtin_amdgcn_permlane16_swap(h[G >> 1], h[G >> 1], false, false);
    return q[G & 1];
}
template <int G>
__device__ __forceinline__ double wt_group(double x) {
    return __hiloint2double(int(wt_group<G>(unsigned(__double2hiint(x)))), int(wt_group<G>(unsigned(__double2loint(x)))));
}
template <int G>
__device__ __forceinline__ float wt_group(float x) {
    return __uint_as_float(wt_group<G>(__float_as_uint(x)));
}
__device__ __forceinline__ float wt_permute(int addr, float x) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(x)));
}
__device__ __forceinline__ double wt_permute(int addr, double x) {
    return __hiloint2double(__builtin_amdgcn_ds_bpermute(addr, __double2hiint(x)),
                            __builtin_amdgcn_ds_bpermute(addr, __double2loint(x)));
}

// The inverse of a single tile (NP <= 16), in the tile layout: the 16 columns are spread over the lane
// groups, so a pivot costs four multiply-adds instead of fifteen with two lane reads each.  The pivot
// column goes to all groups by permlane swaps, each group takes its four entries of the pivot row
// with a permute, and the search runs over 16 lanes in all groups at once.  What is left is the chain
// column - search - reciprocal - multiplier, about 290 cycles a pivot instead of 525 (M13: ROS4 x 1024
// 66 -> 60 ms, 16 launches of 8 steps x 4096 41 -> 35 ms).  The same pivots, the same operations on
// every entry and so the same bits as one row per lane.  Rows and columns from n on are padding: they
// keep their places and are not eliminated.
template <int NP, class T>
__device__ __forceinline__ bool wt_invert_tile(typename WtType<T>::V &X, int lane, int &order, int n) {
    const int c16 = lane & 15;
    bool done = c16 >= n, ok = true;
    int ord = c16 >= n ? c16 : NP;
    T scale = T(1);
    wt_for<0, NP>([&](auto i) {
        constexpr int k = decltype(i)::value, v0 = k >> 2;
        if (k >= n) return;
        const T col = wt_group<(k & 3)>(T(X[v0]));
        const unsigned key = done ? 0u : WtType<T>::key(col);
        unsigned m = key;
        m = max(m, unsigned(__builtin_amdgcn_update_dpp(0, int(m), 0x128, 0xf, 0xf, true)));     // row_ror 8, 4, 2, 1
        m = max(m, unsigned(__builtin_amdgcn_update_dpp(0, int(m), 0x124, 0xf, 0xf, true)));
        m = max(m, unsigned(__builtin_amdgcn_update_dpp(0, int(m), 0x122, 0xf, 0xf, true)));
        m = max(m, unsigned(__builtin_amdgcn_update_dpp(0, int(m), 0x121, 0xf, 0xf, true)));
        ok = ok && __builtin_amdgcn_readfirstlane(int(m)) != 0;
        const int src = __builtin_ctzll(__builtin_amdgcn_ballot_w64(key == m)) & 15;
        const T piv = wt_readlane(col, src);
        const int from = 4 * ((lane & 48) + src);
        T row[4];
#pragma unroll
        for (int v = 0; v < 4; v++) row[v] = 4 * v < NP ? wt_permute(from, T(X[v])) : T(0);
        T rp = WtType<T>::rcp(piv);
        rp = fma(fma(-piv, rp, T(1)), rp, rp);
        rp = fma(fma(-piv, rp, T(1)), rp, rp);
        const bool me = c16 == src;
        const T gm = me ? T(0) : -col * rp;
#pragma unroll
        for (int v = 0; v < 4; v++)
            if (4 * v < NP) X[v] = fma(gm, row[v], T(X[v]));
        X[v0] = (lane >> 4) == (k & 3) ? (me ? T(1) : gm) : T(X[v0]);
        done = done || me;
        scale = me ? rp : scale;
        ord = me ? k : ord;
    });
#pragma unroll
    for (int v = 0; v < 4; v++) X[v] *= scale;
    order = lane < 16 && ord < NP ? ord : NP;
    return ok;
}

// In-place inverse of the leading NP x NP block (the caller pads rows and columns N..NP-1 with a
// nonzero diagonal and the rest with zeros).  On return lane l holds in ord[r] the pivot order of row
// l + 64 r: that row of the tiles is row ord of the inverse, its column 16 J + j the one that belongs
// to the row of pivot order 16 J + j.  False if a pivot column was zero.  n: rows without the padding.
template <int NP, class T>
__device__ __forceinline__ bool wt_invert(typename WtType<T>::V (&X)[WTile<NP>::TR][WTile<NP>::TR], const WScratch &s,
                                          int lane, int (&ord)[WTile<NP>::ROWS], int n) {
    if constexpr (WTile<NP>::TR == 1) return wt_invert_tile<NP, T>(X[0][0], lane, ord[0], n);
    using TT = WtType<T>;
    constexpr int TR = WTile<NP>::TR, PLD = WTile<NP>::PLD, ROWS = WTile<NP>::ROWS;
    const int g = lane >> 4, c16 = lane & 15;
    T *const PNL = reinterpret_cast<T *>(s.PNL);
    bool done[ROWS], ok = true;
#pragma unroll
    for (int r = 0; r < ROWS; r++) {
        done[r] = lane + 64 * r >= NP;
        ord[r] = NP;
    }
#pragma unroll 1
    for (int p = 0; p < TR; p++) {
        // the panel (tile column 0; tile columns rotate) with one or two rows per lane
        T R[ROWS][16];
#pragma unroll
        for (int I = 0; I < TR; I++)
#pragma unroll
            for (int v = 0; v < 4; v++) PNL[(g + 4 * v) * PLD + 16 * I + c16] = X[0][I][v];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROWS; r++)
#pragma unroll
            for (int j = 0; j < 16; j++) R[r][j] = PNL[j * PLD + min(lane + 64 * r, 16 * TR - 1)];
        __syncthreads();
        // Gauss-Jordan in the panel, columns rotating so that the pivot column is R[.][0].  A pivot row
        // stays unscaled (its multiplier is 0, its own entry 1) and takes the factor 1 / pivot once
        // at the end: every later step is linear in the row.
        const int npv = (NP % 16 != 0 && p == TR - 1) ? NP % 16 : 16;
        T scale[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; r++) scale[r] = T(1);
        PivotSearch<T, ROWS> ps;
        ps.start(R, done);
        wt_for<0, 14>([&](auto i) { ps.template stage<decltype(i)::value>(R); });
#pragma unroll 1
        for (int c8 = 0; c8 < npv; c8 += 8) {
            // eight pivots of straight-line code, so that the rotation is register renaming
#pragma unroll
            for (int c = 0; c < 8; c++) {
                ok = ok && ps.any;
                const int src = ps.src;
                T gm[ROWS], last[ROWS];
#pragma unroll
                for (int r = 0; r < ROWS; r++) {
                    const bool me = lane == src && (ROWS == 1 || ps.sel == (r == 1));
                    gm[r] = me ? T(0) : -R[r][0] * ps.rp;
                    last[r] = me ? T(1) : gm[r];
                    done[r] = done[r] || me;
                    scale[r] = me ? ps.rp : scale[r];
                    ord[r] = me ? 16 * p + c8 + c : ord[r];
                }
                // The next pivot's column first, then its search and reciprocal (a chain of about 20
                // dependent instructions) one stage per updated column: the chain's latency is spent
                // on the other columns' lane reads and multiply-adds.  The order is fixed by hand;
                // left to itself the compiler puts most of the chain behind the last column.
                // Each column's lane reads are issued one column early, which covers the wait between a
                // lane read and the vector instruction that takes its scalar result.
                PivotSearch<T, ROWS> nx;
                auto columns = [&](auto which) {
                    constexpr int Q = decltype(which)::value;       // the pivot row's register
                    T pj = wt_readlane(R[Q][1], src);
                    wt_for<1, 16>([&](auto i) {
                        constexpr int j = decltype(i)::value;
                        const T pn = j < 15 ? wt_readlane(R[Q][j < 15 ? j + 1 : 15], src) : T(0);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int r = 0; r < ROWS; r++) R[r][j - 1] = fma(gm[r], pj, R[r][j]);
                        pj = pn;
                        if (j == 2) nx.start(R, done);
                        if (j > 2) nx.template stage<(j > 2 ? j - 3 : 0)>(R);
                        __builtin_amdgcn_sched_barrier(0);
                    });
                };
                if constexpr (ROWS == 1) {
                    columns(std::integral_constant<int, 0>{});
                } else {
                    if (ps.sel) columns(std::integral_constant<int, ROWS - 1>{});
                    else columns(std::integral_constant<int, 0>{});
                }
                nx.template stage<13>(R);
#pragma unroll
                for (int r = 0; r < ROWS; r++) R[r][15] = last[r];
                ps = nx;
            }
        }
        // npv rotations leave column j in R[.][(j - npv) mod 16]
        const int rot = npv & 15;
#pragma unroll
        for (int r = 0; r < ROWS; r++)
            if (lane + 64 * r < 16 * TR) {
#pragma unroll
                for (int j = 0; j < 16; j++) PNL[((j + rot) & 15) * PLD + lane + 64 * r] = R[r][j] * scale[r];
            }
#pragma unroll
        for (int r = 0; r < ROWS; r++) s.ORD[lane + 64 * r] = ord[r];
        __syncthreads();
#pragma unroll
        for (int I = 0; I < TR; I++)
#pragma unroll
            for (int v = 0; v < 4; v++) X[0][I][v] = PNL[(g + 4 * v) * PLD + 16 * I + c16];
        if (TR > 1) {
            int o[TR];
#pragma unroll
            for (int I = 0; I < TR; I++) o[I] = s.ORD[16 * I + c16] - 16 * p;
            __syncthreads();
            // pivot rows of the other columns into UB (= PNL, the panel is in registers) by pivot
            // order, and out of the tiles
#pragma unroll
            for (int I = 0; I < TR; I++)
                if (o[I] >= 0 && o[I] < 16) {
#pragma unroll
                    for (int J = 1; J < TR; J++)
#pragma unroll
                        for (int v = 0; v < 4; v++) {
                            PNL[o[I] * PLD + 16 * J + g + 4 * v] = X[J][I][v];
                            X[J][I][v] = T(0);
                        }
                }
            __syncthreads();
#pragma unroll
            for (int J = 1; J < TR; J++)
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    if (NP % 16 != 0 && 4 * k >= npv) break;     // no pivots of these orders
                    const T u = PNL[(4 * k + g) * PLD + 16 * J + TT::ucol(c16)];
#pragma unroll
                    for (int I = 0; I < TR; I++) X[J][I] = TT::mfma(u, X[0][I][k], X[J][I]);
                }
            __syncthreads();
            // the next panel becomes tile column 0
            typename TT::V t[TR];
#pragma unroll
            for (int I = 0; I < TR; I++) t[I] = X[0][I];
#pragma unroll
            for (int J = 0; J + 1 < TR; J++)
#pragma unroll
                for (int I = 0; I < TR; I++) X[J][I] = X[J + 1][I];
#pragma unroll
            for (int I = 0; I < TR; I++) X[TR - 1][I] = t[I];
        }
    }
    return ok;
}

// Rows of tiles times a vector given by column (BS holds column o at 4 TR (o % 4) + o / 4, so that the
// values a lane needs are contiguous): row l + 64 r on lane l, register r.
template <int NP>
__device__ __forceinline__ int wt_slot(int o) { return 4 * WTile<NP>::TR * (o & 3) + (o >> 2); }
// PJ: the last PJ tile columns are in LDS (wt_park).
template <int NP, class T, int PJ = 0>
__device__ __forceinline__ void wt_rows(const typename WtType<T>::V (&X)[WTile<NP>::TR][WTile<NP>::TR], const T *BS,
                                        int lane, T (&out)[WTile<NP>::ROWS], const T *park = nullptr) {
    constexpr int TR = WTile<NP>::TR;
    const int g = lane >> 4;
    T bs[4 * TR];
#pragma unroll
    for (int k = 0; k < 4 * TR; k++) bs[k] = 4 * k < NP ? BS[4 * TR * g + k] : T(0);
    T z[8];
#pragma unroll
    for (int I = 0; I < TR; I++) {
        T a = 0, b2 = 0;     // two chains
#pragma unroll
        for (int J = 0; J < TR; J++) {
            auto x = [&](int v) {
                return J < TR - PJ ? X[J][I][v] : park[(4 * ((J - (TR - PJ)) * TR + I) + v) * 64 + lane];
            };
            a = fma(x(0), bs[4 * J], a);
            b2 = fma(x(1), bs[4 * J + 1], b2);
            if (16 * J + 8 < NP) {
                a = fma(x(2), bs[4 * J + 2], a);
                b2 = fma(x(3), bs[4 * J + 3], b2);
            }
        }
        z[I] = a + b2;
    }
    // sum over the lane groups; group g keeps row block I = g (and 4 + g)
    auto fold = [&](int I0, int count) {
        if (count == 1) {
            const T h = wt_fold32(z[I0], z[I0]);
            return wt_fold16(h, h);
        }
        if (count == 2) return wt_fold16(wt_fold32(z[I0], z[I0]), wt_fold32(z[I0 + 1], z[I0 + 1]));
        return wt_fold16(wt_fold32(z[I0], z[I0 + 2]), wt_fold32(z[I0 + 1], count == 4 ? z[I0 + 3] : z[I0 + 1]));
    };
    out[0] = fold(0, TR < 4 ? TR : 4);
    if constexpr (WTile<NP>::ROWS == 2) out[1] = fold(4, TR - 4);
}

// The last WTile::PJ tile columns to LDS.
template <int NP>
__device__ __forceinline__ void wt_park(const wd4 (&X)[WTile<NP>::TR][WTile<NP>::TR], double *park, int lane) {
    constexpr int TR = WTile<NP>::TR, PJ = WTile<NP>::PJ;
#pragma unroll
    for (int J = TR - PJ; J < TR; J++)
#pragma unroll
        for (int I = 0; I < TR; I++)
#pragma unroll
            for (int v = 0; v < 4; v++) park[(4 * ((J - (TR - PJ)) * TR + I) + v) * 64 + lane] = X[J][I][v];
}

// x = A^-1 b from the inverted tiles; component l + 64 r of b and x on lane l, register r.
template <int NP, class T, int PJ = 0>
__device__ __forceinline__ void wt_solve(const typename WtType<T>::V (&X)[WTile<NP>::TR][WTile<NP>::TR],
                                         const WScratch &s, int lane, const int (&ord)[WTile<NP>::ROWS],
                                         const T (&b)[WTile<NP>::ROWS], T (&x)[WTile<NP>::ROWS],
                                         const T *park = nullptr) {
    constexpr int ROWS = WTile<NP>::ROWS;
    T *const BS = reinterpret_cast<T *>(s.BS), *const XS = reinterpret_cast<T *>(s.XS);
#pragma unroll
    for (int r = 0; r < ROWS; r++)
        if (ord[r] < NP) BS[wt_slot<NP>(ord[r])] = b[r];
    __syncthreads();
    T z[ROWS];
    wt_rows<NP, T, PJ>(X, BS, lane, z, park);
#pragma unroll
    for (int r = 0; r < ROWS; r++)
        if (ord[r] < NP) XS[ord[r]] = z[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROWS; r++) x[r] = lane + 64 * r < NP ? XS[lane + 64 * r] : T(0);
    __syncthreads();
}

// A x from the tiles of A itself.
template <int NP>
__device__ __forceinline__ void wt_times(const wd4 (&X)[WTile<NP>::TR][WTile<NP>::TR], const WScratch &s, int lane,
                                         const double (&x)[WTile<NP>::ROWS], double (&z)[WTile<NP>::ROWS]) {
#pragma unroll
    for (int r = 0; r < WTile<NP>::ROWS; r++)
        if (lane + 64 * r < NP) s.BS[wt_slot<NP>(lane + 64 * r)] = x[r];
    __syncthreads();
    wt_rows<NP, double>(X, s.BS, lane, z);
    __syncthreads();
}

}  // namespace ck
