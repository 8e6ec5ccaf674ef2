// Mechanism staging: parse the CKMECH text format, pack structure-of-arrays
// tables and upload them in one device allocation (Section 3 data: NASA-7
// thermodynamics per species, modified Arrhenius rates, stoichiometry,
// third-body efficiencies and fall-off parameters per reaction).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <fstream>
#include <numeric>
#include <sstream>
#include <string>

#include "ck_internal.h"

namespace ck {

namespace {

struct Reader {
    std::ifstream in;
    bool ok = true;
    template <class T>
    T get() {
        T v{};
        if (!(in >> v)) ok = false;
        return v;
    }
    bool word(const char *w) {
        std::string s;
        if (!(in >> s) || s != w) ok = false;
        return ok;
    }
};

}  // namespace

int parse_mechanism(const char *path, HostMech &hm) {
    Reader r;
    r.in.open(path);
    if (!r.in) return CK_EIO;
    if (!r.word("CKMECH") || r.get<int>() != 1 || !r.ok) return CK_EPARSE;
    if (!r.word("CONST")) return CK_EPARSE;
    hm.R = r.get<double>();
    hm.p0 = r.get<double>();
    if (!r.word("ELEMENTS")) return CK_EPARSE;
    hm.nel = r.get<int>();
    if (!r.ok || hm.nel < 1 || hm.nel > 64) return CK_EPARSE;
    for (int e = 0; e < hm.nel; e++) {
        r.word("E");
        r.get<std::string>();
        r.get<double>();
    }
    if (!r.word("SPECIES")) return CK_EPARSE;
    hm.nsp = r.get<int>();
    if (!r.ok || hm.nsp < 1 || hm.nsp + 1 > kMaxN) return r.ok ? CK_EUNSUPPORTED : CK_EPARSE;
    hm.W.resize(hm.nsp);
    hm.Tmid.resize(hm.nsp);
    hm.alow.resize(7 * hm.nsp);
    hm.ahigh.resize(7 * hm.nsp);
    for (int k = 0; k < hm.nsp; k++) {
        r.word("S");
        r.get<std::string>();
        hm.W[k] = r.get<double>();
        int nc = r.get<int>();
        if (!r.ok || nc < 0 || nc > hm.nel) return CK_EPARSE;
        for (int c = 0; c < nc; c++) {
            int e = r.get<int>();
            r.get<int>();
            if (e < 0 || e >= hm.nel) return CK_EPARSE;
        }
        r.get<double>();
        hm.Tmid[k] = r.get<double>();
        r.get<double>();
        for (int j = 0; j < 7; j++) hm.alow[7 * k + j] = r.get<double>();
        for (int j = 0; j < 7; j++) hm.ahigh[7 * k + j] = r.get<double>();
        if (!r.ok || !(hm.W[k] > 0)) return CK_EPARSE;
    }
    if (!r.word("REACTIONS")) return CK_EPARSE;
    hm.nrxn = r.get<int>();
    if (!r.ok || hm.nrxn < 0) return CK_EPARSE;
    hm.rx.resize(hm.nrxn);
    for (auto &x : hm.rx) {
        if (!r.word("R")) return CK_EPARSE;
        x.type = r.get<int>();
        x.rev = r.get<int>();
        int nr = r.get<int>();
        if (!r.ok || x.type < 0 || x.type > 3 || nr < 1 || nr > 3) return CK_EPARSE;
        for (int j = 0; j < nr; j++) {
            x.rsp.push_back(r.get<int>());
            x.rnu.push_back(r.get<int>());
        }
        int np = r.get<int>();
        if (!r.ok || np < 1 || np > 3) return CK_EPARSE;
        for (int j = 0; j < np; j++) {
            x.psp.push_back(r.get<int>());
            x.pnu.push_back(r.get<int>());
        }
        for (int j = 0; j < nr; j++)
            if (x.rsp[j] < 0 || x.rsp[j] >= hm.nsp || x.rnu[j] < 1 || x.rnu[j] > 3) return CK_EPARSE;
        for (int j = 0; j < np; j++)
            if (x.psp[j] < 0 || x.psp[j] >= hm.nsp || x.pnu[j] < 1 || x.pnu[j] > 3) return CK_EPARSE;
        x.A = r.get<double>();
        x.beta = r.get<double>();
        x.Ea = r.get<double>();
        if (x.type >= 2) {
            x.A0 = r.get<double>();
            x.beta0 = r.get<double>();
            x.Ea0 = r.get<double>();
        }
        if (x.type == 3) {
            x.ta = r.get<double>();
            x.T3 = r.get<double>();
            x.T1 = r.get<double>();
            x.T2 = r.get<double>();
        }
        if (x.type >= 1) {
            int ne = r.get<int>();
            if (!r.ok || ne < 0 || ne > hm.nsp) return CK_EPARSE;
            for (int j = 0; j < ne; j++) {
                int s = r.get<int>();
                double a = r.get<double>();
                if (s < 0 || s >= hm.nsp) return CK_EPARSE;
                x.eff.emplace_back(s, a);
            }
        }
        if (!r.ok || !(x.A > 0) || (x.type >= 2 && !(x.A0 > 0))) return CK_EPARSE;
    }
    if (!r.word("END")) return CK_EPARSE;
    return CK_OK;
}

}  // namespace ck

using namespace ck;

namespace {

// Byte layout of the single device block: each table starts 256-byte aligned.
struct Packer {
    std::vector<char> buf;
    size_t add(const void *src, size_t bytes) {
        size_t off = (buf.size() + 255) & ~size_t(255);
        buf.resize(off + std::max<size_t>(bytes, 8));
        if (bytes) std::memcpy(buf.data() + off, src, bytes);
        return off;
    }
    template <class T>
    size_t add(const std::vector<T> &v) { return add(v.data(), v.size() * sizeof(T)); }
};

// A pair-form reaction in the order of storage: its stored index and the species of its four slots
// (nsp: the null species).
struct PairUnits {
    int id;
    int sp[4];
    int type;
};

// Cost of the LDS atomics of 16 consecutive lanes.  An FP64 LDS atomic is served 16 lanes at a time,
// two cycles per pass over 16 banks of 8 bytes, and lanes that meet in a bank take turns (measured:
// 8.4 cycles for 64 lanes without a conflict, 16.5 / 32 / 129 with 2 / 4 / 16 lanes per bank, 30 for
// random species).  The cost is the largest bank load, summed over the accesses of a ROS4 step: six
// per slot to the per-species arrays (four in the Jacobian pass, one in each stage source term) and
// the d wdot/dC entries of two column windows of width `win`: those of the wavefront kernels for N <= 56
// and of the workgroup kernels.  (The one-wavefront ROS4 for 64 < N <= 112 stages three or four windows of
// 32 columns, for which this order is not the best one.)
//
// One load is sixteen counters in a vector, so that an exchange of one reaction is two additions per
// access and the maxima of sixteen accesses are taken together.
typedef uint8_t BankLoad __attribute__((vector_size(16)));
constexpr int kNoBank = 16;             // no access
constexpr int kAccesses = 36;           // 0..3: species of slot b; 4 + 16 w + 4 b + a: window w, slot b, row of slot a

struct BankOf {
    uint8_t at[kAccesses];
};

BankOf banks_of(const PairUnits &r, int nsp, int win) {
    BankOf o;
    std::fill(o.at, o.at + kAccesses, uint8_t(kNoBank));
    for (int b = 0; b < 4; b++) {
        if (r.sp[b] == nsp) continue;
        const int col = r.sp[b] + 1, w = col / win;
        o.at[b] = uint8_t(r.sp[b] & 15);
        for (int a = 0; a < 4; a++) o.at[4 + 16 * w + 4 * b + a] = uint8_t((r.sp[a] * (win | 1) + col - win * w) & 15);
    }
    return o;
}

struct LaneGroup {
    BankLoad load[kAccesses] = {};
    int cost = 0;
};

// Both vectors' entries i and i + 8 folded: after four levels one entry of each of sixteen is left.
BankLoad fold_max(BankLoad a, BankLoad b) {
    return __builtin_elementwise_max(
        __builtin_shufflevector(a, b, 0, 16, 1, 17, 2, 18, 3, 19, 4, 20, 5, 21, 6, 22, 7, 23),
        __builtin_shufflevector(a, b, 8, 24, 9, 25, 10, 26, 11, 27, 12, 28, 13, 29, 14, 30, 15, 31));
}
BankLoad fold4(const BankLoad *v) { return fold_max(fold_max(v[0], v[1]), fold_max(v[2], v[3])); }
int sum_bytes(BankLoad v) {             // entries up to 16: the bytes of half a vector add up to 128
    uint64_t h[2];
    std::memcpy(h, &v, sizeof h);
    return int((h[0] * 0x0101010101010101u) >> 56) + int((h[1] * 0x0101010101010101u) >> 56);
}

struct OneHot {
    BankLoad v[kNoBank + 1] = {};
    OneHot() {
        for (int i = 0; i < 16; i++) v[i][i] = 1;
    }
};

// Group g after reaction `out` has given its lane to `in`.
void exchange(const LaneGroup &g, const BankOf &out, const BankOf &in, const OneHot &one, LaneGroup &o) {
    for (int i = 0; i < kAccesses; i++) o.load[i] = g.load[i] - one.v[out.at[i]] + one.v[in.at[i]];
    const BankLoad s = fold4(o.load);   // four accesses, each of whose maxima ends up in four entries
    o.cost = 6 * (sum_bytes(fold_max(fold_max(s, s), fold_max(s, s))) / 4);
    for (int w = 0; w < 2; w++) {
        const BankLoad *x = o.load + 4 + 16 * w;
        o.cost += sum_bytes(fold_max(fold_max(fold4(x), fold4(x + 4)), fold_max(fold4(x + 8), fold4(x + 12))));
    }
}

// Rearranges pair-form reactions over the lanes (within their type, so that the leading blocks keep
// the fall-off reactions) and the two species of a side over their slots, to keep the lanes of a
// group apart in the LDS banks: first-improvement descent over random exchanges, 60 per reaction
// (M53: largest bank load 3.1 -> 2.0 per species access, 2.1 -> 1.6 per Jacobian entry).  Once per
// loaded mechanism, linear in the reactions: 325 of them 1.3 ms, 784 3.4 ms (24 and 77 ms while every
// exchange counted its groups anew).
void spread_over_banks(std::vector<PairUnits> &v, int nsp) {
    const int n = int(v.size()), N = nsp + 1;
    if (n < 2) return;
    const int win = N > 64 ? (N + 15) / 16 * 8 : (N > 32 ? 32 : (N + 15) / 16 * 16);
    const OneHot one;
    BankOf none;
    std::fill(none.at, none.at + kAccesses, uint8_t(kNoBank));
    std::vector<BankOf> bank(n);
    std::vector<LaneGroup> group((n + 15) / 16);
    LaneGroup ti, tj;
    for (int i = 0; i < n; i++) {
        bank[i] = banks_of(v[i], nsp, win);
        LaneGroup &g = group[i / 16];
        exchange(g, none, bank[i], one, g);
    }
    uint32_t seed = 12345;
    auto draw = [&](int m) {
        seed = seed * 1664525u + 1013904223u;
        return int((uint64_t(seed >> 8) * uint64_t(m)) >> 24);
    };
    for (int move = 0; move < 60 * n; move++) {
        const int i = draw(n), gi = i / 16, kind = draw(6);
        if (kind < 2) {
            int &a = v[i].sp[2 * kind], &b = v[i].sp[2 * kind + 1];
            if (a == b || b == nsp) continue;
            std::swap(a, b);
            const BankOf turned = banks_of(v[i], nsp, win);
            exchange(group[gi], bank[i], turned, one, ti);
            if (ti.cost <= group[gi].cost) {
                group[gi] = ti;
                bank[i] = turned;
            } else {
                std::swap(a, b);
            }
        } else {
            const int j = draw(n), gj = j / 16;
            if (gi == gj || v[i].type != v[j].type) continue;
            exchange(group[gi], bank[i], bank[j], one, ti);
            exchange(group[gj], bank[j], bank[i], one, tj);
            if (ti.cost + tj.cost <= group[gi].cost + group[gj].cost) {
                group[gi] = ti;
                group[gj] = tj;
                std::swap(v[i], v[j]);
                std::swap(bank[i], bank[j]);
            }
        }
    }
}

}  // namespace

extern "C" int ck_mechanism_load(const char *path, int device, ck_mech **out) {
    if (!path || !out) return CK_EINVAL;
    *out = nullptr;
    auto *m = new (std::nothrow) ck_mech;
    if (!m) return CK_ENOMEM;
    int rc = parse_mechanism(path, m->host);
    if (rc != CK_OK) {
        delete m;
        return rc;
    }
    const HostMech &hm = m->host;
    const int ns = hm.nsp, nr = hm.nrxn;

    // species block: W, 1/W, Tmid, then the NASA-7 coefficients, each [nsp]
    std::vector<double> spd(size_t(3 + kThermoCoef) * ns);
    for (int k = 0; k < ns; k++) {
        spd[k] = hm.W[k];
        spd[size_t(ns) + k] = 1.0 / hm.W[k];
        spd[size_t(2) * ns + k] = hm.Tmid[k];
        for (int j = 0; j < 7; j++) {
            spd[size_t(3 + j) * ns + k] = hm.alow[7 * k + j];
            spd[size_t(10 + j) * ns + k] = hm.ahigh[7 * k + j];
        }
    }
    // Stored order: reactions that are not pair-form first, then by type, the most complex first.  The
    // kernels hand consecutive blocks of 64 reactions to the lanes of a wavefront, and a block pays
    // for the most complex type it holds, so the few third-body and fall-off reactions share the
    // leading blocks and the ragged last block holds elementary ones only.  Within a type the lanes
    // of pair-form reactions are chosen by their LDS banks, and general reactions with few species go
    // first (a block of 64 can skip the slots that none of its reactions uses).
    std::vector<int> order(nr);
    std::iota(order.begin(), order.end(), 0);
    auto units = [](const std::vector<int> &nu) { return std::accumulate(nu.begin(), nu.end(), 0); };
    auto slots = [&](int i) { return hm.rx[i].rsp.size() + hm.rx[i].psp.size(); };
    auto pair_form = [&](int i) {
        const auto &x = hm.rx[i];
        const int r = units(x.rnu), p = units(x.pnu);
        return x.rev && r >= 1 && r <= 2 && p >= 1 && p <= 2;
    };
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
        if (pair_form(a) != pair_form(b)) return !pair_form(a);
        if (hm.rx[a].type != hm.rx[b].type) return hm.rx[a].type > hm.rx[b].type;
        return !pair_form(a) && slots(a) < slots(b);
    });
    int n_gen = 0, n_fall = 0;
    for (int i = 0; i < nr; i++) {
        n_gen += !pair_form(i);
        n_fall += pair_form(i) && hm.rx[i].type != kElementary;
    }
    std::vector<PairUnits> units_of(nr - n_gen);
    for (int ii = n_gen; ii < nr; ii++) {
        const auto &x = hm.rx[order[ii]];
        PairUnits &u = units_of[ii - n_gen];
        u.id = order[ii];
        u.type = x.type;
        std::fill(u.sp, u.sp + 4, ns);
        for (size_t j = 0, c = 0; j < x.rsp.size(); j++)
            for (int v = 0; v < x.rnu[j]; v++) u.sp[c++] = x.rsp[j];
        for (size_t j = 0, c = 2; j < x.psp.size(); j++)
            for (int v = 0; v < x.pnu[j]; v++) u.sp[c++] = x.psp[j];
    }
    spread_over_banks(units_of, ns);
    for (int ii = n_gen; ii < nr; ii++) order[ii] = units_of[ii - n_gen].id;
    std::vector<PairBlock> pair(std::max((nr - n_gen + 63) / 64, 1));
    std::memset(pair.data(), 0, pair.size() * sizeof(PairBlock));
    std::vector<FactorBlock> factor(std::max((n_fall + 63) / 64, 1));
    std::memset(factor.data(), 0, factor.size() * sizeof(FactorBlock));
    std::vector<RxnRec> rx(std::max(nr, 1));
    std::vector<FallRec> fall;
    std::vector<EffRec> eff;
    std::vector<int> orig(std::max(nr, 1));
    // Rate parameters within the range of the kernels' exp: a rate constant with |E| / R beyond 2e14 K or
    // |beta| beyond 2e11 is 0 or inf at every temperature from 1 K to 1e11 K, and stays that with the bound.
    auto bound = [](double v, double b) { return std::min(std::max(v, -b), b); };
    for (int ii = 0; ii < nr; ii++) {
        const auto &x = hm.rx[order[ii]];
        RxnRec &R = rx[ii];
        std::memset(&R, 0, sizeof(R));
        orig[ii] = order[ii];
        R.lnA = std::log(x.A);
        R.beta = bound(x.beta, 2e11);
        R.EaR = bound(x.Ea / hm.R, 2e14);
        int s = 0, nu = 0, sp[6] = {0, 0, 0, 0, 0, 0};
        for (size_t j = 0; j < x.rsp.size(); j++, s++) {
            sp[s] = x.rsp[j];
            nu |= x.rnu[j] << (2 * s);
        }
        const int nre = s;
        for (size_t j = 0; j < x.psp.size(); j++, s++) {
            sp[s] = x.psp[j];
            nu |= x.pnu[j] << (2 * s);
        }
        R.meta = (x.type & 3) | ((x.rev ? 1 : 0) << 2) | (s << 3) | (nre << 6) | (int(x.eff.size()) << 9);
        R.eff_begin = int(eff.size());
        for (int j = 0; j < 3; j++) R.sp[j] = sp[2 * j] | (sp[2 * j + 1] << 16);
        R.nu = nu;
        R.fall = -1;
        if (x.type >= 2) {
            FallRec F{};
            F.lnA0 = std::log(x.A0);
            F.beta0 = bound(x.beta0, 2e11);
            F.Ea0R = bound(x.Ea0 / hm.R, 2e14);
            if (x.type == 3) {
                F.a = x.ta;
                // exp(-T / T***) and its like are 0 (or inf) long before these bounds
                F.invT3 = bound(1.0 / x.T3, 1e10);
                F.invT1 = bound(1.0 / x.T1, 1e10);
                F.T2 = bound(x.T2, 1e12);
            }
            R.fall = int(fall.size());
            fall.push_back(F);
        }
        if (ii >= n_gen) {
            PairBlock &B = pair[(ii - n_gen) / 64];
            const int l = (ii - n_gen) % 64;
            const int *u = units_of[ii - n_gen].sp;
            B.lnA[l] = R.lnA;
            B.beta[l] = R.beta;
            B.EaR[l] = R.EaR;
            B.off[l] = make_int4(8 * u[0], 8 * u[1], 8 * u[2], 8 * u[3]);
            if (ii - n_gen < n_fall) {
                FactorBlock &F = factor[(ii - n_gen) / 64];
                if (R.fall >= 0) {
                    const FallRec &r = fall[R.fall];
                    F.lnA0[l] = r.lnA0;
                    F.beta0[l] = r.beta0;
                    F.Ea0R[l] = r.Ea0R;
                    F.a[l] = r.a;
                    F.invT3[l] = r.invT3;
                    F.invT1[l] = r.invT1;
                    F.T2[l] = r.T2;
                }
                int o[3] = {8 * ns, 8 * ns, 8 * ns};
                for (size_t j = 0; j < std::min<size_t>(3, x.eff.size()); j++) {
                    o[j] = 8 * x.eff[j].first;
                    F.am1[j][l] = x.eff[j].second - 1.0;
                }
                F.eff[l] = make_int4(o[0], o[1], o[2], x.type | (int(x.eff.size()) << 2));
                F.eff_begin[l] = R.eff_begin;
            }
        }
        for (auto &e : x.eff) {
            EffRec E{};
            E.am1 = e.second - 1.0;
            E.sp = e.first;
            eff.push_back(E);
        }
    }
    for (int b0 = 0; b0 < n_gen; b0 += 64) {
        const int b1 = std::min(n_gen, b0 + 64);
        int most = 0;
        for (int i = b0; i < b1; i++) most = std::max(most, rx_nslot(rx[i].meta));
        for (int i = b0; i < b1; i++) rx[i].blk_slots = most;
    }
    if (fall.empty()) fall.resize(1);
    if (eff.empty()) eff.resize(1);

    Packer pk;
    const size_t ospd = pk.add(spd), orx = pk.add(rx), ofall = pk.add(fall), oeff = pk.add(eff), oorig = pk.add(orig),
                 opair = pk.add(pair), ofactor = pk.add(factor);

    m->device = device;
    int prev = 0;
    if (hipGetDevice(&prev) != hipSuccess) {
        delete m;
        return CK_EHIP;
    }
    if (hipSetDevice(device) != hipSuccess) {
        delete m;
        return CK_EINVAL;
    }
    void *blk = nullptr;
    if (hipMalloc(&blk, pk.buf.size()) != hipSuccess) {
        hipSetDevice(prev);
        delete m;
        return CK_ENOMEM;
    }
    if (hipMemcpy(blk, pk.buf.data(), pk.buf.size(), hipMemcpyHostToDevice) != hipSuccess) {
        hipFree(blk);
        hipSetDevice(prev);
        delete m;
        return CK_EHIP;
    }
    hipSetDevice(prev);
    m->dev_block = blk;
    m->dev_bytes = pk.buf.size();
    char *b = static_cast<char *>(blk);
    DevMech &d = m->dev;
    d.nsp = ns;
    d.nrxn = nr;
    d.N = ns + 1;
    d.n_eff = int(eff.size());
    d.n_gen = n_gen;
    d.n_fall = n_fall;
    d.R = hm.R;
    d.invR = 1.0 / hm.R;
    d.ln_p0_R = std::log(hm.p0 / hm.R);
    d.spd = reinterpret_cast<const double *>(b + ospd);
    d.rx = reinterpret_cast<const RxnRec *>(b + orx);
    d.pair = reinterpret_cast<const PairBlock *>(b + opair);
    d.factor = reinterpret_cast<const FactorBlock *>(b + ofactor);
    d.fall = reinterpret_cast<const FallRec *>(b + ofall);
    d.eff = reinterpret_cast<const EffRec *>(b + oeff);
    d.orig_index = reinterpret_cast<const int *>(b + oorig);
    *out = m;
    return CK_OK;
}

extern "C" void ck_mechanism_free(ck_mech *m) {
    if (!m) return;
    int prev = 0;
    hipGetDevice(&prev);
    hipSetDevice(m->device);
    if (m->dev_block) hipFree(m->dev_block);
    for (auto &w : m->ws)
        if (w.ptr) hipFree(w.ptr);
    hipSetDevice(prev);
    delete m;
}

extern "C" int ck_mechanism_info(const ck_mech *m, int *n_species, int *n_reactions, int *n_elements) {
    if (!m) return CK_EINVAL;
    if (n_species) *n_species = m->host.nsp;
    if (n_reactions) *n_reactions = m->host.nrxn;
    if (n_elements) *n_elements = m->host.nel;
    return CK_OK;
}
