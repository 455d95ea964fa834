// Wide kernel: source terms of 64 states per workgroup, a lane per state (the
// paper's shallow mapping, Sec. 2.1, with species and reactions split over the
// waves of the workgroup).
//
// All lanes of a wave work on the same reaction: its record sits in scalar
// registers, a falloff or third-body reaction costs only its own step, and every
// LDS access is a row of 64 consecutive states, without bank conflicts (an LDS
// FP64 atomic takes 8 cycles so, 17 to 26 at the addresses of kernel_body.h).
// Rates as in gather_body.h: single-molecule slots, reverse rates from one
// exponential per species.  The LDS holds four rows a species,
//
//   C_k, exp(g_k), exp(-g_k), wdot_k
//
// (exp(g) rows hold g where the product of ratios could leave the range);
// enthalpies are evaluated again at the end rather than kept.
//
// What bounds it: FP64 arithmetic.  53 species, 325 reactions, 1048576 states,
// CONP, layout C: 2.41 ms (scatter kernel, 4 states and one wave a workgroup:
// 3.51), about 700 vector instructions a state, half of them the elementary
// part of the rates, a fifth 24 Troe reactions; 110 kB of LDS hold one workgroup
// of 16 waves a compute unit (8 waves 2.94, 4 waves 4.41 ms).  Two reactions go
// through their exponentials together, which a wave alone would wait for (2.74
// ms one after the other).  13 species, 27 reactions: 0.29 ms (0.86).
#pragma once

#include "gather_body.h"

#ifndef PJ_WPE_WIDE
#define PJ_WPE_WIDE 4
#endif

namespace pj {
namespace {

constexpr int WIDE_STATES = 64;

enum { F_C = 0, F_E = 1, F_I = 2, F_W = 3, WIDE_ROWS = 4 };
constexpr int WIDE_THREADS = 1024;
// (at the end T's row holds dT/dt)
enum { WS_T = 0, WS_V, WS_P, WS_SDOT, WS_N };

// LDS of a workgroup in doubles: species records (one double longer than their
// rows: reads and writes along the species meet different banks; two for each
// wave at least, which pass partial sums through rows not in use), scalars of
// the states, powers of P0/RT, flags of the waves
inline int64_t wide_doubles(int ns, int waves) {
    const int records = ns + 1 > 2 * waves ? ns + 1 : 2 * waves;
    return (int64_t)records * (WIDE_ROWS * WIDE_STATES + 1) + (WS_N + 7) * WIDE_STATES + (waves + 1) / 2;
}

template <int FORM, int LAYOUT, int S, bool EXT>
__global__ void __launch_bounds__(WIDE_THREADS) __attribute__((amdgpu_waves_per_eu(PJ_WPE_WIDE)))
pj_wide_source(const GatherMech* const gmp, const long n, const long g0, const long g1, const unsigned per,
               const double* __restrict__ state, const double* __restrict__ param, double* __restrict__ dstate,
               const double* __restrict__ arr) {
    extern __shared__ double lds[];
    const long qg = g0 + (long)(blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (qg >= g1) return;
    constexpr int REC = WIDE_ROWS * S + 1;    // doubles of a species
    GatherPtr gm = (GatherPtr)gmp;
    const int ns = gm->ns, nr = gm->nr, N = ns + 1, bath = ns - 1;
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwave = nthr >> 6;
    static_assert(S == 64, "a lane per state");
    const int s = lane, g = wave, G = nwave;              // state; of the threads of a state
    double* const sp = lds;
    double* const sc = sp + (ns + 1 > 2 * G ? ns + 1 : 2 * G) * REC;
    double* const pw = sc + WS_N * S;
    int* const ints = reinterpret_cast<int*>(pw + 7 * S);
    auto at_ = [&](int k, int f) -> double& { return sp[k * REC + f * S + s]; };

    // ---- states into the C rows (moles) and the scalars
    const uint32_t inv_N = 0xFFFFFFFFu / (uint32_t)N + 1;
    auto by_N = [&](int e) { return (int)__umulhi((uint32_t)e, inv_N); };      // e / N, exact to 2^32 / N
    const long st = qg * S + s, sc_ = st < n ? st : n - 1;
    if (LAYOUT == PJ_LAYOUT_F) {
        for (int i = g; i < N; i += G) {
            const double x = state[(long)i * n + sc_];
            if (i == 0) sc[WS_T * S + s] = x;
            else if (i == 1) sc[(FORM == PJ_CONP ? WS_V : WS_P) * S + s] = x;
            else at_(i - 2, F_C) = x;
        }
    } else {
        // the group's states are contiguous: lanes along them, four loads in flight
        const double* const in = state + qg * (S * (long)N);
        const int total = (int)((n - qg * S < S ? n - qg * S : S)) * N;
        for (int e0 = tid; e0 < S * N; e0 += 4 * nthr) {
            double x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e = e0 + u * nthr;
                x[u] = in[e < total ? e : total - N + (e - by_N(e) * N)];   // (states past the end: the last)
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e = e0 + u * nthr;
                const int q = by_N(e), i = e - q * N;
                if (e >= S * N) break;
                if (i == 0) sc[WS_T * S + q] = x[u];
                else if (i == 1) sc[(FORM == PJ_CONP ? WS_V : WS_P) * S + q] = x[u];
                else sp[(i - 2) * REC + F_C * S + q] = x[u];
            }
        }
    }
    if (tid < S) sc[(FORM == PJ_CONP ? WS_P : WS_V) * S + s] = param[sc_];
    __syncthreads();
    const double T = sc[WS_T * S + s], Vv = sc[WS_V * S + s], P = sc[WS_P * S + s];
    const double invT = 1.0 / T, lnT = log(T), Ctot = P / (RU * T), invV = 1.0 / Vv;

    // ---- thermodynamics of this thread's species, its part of the closure sum
    // and of D' = sum C chat/R
    auto record = [&](int k) {
        union {
            ThermoRec t;
            uint4 w[9];
        } u;
        const PJ_GLOBAL uint4* q = (const PJ_GLOBAL uint4*)gm->th;
        const uint32_t rg = T < at(gm->tmid, (uint32_t)k) ? 0 : 1;
#pragma unroll
        for (int c = 0; c < 9; ++c) u.w[c] = at4(q, (uint32_t)(2 * k + rg) * 9u + c);
        return u.t;
    };
    auto enthalpy = [&](const ThermoRec& t) {
        return t.c[0] + T * (t.c[5] + T * (t.c[6] + T * (t.c[7] + T * t.c[8]))) + t.c[12] * invT;
    };
    auto gibbs = [&](const ThermoRec& t) {
        return enthalpy(t) - (t.c[0] * lnT + T * (t.c[1] + T * (t.c[9] + T * (t.c[10] + T * t.c[11]))) + t.c[13]);
    };
    dd acc{0.0, 0.0};
    double Dp = 0.0, cb_chat = 0.0;
    bool odd = false;
    for (int k = g; k < ns; k += G) {
        const ThermoRec t = record(k);
        const double gk = gibbs(t);
        odd |= !(gk >= G_MIN && gk <= G_MAX);
        const double e = fexp(gk);
        at_(k, F_E) = e;
        at_(k, F_I) = 1.0 / e;
        if (k >= 2 * G) at_(k, F_W) = 0.0;
        const double cp = t.c[0] + T * (t.c[1] + T * (t.c[2] + T * (t.c[3] + T * t.c[4])));
        const double chat = FORM == PJ_CONP ? cp : cp - 1.0;
        if (k < bath) {
            const double m = at_(k, F_C), c = m * invV;
            acc = dd_add(acc, dd{m, 0.0});
            at_(k, F_C) = c;
            Dp += c * chat;
        } else {
            cb_chat = chat;
        }
    }
    // (partial sums in the first 2 G wdot rows)
    at_(2 * g, F_W) = acc.hi;
    at_(2 * g + 1, F_W) = acc.lo;
    if (tid < S) {
        // an empty slot's species, powers of P0/RT
        at_(ns, F_C) = at_(ns, F_E) = at_(ns, F_I) = 1.0;
        if (ns >= 2 * G) at_(ns, F_W) = 0.0;
        const double x = PREF / (RU * T), ix = (RU * T) / PREF;
        pw[0 * S + s] = x * x * x;
        pw[1 * S + s] = x * x;
        pw[2 * S + s] = x;
        pw[3 * S + s] = 1.0;
        pw[4 * S + s] = ix;
        pw[5 * S + s] = ix * ix;
        pw[6 * S + s] = ix * ix * ix;
    }
    {
        const int f = __ballot(odd) ? 1 : 0;
        if (lane == 0) ints[wave] = f;
    }
    __syncthreads();
    int flags = 0;
    for (int w = 0; w < nwave; ++w) flags |= ints[w];
    const bool logs = __builtin_amdgcn_readfirstlane(flags);
    if (tid < S) {
        // n_Ns = P V / (R T) - RN(sum of the others)
        dd a{0.0, 0.0};
        for (int q = 0; q < G; ++q) {
            a = dd_add(a, dd{at_(2 * q, F_W), at_(2 * q + 1, F_W)});
            at_(2 * q, F_W) = at_(2 * q + 1, F_W) = 0.0;
        }
        at_(bath, F_C) = ((P * Vv) / (RU * T) - a.hi) / Vv;
    }
    double lnP = 0.0;
    if (logs) {
        // some g out of range: exponentials of the sums, from g itself
        for (int k = g; k < ns; k += G) at_(k, F_E) = gibbs(record(k));
        if (tid < S) at_(ns, F_E) = 0.0;
        lnP = log(PREF / (RU * T));
    }
    __syncthreads();

    // ---- reactions, four at a time per wave.  One load of 64 words fetches their
    // records, two batches ahead (vector loads: scalar ones return out of order
    // with the LDS reads and would be waited for with them); a reaction's words
    // then go to scalar registers.
    gm = fresh(gm);
    const int nbatch = (nr - wave + 4 * nwave - 1) / (4 * nwave), neff_rec = gm->neff, nfall = gm->nfall;
    const PJ_GLOBAL uint32_t* const recs = (const PJ_GLOBAL uint32_t*)gm->rec;
    const PJ_GLOBAL uint32_t* const effs = (const PJ_GLOBAL uint32_t*)gm->eff;
    const PJ_GLOBAL uint32_t* const falls = (const PJ_GLOBAL uint32_t*)gm->fall;
    const int l16 = lane >> 4, w16 = lane & 15;
    // a batch: reactions wave + nwave (4 b + 0..3), so that every wave has its
    // share of each class; past the end, a record of no kind and empty slots
    auto reaction = [&](int b) {
        const int p = wave + nwave * (4 * b + l16);
        return p < nr ? p : -1;
    };
    auto rec_words = [&](int b) {
        const int p = reaction(b);
        const uint32_t v = at(recs, (uint32_t)(p < 0 ? 0 : p) * 16u + w16);
        return p >= 0 ? v : w16 >= 3 && w16 < 6 ? (uint32_t)ns * 0x10001u : 0u;
    };
    struct Extra {
        uint32_t off, effa, effb, fall;
        double arr;
    };
    // what a batch needs besides its records: third bodies, falloff, the call's
    // own Arrhenius parameters
    auto extra = [&](int b, uint32_t rec) {
        Extra x{0, 0, 0, 0, 0.0};
        if (b >= nbatch) return x;
        // words 3..5, six species, to six lanes as byte offsets of their LDS records
        const int h = w16 >= 3 ? w16 - 3 : 0;
        const uint32_t u = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * ((lane & 48) + 3 + ((h >> 1) & 3)), (int)rec);
        x.off = (h & 1 ? u >> 16 : u & 0xFFFF) * (uint32_t)(REC * 8);
        const int first = wave + nwave * 4 * b, p = reaction(b);
        if (first < neff_rec) {
            const uint32_t e = (uint32_t)(p >= 0 && p < neff_rec ? p + 1 : 0) * 24u;
            x.effa = at(effs, e + w16);
            x.effb = at(effs, e + 16 + (w16 & 7));
        }
        if (first < nfall) x.fall = at(falls, (uint32_t)(p >= 0 && p < nfall ? p : 0) * 16u + w16);
        if (arr) {
            const int o0 = __builtin_amdgcn_readlane(rec, 1), o1 = __builtin_amdgcn_readlane(rec, 17);
            const int o2 = __builtin_amdgcn_readlane(rec, 33), o3 = __builtin_amdgcn_readlane(rec, 49);
            const int o = l16 == 0 ? o0 : l16 == 1 ? o1 : l16 == 2 ? o2 : o3;
            if (w16 < 3) x.arr = arr[w16 * nr + o];
        }
        return x;
    };
    auto word = [&](uint32_t v, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); };
    auto real = [&](uint32_t v, int l) { return __hiloint2double((int)word(v, l + 1), (int)word(v, l)); };
    auto real_of = [&](double v, int l) {
        return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
    };
    char* const mine = reinterpret_cast<char*>(sp + s);
    auto row = [&](int off, int f) -> double& { return *reinterpret_cast<double*>(mine + off + f * (S * 8)); };
    struct Rxn {
        uint32_t w;
        int off[NSLOT];
        double lnA, b, th, c[NSLOT], x[NSLOT], pw;
    };
    auto read = [&](uint32_t rec, const Extra& ex, int l) {
        Rxn r;
        r.w = word(rec, l);
#pragma unroll
        for (int a = 0; a < NSLOT; ++a) r.off[a] = (int)word(ex.off, l + 3 + a);
        if (arr) {
            r.lnA = real_of(ex.arr, l);
            r.b = real_of(ex.arr, l + 1);
            r.th = real_of(ex.arr, l + 2);
        } else {
            r.lnA = real(rec, l + 8);
            r.b = real(rec, l + 10);
            r.th = real(rec, l + 12);
        }
#pragma unroll
        for (int a = 0; a < NSLOT; ++a) {
            // (an empty slot reads the empty species' ones)
            r.c[a] = row(r.off[a], F_C);
            r.x[a] = row(r.off[a], a < MAXSIDE ? F_I : F_E);
        }
        r.pw = pw[((r.w >> 8) & 7) * S + s];
        return r;
    };
    typedef double V1 __attribute__((ext_vector_type(1)));
    // the elementary part of two reactions, without branches: the chain of one
    // exponential fills the gaps of the other's
    typedef double V2 __attribute__((ext_vector_type(2)));
    auto rates = [&](const Rxn& r0, const Rxn& r1, V2& lnkf, V2& q) {
        auto both = [&](auto f) { return V2{f(r0), f(r1)}; };
        lnkf = both([&](const Rxn& r) { return r.lnA + r.b * lnT - r.th * invT; });
        const V2 kf = vmap(lnkf, [](double x) { return fexp_in(x); });
        const V2 Pf = both([](const Rxn& r) { return r.c[0] * r.c[1] * r.c[2]; });
        const V2 Pb = both([](const Rxn& r) { return r.w & GI_REV ? r.c[3] * r.c[4] * r.c[5] : 0.0; });
        // (an irreversible reaction's is 0: its product may overflow with k_f, and inf * 0 is NaN)
        const V2 kq = both([](const Rxn& r) {
            return r.w & GI_REV ? ((r.x[0] * r.x[3]) * (r.x[1] * r.x[4]) * (r.x[2] * r.x[5])) * r.pw : 0.0;
        });
        q = kf * Pf - (kf * kq) * Pb;
    };
    auto rate = [&](const Rxn& r, uint32_t rec, const Extra& ex, int l, double lnkf, double q) {
        const uint32_t w = r.w;
        const int kind = w & 7;
        // what the two together leave out: tabulated rates, exponents near the end
        // of the range, reverse rates from the sum of the exponents
        if (__builtin_expect(logs || __any(!(fabs(lnkf) < -LNK_MIN)) || (EXT && kind_table(kind)), false)) {
            if (EXT && kind_table(kind)) {
                DevMech td{};
                td.tab = gm->tab;
                td.tabd = gm->tabd;
                double a, b;
                lnkf += table_lnk(td, kind, (int)(word(rec, l + 7) & 0xFFFF), T, invT, lnT, P, a, b);
            }
            double dG = 0.0;
            if (logs) {
#pragma unroll
                for (int a = 0; a < NSLOT; ++a) dG += a < MAXSIDE ? -row(r.off[a], F_E) : r.x[a];
                dG -= (double)((int)((w >> 8) & 7) - 3) * lnP;
            } else {
                dG = log(((r.x[0] * r.x[3]) * (r.x[1] * r.x[4]) * (r.x[2] * r.x[5])) * r.pw);
            }
            q = fexp(lnkf) * (r.c[0] * r.c[1] * r.c[2]);
            if (w & GI_REV) q -= fexp(lnkf + dG) * (r.c[3] * r.c[4] * r.c[5]);
        }
        if (kind != K_ELEM && !kind_table(kind)) {
            double M = Ctot;      // + sum (alpha_k - 1) [C]_k
            const int ne = (w >> 24) & 0xF;
            for (int e = 0; e < ne; ++e) {
                const uint32_t u = word(ex.effa, l + (e >> 1));
                const double am1 = e < 6 ? real(ex.effa, l + 4 + 2 * e) : real(ex.effb, l + 2 * (e - 6));
                M += am1 * at_((int)(e & 1 ? u >> 16 : u & 0xFFFF), F_C);
            }
            if (kind == K_THREEBODY) {
                q *= M;
            } else {
                FallRec fr;
                fr.lnA0 = real(ex.fall, l);
                fr.b0 = real(ex.fall, l + 2);
                fr.theta0 = real(ex.fall, l + 4);
#pragma unroll
                for (int c = 0; c < 5; ++c) fr.p[c] = real(ex.fall, l + 6 + 2 * c);
                V1 c = 1.0, d0 = 0.0, d1 = 0.0, d2 = 0.0, d3 = 0.0;
                falloff<EXT, GM_SRC>(fr, kind, CHUNK_SRI | CHUNK_CHEMACT, (w & GI_CHEMACT) != 0, V1(T), V1(invT), V1(lnT),
                                     V1(lnkf), r.b, r.th, V1(M), c, d0, d1, d2, d3);
                q *= c[0];
            }
        }
        return q;
    };
    // (an empty slot adds to the empty species; the third ones are mostly empty)
    auto put = [&](const Rxn& r, double q) {
        atomicAdd(&row(r.off[0], F_W), -q);
        atomicAdd(&row(r.off[1], F_W), -q);
        if (((r.w >> 12) & 3) > 2) atomicAdd(&row(r.off[2], F_W), -q);
        atomicAdd(&row(r.off[3], F_W), q);
        atomicAdd(&row(r.off[4], F_W), q);
        if (((r.w >> 14) & 3) > 2) atomicAdd(&row(r.off[5], F_W), q);
    };
    {
        uint32_t rec0 = rec_words(0), rec1 = rec_words(1);
        Extra ex0 = extra(0, rec0);
        for (int b = 0; b < nbatch; ++b) {
            const uint32_t rec = rec0;
            const Extra ex = ex0;
            rec0 = rec1;
            rec1 = rec_words(b + 2);
            ex0 = extra(b + 1, rec0);
#pragma unroll 1
            for (int l = 0; l < 64; l += 32) {
                const Rxn r0 = read(rec, ex, l), r1 = read(rec, ex, l + 16);
                PJ_READS_FIRST();
                V2 lnkf, q;
                rates(r0, r1, lnkf, q);
                put(r0, rate(r0, rec, ex, l, lnkf[0], q[0]));
                put(r1, rate(r1, rec, ex, l + 16, lnkf[1], q[1]));
            }
        }
    }
    __syncthreads();

    // ---- T and V/P rows: sums of this thread's species, then of the state's threads
    gm = fresh(gm);
    double np = 0.0, om = 0.0;
    for (int k = g; k < ns; k += G) {
        const double wk = at_(k, F_W), h = enthalpy(record(k));
        np += (FORM == PJ_CONP ? h : h - 1.0) * wk;
        om += at(gm->wfac, (uint32_t)k) * wk;
        if (k == bath) Dp += at_(k, F_C) * cb_chat;
    }
    // (through rows of the exponentials, no longer needed)
    at_(g, F_E) = np;
    at_(g, F_I) = om;
    at_(G + g, F_E) = Dp;
    __syncthreads();
    if (tid < S) {
        np = om = Dp = 0.0;
        for (int q = 0; q < G; ++q) {
            np += at_(q, F_E);
            om += at_(q, F_I);
            Dp += at_(G + q, F_E);
        }
        const double Tdot = -T * np / Dp;
        sc[WS_T * S + s] = Tdot;
        sc[WS_SDOT * S + s] = FORM == PJ_CONP ? Vv * Tdot * invT + Vv * RU * T * om / P : P * Tdot * invT + RU * T * om;
    }
    __syncthreads();
    if (LAYOUT == PJ_LAYOUT_F) {
        if (st < n)
            for (int i = g; i < N; i += G)
                dstate[(long)i * n + st] = i == 0 ? sc[WS_T * S + s] : i == 1 ? sc[WS_SDOT * S + s] : Vv * at_(i - 2, F_W);
    } else {
        double* const out = dstate + qg * (S * (long)N);
        const int total = (int)((n - qg * S < S ? n - qg * S : S)) * N;
#pragma unroll 4
        for (int e = tid; e < total; e += nthr) {
            const int q = by_N(e), i = e - q * N;
            out[e] = i == 0 ? sc[WS_T * S + q] : i == 1 ? sc[WS_SDOT * S + q] : sc[WS_V * S + q] * sp[(i - 2) * REC + F_W * S + q];
        }
    }
}

}  // namespace

// (c.waves pairs of waves: a workgroup fills a compute unit with its LDS long
// before 8 waves fill the SIMDs)
template <int FORM, int LAYOUT, bool EXT>
static hipError_t launch_wide_t(const GatherCall& c) {
    auto k = pj_wide_source<FORM, LAYOUT, WIDE_STATES, EXT>;
    const int64_t lds = wide_lds(*c.gm, c.waves);
    if (lds > 65536) {
        static std::atomic<uint64_t> done{0};
        hipError_t e = allow_full_lds((const void*)k, done);
        if (e != hipSuccess) return e;
    }
    // (a grid has fewer than 2^32 threads)
    const int64_t groups = (c.n + WIDE_STATES - 1) / WIDE_STATES, most = 1 << 20;
    for (int64_t g0 = 0; g0 < groups; g0 += most) {
        const int64_t g1 = groups < g0 + most ? groups : g0 + most, per = (g1 - g0 + 7) / 8;
        hipLaunchKernelGGL(k, dim3((unsigned)(8 * per)), dim3(128 * c.waves), (size_t)lds, c.stream, c.d_gm, (long)c.n,
                           (long)g0, (long)g1, (unsigned)per, c.state, c.param, c.dstate, c.arr);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <bool EXT>
hipError_t launch_wide_impl(const GatherCall& c) {
#define PJ_W(F, L) \
    if (c.form == F && c.layout == L) return launch_wide_t<F, L, EXT>(c);
    PJ_W(PJ_CONP, PJ_LAYOUT_C) PJ_W(PJ_CONP, PJ_LAYOUT_F) PJ_W(PJ_CONV, PJ_LAYOUT_C) PJ_W(PJ_CONV, PJ_LAYOUT_F)
#undef PJ_W
    return hipErrorInvalidValue;
}

}  // namespace pj
