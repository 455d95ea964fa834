// Wide kernel: source terms of 64 states per workgroup, a lane per state (the
// paper's shallow mapping, Sec. 2.1, with species and reactions split over the
// waves of the workgroup).
//
// All lanes of a wave work on the same reaction: its record sits in scalar
// registers, a falloff or third-body reaction costs only its own step, and every
// LDS access is a row of 64 consecutive states, without bank conflicts.
// Rates as in gather_body.h: single-molecule slots, reverse rates from one
// exponential per species.  The LDS holds two rows a species,
//
//   C_k, exp(g_k)
//
// (the latter g_k in a state where one exceeds 350), and the
// rates of progress of the reactions that the waves evaluate between two
// barriers; enthalpies are evaluated again at the end rather than kept.
//
// Every sum is formed in a fixed order: the waves write their rates of progress to
// LDS, and each sums its own species over a static list.  Waves that add to
// shared rows with atomics (which need a third row) take 2.42 ms where this takes
// 2.52, but in an order, and with last bits, that vary from run to run; waves that
// add in turn 4.39 ms.
//
// What bounds it: issue of FP64 and, a quarter of the time, of the sums'
// instructions (without the sums 1.95 ms).  53 species, 325 reactions, 1048576
// states, CONP, layout C: 2.52 ms (scatter kernel, 4 states and one wave a
// workgroup: 3.50).  78 kB of LDS let two workgroups of 8 waves share a compute
// unit, one evaluating while the other sums (one of 16 waves 3.23 ms, 4 waves
// 3.38).  Two reactions go through their exponentials together, which a wave alone
// would wait for.  13 species, 27 reactions, 262144 states: 0.09 ms (0.22).
#pragma once

#include "gather_body.h"

#ifndef PJ_WPE_WIDE
#define PJ_WPE_WIDE 4
#endif

namespace pj {
namespace {

constexpr int WIDE_STATES = 64;

// (once the reactions are done, the production rates take the rows of the
// exponentials, the further parts of their sums those of the concentrations: at
// most one for every species but the bath gas)
enum { F_C = 0, F_E = 1, F_W = F_E, F_X = F_C, WIDE_ROWS = 2 };
constexpr int WIDE_THREADS = 1024;
// (at the end T's row holds dT/dt)
enum { WS_T = 0, WS_V, WS_P, WS_SDOT, WS_N };

// LDS of a workgroup in doubles: species records (one double longer than their
// rows: reads and writes along the species meet different banks), scalars of the
// states, powers of P0/RT, the rates of progress of a stage (four rows a wave and
// batch, and one of zeros; also the partial sums that waves pass to each other),
// flags of the waves
inline int64_t wide_doubles(int ns, int waves, int batches) {
    return (int64_t)(ns + 1) * (WIDE_ROWS * WIDE_STATES + 1) + (WS_N + 7 + 4 * waves * batches + 1) * WIDE_STATES +
           2 * waves;
}
// Batches of a stage: as many as the LDS holds without costing a workgroup of a
// compute unit (which holds 16 waves).
inline int wide_batches(const GatherMech& gm, int waves) {
    const int all = (gm.nr + 4 * waves - 1) / (4 * waves);
    const int64_t least = wide_doubles(gm.ns, waves, 1) * 8;
    const int64_t groups = std::max<int64_t>(1, std::min<int64_t>(gm.lds_max / least, 16 / waves));
    int n = 1;
    while (n < all && wide_doubles(gm.ns, waves, n + 1) * 8 <= gm.lds_max / groups) ++n;
    return n;
}

// OWN: the most sums of a wave
// 1 / x for a normal x with a normal reciprocal: two Newton steps from the
// hardware's estimate
__device__ inline double reciprocal(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = fma(y, fma(-x, y, 1.0), y);
    return fma(y, fma(-x, y, 1.0), y);
}

template <int FORM, int LAYOUT, int OWN, bool EXT>
__global__ void __launch_bounds__(WIDE_THREADS) __attribute__((amdgpu_waves_per_eu(PJ_WPE_WIDE)))
pj_wide_source(const GatherMech* const gmp, const long n, const long g0, const long g1, const unsigned per, const int stage,
               const double* __restrict__ state, const double* __restrict__ param, double* __restrict__ dstate,
               const double* __restrict__ arr) {
    extern __shared__ double lds[];
    const long qg = g0 + (long)(blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (qg >= g1) return;
    constexpr int S = WIDE_STATES, REC = WIDE_ROWS * S + 1;    // doubles of a species
    GatherPtr gm = (GatherPtr)gmp;
    const int ns = gm->ns, nr = gm->nr, N = ns + 1, bath = ns - 1;
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwave = nthr >> 6;
    static_assert(S == 64, "a lane per state");
    const int s = lane, g = wave, G = nwave;              // state; of the threads of a state
    double* const sp = lds;
    double* const sc = sp + (ns + 1) * REC;
    double* const pw = sc + WS_N * S;
    double* const qr = pw + 7 * S;
    const int rows = 4 * G * stage;                       // rates of progress of a stage
    uint64_t* const masks = reinterpret_cast<uint64_t*>(qr + (rows + 1) * S);     // states, of each wave
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
    bool odd = false, calm = true;
    for (int k = g; k < ns; k += G) {
        const ThermoRec t = record(k);
        const double gk = gibbs(t);
        odd |= !(fabs(gk) <= G_FAR);
        calm &= fabs(gk) <= G_CALM;
        const double e = fexp(gk);
        at_(k, F_E) = e;
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
    auto part = [&](int i) -> double& { return qr[i * S + s]; };
    part(2 * g) = acc.hi;
    part(2 * g + 1) = acc.lo;
    if (tid < S) {
        // an empty slot's species, powers of P0/RT
        at_(ns, F_C) = at_(ns, F_E) = 1.0;
        part(rows) = 0.0;
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
        const uint64_t f = __ballot(odd), c = __ballot(!calm);
        if (lane == 0) {
            masks[2 * wave] = f;
            masks[2 * wave + 1] = c;
        }
    }
    __syncthreads();
    uint64_t mask = 0, wild = 0;
    for (int w = 0; w < nwave; ++w) {
        mask |= masks[2 * w];
        wild |= masks[2 * w + 1];
    }
    const bool far = (mask >> lane) & 1;       // this state's reactions take the exponential of the sum
    // every state's products of exponentials are in range
    const bool quiet = __builtin_amdgcn_readfirstlane((int)(wild | wild >> 32)) == 0;
    if (tid < S) {
        // n_Ns = P V / (R T) - RN(sum of the others)
        dd a{0.0, 0.0};
        for (int q = 0; q < G; ++q) a = dd_add(a, dd{part(2 * q), part(2 * q + 1)});
        at_(bath, F_C) = ((P * Vv) / (RU * T) - a.hi) / Vv;
    }
    if (far) {
        // g itself in place of its exponential
        for (int k = g; k < ns; k += G) at_(k, F_E) = gibbs(record(k));
        if (tid < S) at_(ns, F_E) = 0.0;
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
            r.x[a] = row(r.off[a], F_E);
        }
        r.pw = pw[((r.w >> 8) & 7) * S + s];
        return r;
    };
    typedef double V1 __attribute__((ext_vector_type(1)));
    // the elementary part of two reactions, without branches: the chain of one
    // exponential fills the gaps of the other's
    typedef double V2 __attribute__((ext_vector_type(2)));
    auto ratio = [&](const Rxn& r, bool& ok) {      // kr / kf
        const double f = r.x[0] * r.x[1] * r.x[2], b = r.x[3] * r.x[4] * r.x[5];
        const double bp = b * r.pw, kq = bp * reciprocal(f);
        ok = true;
        if (!quiet)
            ok = normal(f) && normal(b) && normal(bp) && normal(kq);
        return kq;
    };
    auto rates = [&](const Rxn& r0, const Rxn& r1, V2& lnkf, V2& q, bool& ok0, bool& ok1) {
        auto both = [&](auto f) { return V2{f(r0), f(r1)}; };
        lnkf = both([&](const Rxn& r) { return r.lnA + r.b * lnT - r.th * invT; });
        const V2 kf = vmap(lnkf, [](double x) { return fexp_in(x); });
        const V2 Pf = both([](const Rxn& r) { return r.c[0] * r.c[1] * r.c[2]; });
        const V2 Pb = both([](const Rxn& r) { return r.w & GI_REV ? r.c[3] * r.c[4] * r.c[5] : 0.0; });
        // (an irreversible reaction's is 0: its product may overflow with k_f, and inf * 0 is NaN)
        V2 kq = {ratio(r0, ok0), ratio(r1, ok1)};
        if (!(r0.w & GI_REV)) kq[0] = 0.0, ok0 = true;
        if (!(r1.w & GI_REV)) kq[1] = 0.0, ok1 = true;
        q = kf * Pf - (kf * kq) * Pb;
    };
    auto rate = [&](const Rxn& r, uint32_t rec, const Extra& ex, int l, double lnkf, double q, bool ok) {
        const uint32_t w = r.w;
        const int kind = w & 7;
        const double Pf = r.c[0] * r.c[1] * r.c[2], Pb = r.c[3] * r.c[4] * r.c[5];
        if (EXT && kind_table(kind)) {
            DevMech td{};
            td.tab = gm->tab;
            td.tabd = gm->tabd;
            double a, b;
            lnkf += table_lnk(td, kind, (int)(word(rec, l + 7) & 0xFFFF), T, invT, lnT, P, a, b);
            const double kf = fexp(lnkf);
            q = kf * Pf;
            if (w & GI_REV) q -= kf * ratio(r, ok) * Pb;
        }
        // states where the two together could not hold the factors
        const bool bad = far || !ok || !(fabs(lnkf) < LNK_FAR);
        if (__builtin_expect(__any(bad), false)) {
            double y = fexp(lnkf) * Pf;
            if (w & GI_REV) {
                double x = lnkf, mf = 1.0, mb = r.pw;
                int e = 0;
                if (far) {
                    x -= (double)((int)((w >> 8) & 7) - 3) * log(PREF / (RU * T));
                    mb = 1.0;
                }
#pragma unroll
                for (int a = 0; a < NSLOT; ++a) {
                    if (far) {
                        x += a < MAXSIDE ? -r.x[a] : r.x[a];
                    } else {
                        (a < MAXSIDE ? mf : mb) *= __builtin_amdgcn_frexp_mant(r.x[a]);
                        e += a < MAXSIDE ? -__builtin_amdgcn_frexp_exp(r.x[a]) : __builtin_amdgcn_frexp_exp(r.x[a]);
                    }
                }
                y -= scaled_exp(x, mb / mf, e) * Pb;
            }
            q = bad ? y : q;
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
    // Production rates: the rates of progress of `stage` batches go to rows in LDS,
    // then each wave adds the words of its sums, by ascending reaction: no addition
    // depends on the order of the waves.  The sums wait in registers, found by an index
    // that the wave shares; 64 words are loaded a stage ahead, four rows read at a time
    // (53 species, 1048576 states: 2.54 ms; eight 2.58, twelve 2.61).
    const PJ_GLOBAL uint32_t* const words = (const PJ_GLOBAL uint32_t*)gm->wl;
    typedef double Sums __attribute__((ext_vector_type(OWN)));
    Sums sum = 0.0;
    int cur = uniform_load(gm->wo[nwave >> 1], wave);
    const int last = uniform_load(gm->wo[nwave >> 1], wave + 1);
    uint32_t wv = at(words, (uint32_t)(cur + lane));
    auto sums = [&](int p0) {
        for (;;) {
            // of 64 words those of the wave and the stage: row's offset, sum and sign;
            // the others the row of zeros
            const bool in = lane < last - cur && (int)(wv & 0x7FFF) < p0 + rows;
            const int n = __builtin_popcountll(__ballot(in));
            const uint32_t x = (in ? (wv & 0x7FFF) - (uint32_t)p0 : (uint32_t)rows) * (S * 8) | (wv >> 15 & 62) | (wv & 0x80000000u);
            for (int j = 0; j < n; j += 4) {
                double v[4];
                uint32_t u[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    u[c] = word(x, j + c);
                    v[c] = *reinterpret_cast<const double*>(reinterpret_cast<const char*>(qr) + ((u[c] & 0x7FFFFE00u) | (uint32_t)(8 * s)));
                }
                PJ_READS_FIRST();
#pragma unroll
                for (int c = 0; c < 4; ++c) sum[(u[c] & 62) >> 1] += sign31(u[c]) * v[c];
            }
            cur += n;
            wv = at(words, (uint32_t)(cur + lane));
            if (n < 64) break;
        }
    };
    {
        uint32_t rec0 = rec_words(0), rec1 = rec_words(1);
        Extra ex0 = extra(0, rec0);
        const int nb = (nr + 4 * nwave - 1) / (4 * nwave);      // (of the first wave: all meet at the barriers)
        for (int b = 0, t = 0; b < nb; ++b) {
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
                bool ok0, ok1;
                rates(r0, r1, lnkf, q, ok0, ok1);
                q[0] = rate(r0, rec, ex, l, lnkf[0], q[0], ok0);
                q[1] = rate(r1, rec, ex, l + 16, lnkf[1], q[1], ok1);
                // the stage before has been added by all
                if (t == 0 && l == 0) __syncthreads();
                part(wave + nwave * (4 * t + (l >> 4))) = q[0];
                part(wave + nwave * (4 * t + (l >> 4) + 1)) = q[1];
            }
            if (++t == stage || b + 1 == nb) {
                __syncthreads();
                sums(4 * nwave * (b + 1 - t));
                t = 0;
            }
        }
    }
    // (every wave is past its last reaction)
#pragma unroll
    for (int o = 0; o < OWN; ++o) {
        const int to = uniform_load(gm->wt[nwave >> 1], wave * WIDE_OWN + o);
        if (to < 0) continue;
        if (to < ns) at_(to, F_W) = sum[o];
        else at_(to - ns, F_X) = sum[o];
    }
    __syncthreads();

    // ---- T and V/P rows: sums of this thread's species, then of the state's threads
    gm = fresh(gm);
    double np = 0.0, om = 0.0;
    for (int k = g; k < ns; k += G) {
        double wk = at_(k, F_W);
        const int x0 = uniform_load(gm->xs[nwave >> 1], k), x1 = uniform_load(gm->xs[nwave >> 1], k + 1);
        for (int x = x0; x < x1; ++x) wk += at_(x, F_X);
        if (x1 > x0) at_(k, F_W) = wk;
        const double h = enthalpy(record(k));
        np += (FORM == PJ_CONP ? h : h - 1.0) * wk;
        om += at(gm->wfac, (uint32_t)k) * wk;
        if (k == bath) Dp += at_(k, F_C) * cb_chat;
    }
    part(g) = np;
    part(G + g) = om;
    part(2 * G + g) = Dp;
    __syncthreads();
    if (tid < S) {
        np = om = Dp = 0.0;
        for (int q = 0; q < G; ++q) {
            np += part(q);
            om += part(G + q);
            Dp += part(2 * G + q);
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
template <int FORM, int LAYOUT, int OWN, bool EXT>
static hipError_t launch_wide_t(const GatherCall& c) {
    auto k = pj_wide_source<FORM, LAYOUT, OWN, EXT>;
    const int stage = wide_batches(*c.gm, 2 * c.waves);
    const int64_t lds = wide_doubles(c.gm->ns, 2 * c.waves, stage) * 8;
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
                           (long)g0, (long)g1, (unsigned)per, stage, c.state, c.param, c.dstate, c.arr);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <bool EXT>
hipError_t launch_wide_impl(const GatherCall& c) {
    const bool few = c.gm->own[c.waves] <= 8;
#define PJ_W(F, L) \
    if (c.form == F && c.layout == L) \
        return few ? launch_wide_t<F, L, 8, EXT>(c) : launch_wide_t<F, L, WIDE_OWN, EXT>(c);
    PJ_W(PJ_CONP, PJ_LAYOUT_C) PJ_W(PJ_CONP, PJ_LAYOUT_F) PJ_W(PJ_CONV, PJ_LAYOUT_C) PJ_W(PJ_CONV, PJ_LAYOUT_F)
#undef PJ_W
    return hipErrorInvalidValue;
}

}  // namespace pj
