// Gather kernels: source terms and sparse / dense Jacobian without atomic
// additions (Curtis, Niemeyer & Sung, pyJac v2, Sec. 2.2 and Sec. 3.4).
//
// kernel_body.h scatters: every reaction adds its products of partials to the
// accumulators of its rows and columns, about 49,000 lane-additions per state
// for 111 species and 784 reactions.  An LDS FP64 atomic at such addresses
// takes 17 to 26 cycles per wave instruction and compute unit here, an LDS
// read 5 to 7, and each guarded addition about ten other instructions: the
// scatter was most of that kernel.  Here a reaction writes only the few
// numbers the sums are made of, and the sums are gathered:
//
//   pool   F_i = c_i kf_i prod C, B_i = c_i kr_i prod C (the two one-way rates
//          of progress), T_ik = Q_M,i (alpha_ik - 1) C_k of its third bodies,
//          q_i, dq_i/dT, dq_i/dS, dE_i
//   rows   d wdot_k / d[C]_j = 1/[C]_j (sum nu_ki (nu'_ij F_i - nu''_ij B_i) + sum nu_ki T_ij)
//
// since dq/d[C]_j of a mass-action rate is its order times the rate over
// [C]_j.  That takes two values per reaction where the partials themselves
// take one for each of its species, so the pool of a state fits beside
// another's in the LDS.  A species that is absent (|C| < 1e-150) enters the
// products as +-1e-150, which leaves every partial by it exact and adds less
// than 1e-100 of anything to the others.
// Coefficients are 1: a coefficient of 2 takes two molecule slots, so a
// contribution is a pool element with a sign, 16 bits in the list.  Sums with
// the same number of contributions share a wave; long ones are spread over
// 2^k neighbouring lanes.  No addition depends on the order of the waves, so
// results are bitwise reproducible at any launch shape.
//
// Reverse rates: kr / kf = prod exp(g_k)^nu (P0/RT)^-dnu from one exponential
// per species in place of one per reaction.  A reaction whose product leaves the
// range of normal numbers, or whose kf would, takes the product of the mantissas
// and the sum of the exponents instead (scaled_exp); a state with a |g_k| above
// 350 (a carbon atom below 240 K), of which two exponentials together need not be
// in range, the exponential of the sum.  Either
// is decided for each state by itself: its results don't depend on its neighbours.
//
// A workgroup evaluates NV states, NV compile-time; every lane works for all
// of them, except that in a Jacobian each wave takes the reactions of one
// state (two states' values would not fit 128 registers).  Phases, each after a
// barrier: (1) one wave the bath-gas closure, the others the species'
// thermodynamics; (2) reactions; (3a) the T and V/P columns from dq/dT and
// dq/dS, (3b) in the same LDS space production rates and the column sums from q
// and dE, which waited in registers; (4) Jacobian entries into an LDS buffer
// (over the same space, in rounds of rows if they don't fit); (5) output,
// coalesced.
//
// Sparse Jacobian of 111 species and 784 reactions, CONP, layout C, 262144
// states: 8.26 ms against the scatter kernels' 11.21 (4 states and 8 waves a
// workgroup, the best of their shapes).  14,100 vector instructions a
// state, 74% of the issue slots of the four SIMDs: list words decoded, reads and
// additions are about 60% of them, the reactions 30%; LDS reads take 44% of the compute
// unit's time, bank conflicts 45% of that.  Writing the output alone takes 1.4
// ms at the fill rate.  Four waves a state: the 40 kB of a state let four
// workgroups share a compute unit, which at 128 registers is all the waves it
// holds (3 waves 9.5 ms, 8 waves 11.3; two states with 8 waves 8.3).  Lists
// sorted so that all lanes of a group add or subtract together save a tenth of
// the instructions, but what they are padded with costs more reads: 8.9 ms.
#pragma once

#include <type_traits>

#include "kernel_body.h"

#ifndef PJ_WPE_SRC
#define PJ_WPE_SRC 4
#define PJ_WPE_JAC 4
#define PJ_WPE_ADJ 3
#endif

namespace pj {
namespace {

// per-state scalars in LDS
enum { SC_LNT = 0, SC_NSUM, SC_CB, SC_ICB, SC_DP, SC_DDP, SC_TT, SC_TS, SC_ST, SC_SS, SC_TDOT, SC_SDOT, SC_OM, SC_SCW,
       SC_T, SC_V, SC_P, SC_INVT, SC_INVV, SC_INVRT, SC_CTOT,
       SC_KAP, SC_VT, SC_VS, SC_LB, SC_N };
// fields of a species record in LDS: {exp g, C, exp -g, h, chat/R}, after the
// reactions {wdot, 1/C, T column sum, h, chat/R}; the adjoint's also {what a unit
// of wdot_k adds to v . f, v of its row}.  The adjoint, which reads six of a
// species at once, keeps them together, an odd number apart (one address; 111
// species, 262144 states 5.83 ms against 5.93 with an array per field); the
// Jacobian, whose lists read single fields, an array each (8.65 ms against 9.28).
enum { A_E = 0, A_C = 1, A_I = 2, A_H = 3, A_CP = 4, A_Y = 5, A_VV = 6, A_W = 0, A_IC = 1, A_VT = 2 };
constexpr double C_TINY = 1e-150;
// |g| up to which two exponentials together are a normal number, and six are
constexpr double G_FAR = 350.0, G_CALM = 115.0;
constexpr double LNK_FAR = 690.0;
__device__ inline bool normal(double x) { return __builtin_amdgcn_class(x, 0x108); }

// The description is read through a pointer into constant memory, made opaque
// again for each phase: its fields then are scalar loads where they are used
// instead of a hundred scalar registers held (and spilled) from the start.
typedef const __attribute__((address_space(4))) GatherMech* GatherPtr;
__device__ inline GatherPtr fresh(GatherPtr p) {
    asm volatile("" : "+s"(p));
    return p;
}
// read at an address that is the same for the whole wave: scalar loads
template <class T>
__device__ inline T uniform_load(const PJ_GLOBAL T* p, int i) {
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(sizeof(T) % 4 == 0, "words");
    union {
        T t;
        uint32_t w[sizeof(T) / 4];
    } u;
    const __attribute__((address_space(4))) uint32_t* q = (const __attribute__((address_space(4))) uint32_t*)(p + i);
#pragma unroll
    for (int k = 0; k < (int)(sizeof(T) / 4); ++k) u.w[k] = q[k];
    return u.t;
#else
    return p[i];
#endif
}
// table element at a 32-bit offset from a uniform base
template <class T>
__device__ inline T at(const PJ_GLOBAL T* base, uint32_t i) {
    return *(const PJ_GLOBAL T*)((const PJ_GLOBAL char*)base + i * (uint32_t)sizeof(T));
}
__device__ inline uint4 at4(const PJ_GLOBAL uint4* base, uint32_t i) {
    const PJ_GLOBAL uint32_t* q = (const PJ_GLOBAL uint32_t*)((const PJ_GLOBAL char*)base + i * 16u);
    typedef uint32_t v4 __attribute__((ext_vector_type(4)));
    const v4 v = *(const PJ_GLOBAL v4*)q;
    return make_uint4(v.x, v.y, v.z, v.w);
}
// Keeps the LDS reads before it ahead of the arithmetic after it: left to
// itself the scheduler, minding registers, waits for each read at its use.
#define PJ_READS_FIRST() __builtin_amdgcn_sched_barrier(0)

__device__ inline double clamp_c(double c) { return fabs(c) < C_TINY ? copysign(C_TINY, c) : c; }
// +1 or -1 from bit 0 / bit 16 / bit 15 / bit 31 of a list word
__device__ inline double sign0(uint32_t w) { return __hiloint2double((int)((w << 31) | 0x3FF00000u), 0); }
__device__ inline double sign16(uint32_t w) { return __hiloint2double((int)(((w << 15) & 0x80000000u) | 0x3FF00000u), 0); }
__device__ inline double sign15(uint32_t w) { return __hiloint2double((int)(((w << 16) & 0x80000000u) | 0x3FF00000u), 0); }
__device__ inline double sign31(uint32_t w) { return __hiloint2double((int)((w & 0x80000000u) | 0x3FF00000u), 0); }

// A constant in scalar registers: an addend held there goes straight into the
// multiply-add, where a literal would first be moved into two vector registers.
__device__ inline double sconst(double c) {
    long b = __builtin_bit_cast(long, c);
    asm("" : "+s"(b));
    return __builtin_bit_cast(double, b);
}
// exp(x): x = n ln 2 + r, |r| <= ln(2)/2, in two steps (Cody and Waite), then
// 1 + r + r^2 q(r) with q of degree 9 interpolating (exp(r) - 1 - r)/r^2 at the
// Chebyshev nodes (error 1.3e-17), and the scale by 2^n.
// fexp_in: |x| < 708.
__device__ inline double fexp_in(double x) {
    const double n = __builtin_rint(x * sconst(0x1.71547652b82fep+0));
    double r = fma(-n, sconst(0x1.62e42fefa39efp-1), x);
    r = fma(-n, sconst(0x1.abc9e3b39803fp-56), r);
    double q = sconst(0x1.af38a9b0ec855p-26);
    q = fma(q, r, sconst(0x1.289185613a3d6p-22));
    q = fma(q, r, sconst(0x1.71de0dae63bb3p-19));
    q = fma(q, r, sconst(0x1.a019b90d2ae7ap-16));
    q = fma(q, r, sconst(0x1.a01a01a7c41d5p-13));
    q = fma(q, r, sconst(0x1.6c16c1788bd90p-10));
    q = fma(q, r, sconst(0x1.11111111109b3p-7));
    q = fma(q, r, sconst(0x1.5555555553d63p-5));
    q = fma(q, r, sconst(0x1.5555555555556p-3));
    q = fma(q, r, 0.5);
    return ldexp(1.0 + fma(r * r, q, r), (int)n);
}
// m 2^e exp(x) where the parts may be out of range, for m in [1e-8, 1e8], |e| <
// 2^13
__device__ inline double scaled_exp(double x, double m, int e) {
    const double c = fmin(fmax(x, -1e4), 1e4);
    const double n = __builtin_rint(c * 0x1.71547652b82fep+0);
    double r = fma(-n, 0x1.62e42fefa39efp-1, c);
    r = fma(-n, 0x1.abc9e3b39803fp-56, r);
    const double y = ldexp(fexp_in(r) * m, (int)n + e);
    return x != x ? x : y;
}
__device__ inline double fexp(double x) {
    double y = fexp_in(x);
    y = x > 710.0 ? __builtin_inf() : y;
    return x < -746.0 ? 0.0 : y;
}

// f on every element
template <class V, class F>
__device__ inline V vmap(V x, F f) {
#pragma unroll
    for (int v = 0; v < (int)(sizeof(x) / 8); ++v) x[v] = f(x[v]);
    return x;
}
template <class V>
__device__ inline V vexp(const V& x) { return vmap(x, [](double y) { return fexp(y); }); }
template <class V>
__device__ inline V vlog10(const V& x) { return vmap(x, [](double y) { return log10(y); }); }

// Pressure modification c of a falloff reaction and its derivatives by [M] and
// T; adjoint: Pr dc/dPr at fixed [M] and the factor qA (dq/d ln A = q qA - R Pr dc/dPr).
template <bool EXT, int MODE, class V>
__device__ __forceinline__ void falloff(const FallRec& fr_, int kind, uint32_t cm, bool chemact, const V& T, const V& invT,
                                        const V& lnT, const V& lnkf, double bexp, double th, const V& M, V& c, V& dcdM,
                                        V& dcdT, V& Pr_dcdPr, V& qA) {
    constexpr bool DER = MODE != GM_SRC, ADJ = MODE == GM_ADJ;
    const V rk = vexp(fr_.lnA0 + fr_.b0 * lnT - fr_.theta0 * invT - lnkf);     // k0 / k_inf
    const V Pr = M * rk;
    V F = 1.0, dlF_dlP = 0.0, dlF_dT = 0.0;
    if (kind == K_TROE) {
        const double al = fr_.p[0], i3 = fr_.p[1], i1 = fr_.p[2], t2 = fr_.p[3];
        const V e3 = vexp(-T * i3), e1x = vexp(-T * i1), e2 = vexp(-t2 * invT);
        const V Fc = (1.0 - al) * e3 + al * e1x + e2;
        const V lf = vlog10(Fc);
        const V cc = -0.4 - 0.67 * lf;
        const V nn = 0.75 - 1.27 * lf;
        const V Aa = vlog10(Pr) + cc;
        const V Bd = nn - 0.14 * Aa;
        const V f = Aa / Bd;
        const V den = 1.0 + f * f;
        const V lF = lf / den;
        F = vexp(LN10 * lF);
        if (DER) {
            const V gg = -2.0 * lf * f / (den * den);
            dlF_dlP = gg * nn / (Bd * Bd);
            const V df_dL = (-0.67 * Bd + 1.1762 * Aa) / (Bd * Bd);
            const V dlF_dL = 1.0 / den + gg * df_dL;
            const V dFc = -(1.0 - al) * i3 * e3 - al * i1 * e1x + t2 * invT * invT * e2;
            dlF_dT = dlF_dL * dFc / (Fc * LN10);
        }
    } else if (EXT && (cm & CHUNK_SRI) && kind == K_SRI) {
        const double a = fr_.p[0], bb = fr_.p[1], ic = fr_.p[2], ee = fr_.p[4];
        const V lP = vlog10(Pr);
        const V Xs = 1.0 / (1.0 + lP * lP);
        const V eb = vexp(-bb * invT), ec = vexp(-T * ic);
        const V base = a * eb + ec;
        const V lb = vlog10(base);
        const V lF = fr_.p[3] + Xs * lb + ee * lnT * (1.0 / LN10);
        F = vexp(LN10 * lF);
        if (DER) {
            dlF_dlP = -2.0 * lb * lP * Xs * Xs;
            const V dbase = a * bb * invT * invT * eb - ic * ec;
            dlF_dT = (Xs * dbase / base + ee * invT) * (1.0 / LN10);
        }
    }
    const V ip = 1.0 / (1.0 + Pr);
    const bool chem = EXT && (cm & CHUNK_CHEMACT) && chemact;
    c = chem ? F * rk * ip : F * Pr * ip;
    if (DER) {
        const V dlnPr = (fr_.b0 + fr_.theta0 * invT) * invT - (bexp + th * invT) * invT;
        if (!chem) {
            const V dc_dPr = F * ip * ip + F * ip * dlF_dlP;
            dcdM = dc_dPr * rk;
            if (ADJ) Pr_dcdPr = Pr * dc_dPr;
            dcdT = dc_dPr * Pr * dlnPr + c * LN10 * dlF_dT;
        } else {
            dcdM = c * (dlF_dlP / M - rk * ip);
            dcdT = c * (ip + dlF_dlP) * dlnPr + c * LN10 * dlF_dT;
            if (ADJ) qA = Pr * ip - dlF_dlP;
        }
    }
}

// a value that all lanes hold, in scalar registers
__device__ inline double uniform(double v) {
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                            __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

template <int CTRL>
__device__ inline double dpp(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
// a value and that of lane ^ 16 / lane ^ 32, in the same order in both lanes
__device__ inline void both_x16(double v, double& a, double& b) {
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto x = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto y = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    a = __hiloint2double((int)y[0], (int)x[0]);
    b = __hiloint2double((int)y[1], (int)x[1]);
}
__device__ inline void both_x32(double v, double& a, double& b) {
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto x = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto y = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    a = __hiloint2double((int)y[0], (int)x[0]);
    b = __hiloint2double((int)y[1], (int)x[1]);
}
__device__ inline double add_x16(double v) {
    double a, b;
    both_x16(v, a, b);
    return a + b;
}
__device__ inline double add_x32(double v) {
    double a, b;
    both_x32(v, a, b);
    return a + b;
}
// double-double sum over the wave (data-parallel moves: a shuffle through the
// LDS would add its latency twelve times to the chain)
__device__ inline dd wave_total(dd v) {
    v = dd_add(v, dd{dpp<0xB1>(v.hi), dpp<0xB1>(v.lo)});
    v = dd_add(v, dd{dpp<0x4E>(v.hi), dpp<0x4E>(v.lo)});
    v = dd_add(v, dd{dpp<0x141>(v.hi), dpp<0x141>(v.lo)});
    v = dd_add(v, dd{dpp<0x140>(v.hi), dpp<0x140>(v.lo)});
    double a, b, c, d;
    both_x16(v.hi, a, b);
    both_x16(v.lo, c, d);
    v = dd_add(dd{a, c}, dd{b, d});
    both_x32(v.hi, a, b);
    both_x32(v.lo, c, d);
    return dd_add(dd{a, c}, dd{b, d});
}
// sum over the wave
__device__ inline double wave_total(double v) {
    v += dpp<0xB1>(v);       // lane ^ 1
    v += dpp<0x4E>(v);       // lane ^ 2
    v += dpp<0x141>(v);      // the other four of eight
    v += dpp<0x140>(v);      // the other eight of sixteen
    return add_x32(add_x16(v));
}
// sum over this lane's 2^lp neighbours (at most 2^most in the wave), complete
// in the first of them
__device__ inline double fold(double v, int most, int lp) {
    if (most > 0) { const double t = v + dpp<0xB1>(v); v = lp > 0 ? t : v; }
    if (most > 1) { const double t = v + dpp<0x4E>(v); v = lp > 1 ? t : v; }
    if (most > 2) { const double t = v + dpp<0x141>(v); v = lp > 2 ? t : v; }
    if (most > 3) { const double t = v + dpp<0x140>(v); v = lp > 3 ? t : v; }
    if (most > 4) { const double t = add_x16(v); v = lp > 4 ? t : v; }
    if (most > 5) { const double t = add_x32(v); v = lp > 5 ? t : v; }
    return v;
}

}  // namespace

// One group of NV consecutive states; every lane works for all of them, NV
// values at a time (list words, records and addresses are shared by the
// states, an LDS element is one access of NV doubles).
template <int FORM, int LAYOUT, int MODE, int NV, bool EXT>
__device__ __forceinline__ void gather_group(GatherPtr gmp, const long n,
                                             const double* __restrict__ state, const double* __restrict__ param,
                                             double* __restrict__ dstate, double* __restrict__ jac,
                                             const double* __restrict__ arr, const long qg,
                                             const double* __restrict__ vin = nullptr, double* const GR = nullptr) {
    extern __shared__ double lds[];
    typedef double V __attribute__((ext_vector_type(NV)));
    constexpr bool JAC = MODE == GM_JAC || MODE == GM_DENSE, dense = MODE == GM_DENSE, ADJ = MODE == GM_ADJ;
    static_assert(!ADJ || NV == 1, "an adjoint's workgroup holds one state");
    constexpr bool DER = MODE != GM_SRC;
    constexpr int RB = GATHER_BLOCKS;    // most blocks of reactions of a wave
    constexpr int layout = LAYOUT;
    const int ns = gmp->ns, nr = gmp->nr, N = ns + 1, bath = ns - 1;
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwave = nthr >> 6;

    double* const pool = lds;
    // source terms: the pool holds q only (and an empty reaction's zero)
    // (the adjoint: without the elements from b3 on)
    const int npool = JAC ? gmp->npool : ADJ ? gmp->b3 : ((nr + 2) & ~1);
    double* const A = pool + npool * NV;
    constexpr int AS = ADJ ? 7 : 5;                 // fields of a species
    auto fld = [&](int k, int f) { return ADJ ? k * AS + f : f * (ns + 1) + k; };
    double* const VS = A + AS * (ns + 1) * NV;      // V/P column sums; before them dCp/dT
    double* const TQ = VS + (DER ? (ns + 1) * NV : 0);
    double* const SQ = TQ + (JAC ? (ns + 1) * NV : 0);
    double* const BB = SQ + (JAC ? (ns + 1) * NV : 0);
    double* const PW = BB + (JAC ? (gmp->n_dense_rows + 1) * NV : 0);
    double* const SC = PW + 7 * NV;
    constexpr int NRS = ADJ ? 7 : JAC ? 4 : 0;      // the waves' sums over reactions
    double* const RS = SC + SC_N * NV;
    int* const ints = reinterpret_cast<int*>(RS + NRS * (MAX_THREADS / 64) * NV);   // flags of the waves
    // (dynamic LDS starts at address 0: the kernels have no other)
    typedef __attribute__((address_space(3))) V LV;
    auto vec = [](double* p, int i) -> V& { return *reinterpret_cast<V*>(p + i * NV); };
    auto PO = [&](int i) -> V& { return vec(pool, i); };
    auto SP = [&](int k, int f) -> V& { return vec(A, fld(k, f)); };
    auto K = [&](int q) { return vec(SC, q); };
    auto vclamp = [&](const auto& x) { return vmap(x, [](double y) { return clamp_c(y); }); };
    // the reactions of a Jacobian hold too much in registers for several
    // states: there each wave works for one, state rst
    constexpr int RN = DER ? 1 : NV;
    typedef double RV __attribute__((ext_vector_type(RN)));
    const int rst = RN == NV ? 0 : wave % NV, rwave = RN == NV ? wave : wave / NV, rnw = RN == NV ? nwave : nwave / NV;
    auto rvec = [&](double* p, int i) -> RV& { return *reinterpret_cast<RV*>(p + rst + i * NV); };

    // blocks of 64 reactions: the costliest (first-sorted) go to the waves in
    // turn, the next ones in the reverse turn, so that a wave with a falloff
    // block takes fewer; the first record is loaded at once
    const int nblk = (nr + 63) >> 6;
    auto block_of = [&](int r) { return r * rnw + (r & 1 ? rnw - 1 - rwave : rwave); };
    auto rec_at = [&](GatherPtr gm, int b) {
        const uint32_t p = (uint32_t)(b * 64 + lane);
        const PJ_GLOBAL uint4* q = (const PJ_GLOBAL uint4*)gm->rec;
        union {
            FastRec r;
            uint4 v[4];
        } u;
        const uint32_t i = (p < (uint32_t)nr ? p : (uint32_t)nr - 1) * 4u;
#pragma unroll
        for (int k = 0; k < 4; ++k) u.v[k] = at4(q, i + k);
        return u.r;
    };
    FastRec nxt = rec_at(gmp, block_of(0));

    // ---- (1) closure (wave 0), thermodynamics (the others; with one wave all)
    const int tb = nwave > 1 ? 64 : 0;
    bool odd_c = false;
    int far_g = 0;                               // by state
    // (a state past the end computes a copy of the last)
    auto clamp_state = [&](int v) { const long q = qg * NV + v; return q < n ? q : n - 1; };
    auto X = [&](long sc, int i) -> double { return layout == PJ_LAYOUT_F ? state[(long)i * n + sc] : state[sc * (long)N + i]; };
    if (wave == 0) {
        // n_Ns = P V / (R T) - RN(sum of the others)
        dd acc[NV];
        double T[NV], Sv[NV], Q[NV], vT[NV], vS[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const long sc = clamp_state(v);
            T[v] = X(sc, 0);
            Sv[v] = X(sc, 1);
            Q[v] = param[sc];
            if (ADJ) {
                vT[v] = layout == PJ_LAYOUT_F ? vin[sc] : vin[sc * (long)N];
                vS[v] = layout == PJ_LAYOUT_F ? vin[n + sc] : vin[sc * (long)N + 1];
            }
            acc[v] = dd{0.0, 0.0};
        }
        for (int k = lane; k < ns - 1; k += 64)
#pragma unroll
            for (int v = 0; v < NV; ++v) acc[v] = dd_add(acc[v], dd{X(clamp_state(v), 2 + k), 0.0});
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[v] = wave_total(acc[v]);
        // lane v finishes state v
        double t = T[0], sv = Sv[0], q = Q[0], nsum = acc[0].hi, wt = ADJ ? vT[0] : 0.0, ws = ADJ ? vS[0] : 0.0;
#pragma unroll
        for (int v = 1; v < NV; ++v)
            if (lane == v) {
                t = T[v];
                sv = Sv[v];
                q = Q[v];
                nsum = acc[v].hi;
                if (ADJ) {
                    wt = vT[v];
                    ws = vS[v];
                }
            }
        const double Vv = FORM == PJ_CONP ? sv : q, P = FORM == PJ_CONP ? q : sv;
        const double cb = ((P * Vv) / (RU * t) - nsum) / Vv;
        odd_c |= !(fabs(cb) >= C_TINY);
        if (lane < NV) {
            auto put = [&](double* p, int i, double x) { p[i * NV + lane] = x; };
            put(A, fld(bath, A_C), cb);
            put(A, fld(ns, A_E), 1.0);
            put(A, fld(ns, A_C), 1.0);
            put(A, fld(ns, A_I), 1.0);
            put(A, fld(ns, A_H), 0.0);
            put(SC, SC_NSUM, nsum);
            put(SC, SC_CB, cb);
            put(SC, SC_ICB, 1.0 / clamp_c(cb));
            put(SC, SC_T, t);
            put(SC, SC_V, Vv);
            put(SC, SC_P, P);
            put(SC, SC_INVT, 1.0 / t);
            put(SC, SC_INVV, 1.0 / Vv);
            put(SC, SC_INVRT, 1.0 / (RU * t));
            put(SC, SC_CTOT, P / (RU * t));
            const double x = PREF / (RU * t), ix = (RU * t) / PREF;
            put(PW, 0, x * x * x);
            put(PW, 1, x * x);
            put(PW, 2, x);
            put(PW, 3, 1.0);
            put(PW, 4, ix);
            put(PW, 5, ix * ix);
            put(PW, 6, ix * ix * ix);
            if (JAC) {
                put(pool, gmp->zero, 0.0);
                put(BB, 0, 0.0);
                put(pool, gmp->b3 + 2 * nr, 0.0);
                put(pool, gmp->b3 + 2 * nr + 1, 0.0);
            } else if (ADJ) {
                put(SC, SC_VT, wt);
                put(SC, SC_VS, ws);
                put(pool, gmp->zero, 0.0);
                put(A, fld(ns, A_CP), 0.0);
                put(A, fld(ns, A_Y), 0.0);
                put(A, fld(ns, A_VV), 0.0);
            } else {
                put(pool, nr, 0.0);
            }
        }
    }
    // one species of one state per lane
    auto thermo = [&](int logs) {
        const GatherPtr gm = fresh(gmp);
        for (int it = tid - tb; it < ns * NV; it += nthr - tb) {
            const int k = NV == 1 ? it : it / NV, v = NV == 1 ? 0 : it - k * NV;
            if (logs && !((logs >> v) & 1)) continue;
            const long sc = clamp_state(v);
            const double T = X(sc, 0);
            const int rg = T < at(gm->tmid, (uint32_t)k) ? 0 : 1;
            ThermoRec tr;
            {
                union {
                    ThermoRec t;
                    uint4 w[9];
                } u;
                const PJ_GLOBAL uint4* q = (const PJ_GLOBAL uint4*)gm->th;
#pragma unroll
                for (int c = 0; c < 9; ++c) u.w[c] = at4(q, (uint32_t)(2 * k + rg) * 9u + c);
                tr = u.t;
            }
            if (!logs && k < ns - 1) {
                const double c = X(sc, 2 + k) / (FORM == PJ_CONP ? X(sc, 1) : param[sc]);
                odd_c |= !(fabs(c) >= C_TINY);
                A[fld(k, A_C) * NV + v] = c;
            }
            const double lnT = log(T), invT = 1.0 / T;
            if (k == 0) SC[SC_LNT * NV + v] = lnT;
            auto a = [&](int q) { return tr.c[q]; };
            const double a0 = a(0), a1 = a(1);
            const double cp = a0 + T * (a1 + T * (a(2) + T * (a(3) + T * a(4))));
            const double h = a0 + T * (a(5) + T * (a(6) + T * (a(7) + T * a(8)))) + a(12) * invT;
            const double sr = a0 * lnT + T * (a1 + T * (a(9) + T * (a(10) + T * a(11)))) + a(13);
            const double g = h - sr;
            if (!(fabs(g) <= G_FAR)) far_g |= 1 << v;
            if (logs) {
                A[fld(k, A_E) * NV + v] = g;
            } else {
                const double e = fexp(g);
                A[fld(k, A_E) * NV + v] = e;
                A[fld(k, A_I) * NV + v] = 1.0 / e;
                A[fld(k, A_H) * NV + v] = h;
                A[fld(k, A_CP) * NV + v] = FORM == PJ_CONP ? cp : cp - 1.0;
                if (ADJ) A[fld(k, A_VV) * NV + v] = k < ns - 1 ? layout == PJ_LAYOUT_F ? vin[(2 + k) * (long)n + sc] : vin[sc * (long)N + 2 + k] : 0.0;
                if (DER) VS[k * NV + v] = a1 + T * (a(14) + T * (a(15) + T * a(16)));
            }
        }
    };
    if (tid >= tb) thermo(0);
    {
        int f = __ballot(odd_c) ? 1 << NV : 0;
#pragma unroll
        for (int v = 0; v < NV; ++v) f |= __ballot((far_g >> v) & 1) ? 1 << v : 0;
        if (lane == 0) ints[wave] = f;
    }
    __syncthreads();
    int flags = 0;
    for (int w = 0; w < nwave; ++w) flags |= ints[w];
    flags = __builtin_amdgcn_readfirstlane(flags);
    const int logs = flags & ((1 << NV) - 1);       // states whose reactions take the exponential of the sum
    const bool tiny = flags >> NV;
    if (logs) {
        // g itself in place of its exponential
        if (tid >= tb) thermo(logs);
        if (tid < NV && (logs >> tid) & 1) A[fld(ns, A_E) * NV + tid] = 0.0;
        __syncthreads();
    }

    // adjoint: J^T v of the reactions is sum_i lambda_i grad q_i with lambda_i =
    // v_T dTdot/dq_i + v_S dSdot/dq_i + V sum_k nu_ki v_k = sum_k nu_ki Y_k
    if constexpr (ADJ) {
        const GatherPtr gm = fresh(gmp);
        V d0 = 0.0;
        for (int k = lane; k < ns; k += 64) d0 += SP(k, A_C) * SP(k, A_CP);
        const V Dp = vmap(d0, [](double x) { return wave_total(x); });
        if (wave == 0 && lane == 0) vec(SC, SC_DP) = Dp;
        for (int k = tid; k < ns; k += nthr) {
            const double T = SC[SC_T], Vv = SC[SC_V], P = SC[SC_P], vT = SC[SC_VT], vS = SC[SC_VS];
            const double a = -(vT + vS * (FORM == PJ_CONP ? Vv : P) * SC[SC_INVT]) / Dp[0];
            const double b = vS * RU * T * (FORM == PJ_CONP ? Vv / P : 1.0);
            const double h = A[fld(k, A_H)];
            A[fld(k, A_Y)] = Vv * A[fld(k, A_VV)] + (a * T) * (FORM == PJ_CONP ? h : h - 1.0) + b * at(gm->wfac, (uint32_t)k);
            if (k == 0) SC[SC_KAP] = a;
        }
        __syncthreads();
    }

    // ---- (2) reactions
    if (wave == nwave - 1) {
        V d0 = 0.0, d1 = 0.0;   // D' = sum C chat/R, dD'/dT = sum C dCp/R/dT
        for (int k = lane; k < ns; k += 64) {
            const V c = SP(k, A_C);
            d0 += c * SP(k, A_CP);
            if (DER) d1 += c * vec(VS, k);
        }
        d0 = vmap(d0, [](double x) { return wave_total(x); });
        if (DER) d1 = vmap(d1, [](double x) { return wave_total(x); });
        if (lane == 0) {
            if (!ADJ) vec(SC, SC_DP) = d0;
            if (DER) vec(SC, SC_DDP) = d1;
        }
    }
    // q and dE of this lane's reactions wait in registers while dq/dT and dq/dS
    // are summed in the same LDS space
    RV hq[RB], he[RB];
    {
        const GatherPtr gm = fresh(gmp);
        typedef RV V;
        auto vec = rvec;
        auto PO = [&](int i) -> V& { return vec(pool, i); };
        auto SP = [&](int k, int f) -> V& { return vec(A, fld(k, f)); };
        auto K = [&](int q) { return vec(SC, q); };
        auto U = [&](int q) { return RN == 1 ? vmap(K(q), [](double x) { return uniform(x); }) : K(q); };
        const V T = U(SC_T), lnT = U(SC_LNT), invT = U(SC_INVT), Ctot = U(SC_CTOT);
        const int b3 = DER ? gm->b3 : 0, neff_rec = gm->neff;
        auto far = [&](int v) { return ((logs >> (RN == NV ? v : rst)) & 1) != 0; };
        // sums over reactions: dE dq/dT, dE dq/dS, dOmega dq/dT, dOmega dq/dS;
        // adjoint: lambda dq/dT, lambda dq/dS, lambda dq/dC_Ns, then the energy, mole,
        // heat capacity and (CONP) v weighted rates
        V s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0, s4 = 0.0, s5 = 0.0, s6 = 0.0;
        for (int r = 0; block_of(r) < nblk; ++r) {
            int p = block_of(r) * 64 + lane;
            const bool act = p < nr;
            if (!act) p = nr - 1;
            const FastRec rr = nxt;
            const uint32_t ei = (uint32_t)(p < neff_rec ? p + 1 : 0) * 6u;
            const PJ_GLOBAL uint4* const eq = (const PJ_GLOBAL uint4*)gm->eff;
            const uint32_t cm = __builtin_amdgcn_readfirstlane(rr.chunk);
            const uint32_t w = rr.info;
            const int kind = w & 7;
            const bool rev = w & GI_REV;
            double lnA = rr.lnA, bexp = rr.b, th = rr.theta;
            if (arr) {
                const int o = gm->orig[p];
                lnA = arr[o];
                bexp = arr[nr + o];
                th = arr[2 * nr + o];
            }
            // PLAIN: every reaction of the chunk is elementary (c = 1)
            auto react = [&](auto plain) {
            constexpr bool PLAIN = decltype(plain)::value;
            // (written as multiply-adds: th invT has other uses, and a rounding of
            // its own would show in k_f)
            V lnkf;
#pragma unroll
            for (int v = 0; v < RN; ++v) lnkf[v] = fma(-th, invT[v], fma(bexp, lnT[v], lnA));
            V dlkt_dT = 0.0, dlkt_dP = 0.0;
            if (EXT && !PLAIN && (cm & CHUNK_TAB) && kind_table(kind)) {
                DevMech td{};
                td.tab = gm->tab;
                td.tabd = gm->tabd;
#pragma unroll
                for (int v = 0; v < RN; ++v) {
                    double a, b;
                    lnkf[v] += table_lnk(td, kind, rr.tab, T[v], invT[v], lnT[v], K(SC_P)[v], a, b);
                    dlkt_dT[v] = a;
                    dlkt_dP[v] = b;
                }
            }
            // slots: concentration products, ratio kr / kf, dH
            V Pf = 1.0, Pb = 1.0, kq = 1.0, dH = 0.0, Pft = 1.0, Pbt = 1.0, lam = 0.0, dcp = 0.0, dvv = 0.0;
            // the product of the exponentials is precise: every step normal (tested always:
            // a branch round the test costs more)
            bool fits[RN];
#pragma unroll
            for (int v = 0; v < RN; ++v) fits[v] = true;
            {
                V xs[NSLOT][3];
#pragma unroll
                for (int a = 0; a < NSLOT; ++a) {
                    xs[a][0] = xs[a][1] = 1.0;
                    xs[a][2] = 0.0;
                    if ((cm >> a) & 1) {
                        const int k = rr.sp[a];
                        xs[a][0] = SP(k, A_C);
                        xs[a][1] = SP(k, a < MAXSIDE ? A_I : A_E);
                        if (DER) xs[a][2] = SP(k, A_H);
                    }
                }
                PJ_READS_FIRST();
                Pf = xs[0][0] * xs[1][0] * xs[2][0];
                Pb = xs[3][0] * xs[4][0] * xs[5][0];
                const V k0 = xs[0][1] * xs[3][1], k1 = xs[1][1] * xs[4][1], k2 = xs[2][1] * xs[5][1], k01 = k0 * k1;
                kq = k01 * k2 * vec(PW, (w >> 8) & 7);
#pragma unroll
                    for (int v = 0; v < RN; ++v)
                        fits[v] = normal(k01[v]) && normal((k01 * k2)[v]) && normal(kq[v]);
                if (DER) dH = ((xs[3][2] - xs[0][2]) + (xs[4][2] - xs[1][2])) + (xs[5][2] - xs[2][2]);
                if (DER && tiny) {
                    // absent species at 1e-150
                    Pft = vclamp(xs[0][0]) * vclamp(xs[1][0]) * vclamp(xs[2][0]);
                    Pbt = vclamp(xs[3][0]) * vclamp(xs[4][0]) * vclamp(xs[5][0]);
                }
            }
            if constexpr (ADJ) {
                // read after the products are formed: the registers of both
                // sets at once would spill
                PJ_READS_FIRST();
                V xa[NSLOT][3];
#pragma unroll
                for (int a = 0; a < NSLOT; ++a) {
                    xa[a][0] = xa[a][1] = xa[a][2] = 0.0;
                    if ((cm >> a) & 1) {
                        const int k = rr.sp[a];
                        xa[a][0] = SP(k, A_Y);
                        xa[a][1] = SP(k, A_CP);
                        if (FORM == PJ_CONP) xa[a][2] = SP(k, A_VV);
                    }
                }
                PJ_READS_FIRST();
                auto delta = [&](int f) { return ((xa[3][f] - xa[0][f]) + (xa[4][f] - xa[1][f])) + (xa[5][f] - xa[2][f]); };
                lam = delta(0);
                dcp = delta(1);
                if (FORM == PJ_CONP) dvv = delta(2);
            }
            const double dnu = (double)((int)((w >> 8) & 7) - 3);
            const V kf = vexp(lnkf);
            V kr = kf * kq;
            bool bad[RN], some = false;
#pragma unroll
            for (int v = 0; v < RN; ++v) {
                bad[v] = rev && (!fits[v] || far(v) || !(fabs(lnkf[v]) < LNK_FAR));
                some |= bad[v];
            }
            if (__builtin_expect(__any(some), false)) {
#pragma unroll
                for (int v = 0; v < RN; ++v) {
                    double x = lnkf[v], m = vec(PW, (w >> 8) & 7)[v];
                    int e = 0;
                    if (far(v)) {
                        x -= dnu * log(PREF / (RU * K(SC_T)[v]));
                        m = 1.0;
                    }
#pragma unroll
                    for (int a = 0; a < NSLOT; ++a)
                        if ((cm >> a) & 1) {
                            if (far(v)) {
                                const double g = SP(rr.sp[a], A_E)[v];
                                x += a < MAXSIDE ? -g : g;
                            } else {
                                const double y = SP(rr.sp[a], a < MAXSIDE ? A_I : A_E)[v];
                                m *= __builtin_amdgcn_frexp_mant(y);
                                e += __builtin_amdgcn_frexp_exp(y);
                            }
                        }
                    x = scaled_exp(x, m, e);
                    kr[v] = bad[v] ? x : kr[v];
                }
            }
            if (!rev) kr = 0.0;
            const V Rf = kf * Pf;
            const V Rr = kr * Pb;
            const V R = Rf - Rr;

            const int neffc = PLAIN ? 0 : (cm >> 8) & 0xF;
            V Meff = 0.0;   // sum_k (alpha_k - 1) [C]_k
            if (!PLAIN && neffc) {
                const uint4 es4 = at4(eq, ei);
                const uint32_t es[4] = {es4.x, es4.y, es4.z, es4.w};
#pragma unroll
                for (int h = 0; h < MAXEFF / 2; ++h)
                    if (2 * h < neffc) {
                        const uint4 u = at4(eq, ei + 1 + h);
                        Meff += __hiloint2double(u.y, u.x) * SP(es[h] & 0xFFFF, A_C);
                        if (2 * h + 1 < neffc) Meff += __hiloint2double(u.w, u.z) * SP(es[h] >> 16, A_C);
                    }
            }
            // pressure modification
            V c = 1.0, dcdM = 0.0, dcdT = 0.0, Pr_dcdPr = 0.0, qA = 1.0;
            if (!PLAIN && kind == K_THREEBODY) {
                c = Ctot + Meff;
                dcdM = 1.0;
            } else if (!PLAIN && kind_falloff(kind)) {
                const V M = Ctot + Meff;
                FallRec fr_;
                {
                    union {
                        FallRec f;
                        uint4 v[4];
                    } u;
                    const PJ_GLOBAL uint4* q = (const PJ_GLOBAL uint4*)gm->fall;
#pragma unroll
                    for (int k = 0; k < 4; ++k) u.v[k] = at4(q, (uint32_t)p * 4u + k);
                    fr_ = u.f;
                }
                falloff<EXT, MODE>(fr_, kind, cm, (w & GI_CHEMACT) != 0, T, invT, lnT, lnkf, bexp, th, M, c, dcdM, dcdT, Pr_dcdPr, qA);
            }
            const V q = PLAIN ? R : c * R;
            if constexpr (!DER) {
                if (act) PO(p) = q;
            } else {
                const V invV = K(SC_INVV);
                const V dlnkf = (bexp + th * invT) * invT + dlkt_dT;
                const V dlnkr = dlnkf - (dH - dnu) * invT;
                V Fw = PLAIN ? Rf : c * Rf, Bk = PLAIN ? Rr : c * Rr;
                const V QM = PLAIN ? V(0.0) : R * dcdM;
                const V qT = PLAIN ? Rf * dlnkf - Rr * dlnkr : c * (Rf * dlnkf - Rr * dlnkr) + R * dcdT;
                // sum_j Q_j C_j: each one-way rate times its molecularity
                V sQC = (double)((w >> 12) & 3) * Fw - (double)((w >> 14) & 3) * Bk;
                if (!PLAIN) sQC += QM * Meff;
                if (tiny) {
                    Fw = PLAIN ? kf * Pft : c * (kf * Pft);
                    Bk = PLAIN ? kr * Pbt : c * (kr * Pbt);
                }
                V Qb = 0.0;
                if (w & GI_BATH) {
                    const uint4 u = PLAIN ? make_uint4(0, 0, 0, 0) : at4(eq, ei + 5);
#pragma unroll
                    for (int a = 0; a < MAXSIDE; ++a) {
                        if ((w >> (16 + a)) & 1) Qb += Fw;
                        if ((w >> (19 + a)) & 1) Qb -= Bk;
                    }
                    Qb = Qb * K(SC_ICB) + QM * __hiloint2double(u.y, u.x);
                    sQC -= Qb * K(SC_CB);
                }
                const V Qc = PLAIN ? Qb : Qb + QM;
                const V dqdT = qT - Ctot * invT * Qc;
                const V dqdS = FORM == PJ_CONP ? -(sQC - Qb * (K(SC_NSUM) * invV)) * invV
                                               : Qc * K(SC_INVRT) + q * dlkt_dP;
                const V dE = FORM == PJ_CONP ? dH : dH - dnu;
                if constexpr (JAC) {
#pragma unroll
                    for (int k = 0; k < RB; ++k)
                        if (r == k) {
                            hq[k] = q;
                            he[k] = dE;
                        }
                    if (act) {
                        PO(p) = Fw;
                        if (rev) PO(rr.bpos) = Bk;
                        PO(b3 + 2 * p) = dqdT;
                        PO(b3 + 2 * p + 1) = dqdS;
                        if ((w & GI_BATH) && !gm->approx) PO(rr.qbpos) = Qb;
                        s0 += dE * dqdT;
                        s1 += dE * dqdS;
                        s2 += rr.domega * dqdT;
                        s3 += rr.domega * dqdS;
                    }
                } else if (act) {
                    PO(p) = lam * Fw;
                    if (rev) PO(rr.bpos) = lam * Bk;
                    s0 += lam * dqdT;
                    s1 += lam * dqdS;
                    if (w & GI_BATH) s2 += lam * Qb;
                    s3 += q * dE;
                    s4 += rr.domega * q;
                    s5 += q * dcp;
                    if (FORM == PJ_CONP) s6 += q * dvv;
                    if (GR) {
                        // (this lane's own element: added to without atomics)
                        const double g = (PLAIN ? lam * q : lam * (q * qA - R * Pr_dcdPr))[0];
                        GR[p] += g;
                        GR[nr + p] += g * lnT[0];
                        GR[2 * nr + p] -= g * invT[0];
                    }
                }
                const V QMl = ADJ ? lam * QM : QM;
                if (!PLAIN && neffc) {
                    // third-body terms Q_M (alpha_k - 1) C_k, the record read again (cache hit)
                    const int neff = act ? (int)((w >> 24) & 0xF) : 0;
                    const uint4 es4 = at4(eq, ei);
                    const uint32_t es[4] = {es4.x, es4.y, es4.z, es4.w};
#pragma unroll
                    for (int h = 0; h < MAXEFF / 2; ++h)
                        if (2 * h < neffc) {
                            const uint4 u = at4(eq, ei + 1 + h);
                            if (2 * h < neff)
                                PO(rr.tpos + 2 * h) = QMl * __hiloint2double(u.y, u.x) * vclamp(SP(es[h] & 0xFFFF, A_C));
                            if (2 * h + 1 < neff)
                                PO(rr.tpos + 2 * h + 1) = QMl * __hiloint2double(u.w, u.z) * vclamp(SP(es[h] >> 16, A_C));
                        }
                }
            }
            };
            if (!(cm & CHUNK_PRESSURE)) react(std::true_type());
            else react(std::false_type());
            if (block_of(r + 1) < nblk) nxt = rec_at(gm, block_of(r + 1));
        }
        if constexpr (DER) {
            V sums[7] = {s0, s1, s2, s3, s4, s5, s6};
#pragma unroll
            for (int c = 0; c < NRS; ++c) {
                sums[c] = vmap(sums[c], [](double y) { return wave_total(y); });
                if (lane == 0) vec(RS, NRS * rwave + c) = sums[c];
            }
        }
    }

    // ---- (3) sums over reactions.  A task is a group of lists; tasks go to
    // the waves in turn, a task's lists loaded while the one before is summed.
    struct Task {
        uint4 h, x;
        uint2 d;
    };
    typedef const __attribute__((address_space(4))) SumLists SumListsRef;
    auto list_at = [&](SumListsRef& l, int g) {
        Task k;
        k.h = at4(l.head, (uint32_t)(g * 64 + lane));
        k.x = at4(l.ext, (uint32_t)(g * 64 + lane));
        k.d = uniform_load(l.desc, g);
        return k;
    };
    auto no_task = []() {
        Task k;
        k.h = make_uint4(0xFFFFFFFFu, 0, 0, 0);
        k.x = make_uint4(0, 0, 0, 0);
        k.d = make_uint2(0, 0);
        return k;
    };
    // (a task's descriptor is the wave's: told to the compiler, which has it in
    // vector registers once it has been through the loop)
    auto desc_x = [](const Task& k) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)k.d.x); };
    auto desc_y = [](const Task& k) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)k.d.y); };
    auto task_of = [&](const Task& k, int& most, int& nm, bool& first, int& lp, int& what) {
        most = (int)(desc_x(k) & 0xFF);
        nm = (int)(desc_x(k) >> 8);
        // the first lane of a sum names it; the others hold all ones, which as
        // a number of lanes lets every level add: they are not read
        first = k.h.x != 0xFFFFFFFFu;
        lp = (int)(k.h.x >> 28);
        what = (int)(k.h.x & 0x0FFFFFFFu);
    };
    // sums of the species' reactions: f(reaction, sign) per contribution, four
    // contributions at a time
    auto species_sum = [&](SumListsRef& l, const Task& k, int nm, auto read, auto add) {
        auto words = [&](uint32_t a, uint32_t b) {
            const uint32_t x[2] = {a, b};
            decltype(read(0)) v[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = read((int)((c & 1 ? x[c / 2] >> 16 : x[c / 2]) & 0x7FFF));
            PJ_READS_FIRST();
#pragma unroll
            for (int c = 0; c < 4; ++c) add(c & 1 ? sign31(x[c / 2]) : sign15(x[c / 2]), v[c]);
        };
        const uint32_t none = (uint32_t)nr | (uint32_t)nr << 16;
        words(k.h.y, k.h.z);
        words(k.h.w, k.x.x);
        words(k.x.y, k.x.z);
        words(k.x.w, none);
        for (int c = 0; c < nm; ++c) {
            const uint4 y = at4(l.more, (desc_y(k) + c) * 64 + lane);
            words(y.x, y.y);
            words(y.z, y.w);
        }
    };
    if constexpr (ADJ) {
        // columns: sum over the reactions that depend on species j, over [C]_j
        const GatherPtr gm = fresh(gmp);
        const int ntask = gm->cl.n;
        auto load = [&](int t) { return t < ntask ? list_at(gm->cl, t) : no_task(); };
        Task nx = load(wave);
        __syncthreads();
        if (wave == nwave - 1) {
            V t[NRS];
#pragma unroll
            for (int c = 0; c < NRS; ++c) {
                t[c] = 0.0;
                for (int w = 0; w < rnw; ++w) t[c] += vec(RS, NRS * w + c);
            }
            const V T = K(SC_T), Vv = K(SC_V), P = K(SC_P), iT = K(SC_INVT), iV = K(SC_INVV), ct = K(SC_CTOT), Dp = K(SC_DP);
            const V kap = K(SC_KAP), vS = K(SC_VS), cpb = SP(bath, A_CP);
            const V Tdot = -T * t[3] / Dp, Om = t[4];
            const V dDdT = K(SC_DDP) - cpb * ct * iT;
            const V dDdS = FORM == PJ_CONP ? -((Dp - cpb * K(SC_CB)) - cpb * (K(SC_NSUM) * iV)) * iV : cpb / (RU * T);
            const V X = FORM == PJ_CONP ? Vv : P;
            const V jT = t[0] + kap * (t[5] + Tdot * dDdT) +
                         vS * ((FORM == PJ_CONP ? Vv * (RU / P) * Om : RU * Om) - X * Tdot * iT * iT);
            V jS = t[1] + kap * Tdot * dDdS + vS * Tdot * iT;
            if (FORM == PJ_CONP) jS += vS * (RU * T / P) * Om + t[6];
            if (lane == 0) {
                vec(SC, SC_TT) = jT;
                vec(SC, SC_TS) = jS;
                vec(SC, SC_LB) = gm->approx ? V(0.0) : t[2];
                vec(SC, SC_KAP) = kap * Tdot * iV;
                vec(SC, SC_CB) = gm->approx ? V(0.0) : cpb;
            }
        }
        for (int t = wave; t < ntask; t += nwave) {
            const Task k = nx;
            nx = load(t + nwave);
            int most, nm, lp, what;
            bool first;
            task_of(k, most, nm, first, lp, what);
            V w0 = 0.0;
            auto words = [&](const uint32_t* x, auto nw) {
                constexpr int NW = decltype(nw)::value;
                V v[NW];
#pragma unroll
                for (int c = 0; c < NW; ++c) v[c] = PO((int)((x[c] & 0xFFF8) >> 3));
                PJ_READS_FIRST();
#pragma unroll
                for (int c = 0; c < NW; ++c) w0 += sign0(x[c]) * v[c];
            };
            const uint32_t hw[7] = {k.h.y, k.h.z, k.h.w, k.x.x, k.x.y, k.x.z, k.x.w};
            words(hw, std::integral_constant<int, 7>());
            for (int c = 0; c < nm; ++c) {
                const uint4 y = at4(gm->cl.more, (desc_y(k) + c) * 64 + lane);
                const uint32_t x[4] = {y.x, y.y, y.z, y.w};
                words(x, std::integral_constant<int, 4>());
            }
            w0 = vmap(w0, [&](double y) { return fold(y, most, lp); });
            if (first) SP(what, A_E) = w0 / vclamp(SP(what, A_C));
        }
        __syncthreads();
        const double lb = SC[SC_LB], kt = SC[SC_KAP], cpb = SC[SC_CB], iV = SC[SC_INVV];
        for (int i = tid; i < N; i += nthr) {
            const double y = i == 0 ? SC[SC_TT] : i == 1 ? SC[SC_TS] : iV * (A[fld(i - 2, A_E)] - lb) + kt * (A[fld(i - 2, A_CP)] - cpb);
            if (layout == PJ_LAYOUT_F) jac[(long)i * n + qg] = y;
            else jac[qg * (long)N + i] = y;
        }
        return;
    }
    if constexpr (JAC) {
        // (3a) T and V/P columns of the species rows; bath-gas partials
        const GatherPtr gm = fresh(gmp);
        const int nsl = gm->sl.n, ntask = nsl + gm->bl.n, b3 = gm->b3;
        auto load = [&](int t) { return t < nsl ? list_at(gm->sl, t) : t < ntask ? list_at(gm->bl, t - nsl) : no_task(); };
        Task nx = load(wave);
        __syncthreads();
        for (int t = wave; t < ntask; t += nwave) {
            const Task k = nx;
            nx = load(t + nwave);
            int most, nm, lp, what;
            bool first;
            task_of(k, most, nm, first, lp, what);
            auto folded = [&](const V& x) { return vmap(x, [&](double y) { return fold(y, most, lp); }); };
            if (t < nsl) {
                typedef double V2 __attribute__((ext_vector_type(2 * NV)));
                V2 w = 0.0;
                species_sum(gm->sl, k, nm, [&](int p) { return *reinterpret_cast<const V2*>(pool + (b3 + 2 * p) * NV); },
                            [&](double sg, const V2& v) { w += sg * v; });
                V w1, w2;
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    w1[v] = w[v];
                    w2[v] = w[NV + v];
                }
                w1 = folded(w1);
                w2 = folded(w2);
                if (first) {
                    SP(what, A_VT) = w1;
                    vec(VS, what) = w2;
                }
            } else {
                V w0 = 0.0;
                auto two = [&](uint32_t x) {
                    const V a = PO((int)((x & 0xFFF8) >> 3)), b = PO((int)((x >> 19) & 0x1FFF));
                    w0 += sign0(x) * a;
                    w0 += sign16(x) * b;
                };
                auto four = [&](const uint4& y) { two(y.x), two(y.y), two(y.z), two(y.w); };
                two(k.h.y), two(k.h.z), two(k.h.w);
                four(k.x);
                for (int c = 0; c < nm; ++c) four(at4(gm->bl.more, (desc_y(k) + c) * 64 + lane));
                w0 = folded(w0);
                if (first) vec(BB, 1 + what) = w0;
            }
        }
    }
    {
        // (3b) production rates; the columns' energy- and mole-weighted sums, 1/C
        const GatherPtr gm = fresh(gmp);
        const int nsl = gm->sl.n, ntask = nsl + (JAC ? gm->cl.n : 0), b3 = JAC ? gm->b3 : 0;
        auto load = [&](int t) {
            return t < nsl ? list_at(gm->sl, t) : JAC && t < ntask ? list_at(gm->cl, t - nsl) : no_task();
        };
        Task nx = load(wave);
        __syncthreads();
        if (JAC) {
#pragma unroll
            for (int k = 0; k < RB; ++k) {
                const int p = block_of(k) * 64 + lane;
                if (p < nr) {
                    rvec(pool, b3 + p) = hq[k];
                    rvec(pool, b3 + nr + 1 + p) = he[k];
                }
            }
            if (tid < NV) pool[(b3 + nr) * NV + tid] = 0.0;
            __syncthreads();
        }
        for (int t = wave; t < ntask; t += nwave) {
            const Task k = nx;
            nx = load(t + nwave);
            int most, nm, lp, what;
            bool first;
            task_of(k, most, nm, first, lp, what);
            auto folded = [&](const V& x) { return vmap(x, [&](double y) { return fold(y, most, lp); }); };
            if (t < nsl) {
                V w0 = 0.0;
                species_sum(gm->sl, k, nm, [&](int p) { return PO(b3 + p); }, [&](double sg, const V& v) { w0 += sg * v; });
                w0 = folded(w0);
                if (first) SP(what, A_W) = w0;
            } else if (JAC) {
                V w0 = 0.0, w1 = 0.0;
                auto words = [&](const uint32_t* x, auto nw) {
                    constexpr int NW = decltype(nw)::value;
                    V v[NW][2];
#pragma unroll
                    for (int c = 0; c < NW; ++c) {
                        v[c][0] = PO((int)((x[c] & 0xFFF8) >> 3));
                        v[c][1] = PO(b3 + nr + 1 + (int)((x[c] >> 16) & 0x1FFF));
                    }
                    PJ_READS_FIRST();
#pragma unroll
                    for (int c = 0; c < NW; ++c) {
                        const V q = sign0(x[c]) * v[c][0];
                        w0 += v[c][1] * q;
                        w1 += (double)((int)x[c] >> 29) * q;     // dOmega
                    }
                };
                const uint32_t hw[7] = {k.h.y, k.h.z, k.h.w, k.x.x, k.x.y, k.x.z, k.x.w};
                words(hw, std::integral_constant<int, 7>());
                auto four = [&](const uint4& y) {
                    const uint32_t x[4] = {y.x, y.y, y.z, y.w};
                    words(x, std::integral_constant<int, 4>());
                };
                for (int c = 0; c < nm; ++c) four(at4(gm->cl.more, (desc_y(k) + c) * 64 + lane));
                w0 = folded(w0);
                w1 = folded(w1);
                if (first) {
                    const V ic = 1.0 / vclamp(SP(what, A_C));
                    SP(what, A_IC) = ic;
                    vec(TQ, what) = w0 * ic;
                    vec(SQ, what) = w1 * ic;
                }
            }
        }
    }

    // the first Jacobian lists are on their way before the barrier
    Task hv = no_task();
    if (JAC) {
        const GatherPtr gm = fresh(gmp);
        const JacRound R = uniform_load(gm->rounds, 0);
        if (R.heavy0 + wave < R.heavy1) hv = list_at(gm->jh, R.heavy0 + wave);
    }
    __syncthreads();

    // ---- source terms (one wave; the others begin with the Jacobian entries)
    if (wave == nwave - 1) {
        const GatherPtr gm = fresh(gmp);
        V np = 0.0, om = 0.0, scw = 0.0;
        for (int k = lane; k < ns; k += 64) {
            const V wk = SP(k, A_W), h = SP(k, A_H);
            np += (FORM == PJ_CONP ? h : h - 1.0) * wk;
            om += at(gm->wfac, (uint32_t)k) * wk;
            if (JAC) scw += SP(k, A_CP) * wk;
        }
        auto all = [&](const V& x) { return vmap(x, [](double y) { return wave_total(y); }); };
        np = all(np);
        om = all(om);
        if (JAC) scw = all(scw);
        const V T = K(SC_T), Vv = K(SC_V), P = K(SC_P), invT = K(SC_INVT);
        const V Tdot = -T * np / K(SC_DP);
        if (lane == 0) {
            vec(SC, SC_TDOT) = Tdot;
            vec(SC, SC_SDOT) = FORM == PJ_CONP ? Vv * Tdot * invT + Vv * RU * T * om / P : P * Tdot * invT + RU * T * om;
            if (JAC) {
                vec(SC, SC_OM) = om;
                vec(SC, SC_SCW) = scw;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    V t = 0.0;
                    for (int w = 0; w < rnw; ++w) t += vec(RS, NRS * w + c);
                    vec(SC, SC_TT + c) = t;
                }
            }
        }
    }
    // output: thread t writes for state s2; in layout C whole states (threads
    // of one state take consecutive values), in layout F the states of a value
    const int G = nthr / NV;
    const int s2 = NV == 1 ? 0 : layout == PJ_LAYOUT_F ? tid % NV : tid / G;
    const int g2 = NV == 1 ? tid : layout == PJ_LAYOUT_F ? tid / NV : tid - s2 * G;
    const long st2 = qg * NV + s2;
    auto C_ = [&](int q) { return SC[q * NV + s2]; };
    auto write_source = [&]() {
        if (!dstate || st2 >= n) return;
        const double V2 = C_(SC_V);
        for (int i = g2; i < N; i += G) {
            const double v = i < 2 ? C_(i == 0 ? SC_TDOT : SC_SDOT) : V2 * A[fld(i - 2, A_W) * NV + s2];
            if (layout == PJ_LAYOUT_F) dstate[(long)i * n + st2] = v;
            else dstate[st2 * (long)N + i] = v;
        }
    };
    if constexpr (!JAC) {
        __syncthreads();
        write_source();
        return;
    } else {
    double* const buf = pool + gmp->b3 * NV;
    const int n_rounds = gmp->n_rounds;
    for (int rd = 0; rd < n_rounds; ++rd) {
        const GatherPtr gm = fresh(gmp);
        const JacRound R = uniform_load(gm->rounds, rd);
        const int row0 = R.row0, row1 = R.row1, e0 = R.e0, ne = R.ne;
        // ---- (4) entries of the species rows: 1/C_j sum - bath partial
        auto val = [&](uint32_t off) -> V { return *(const LV*)(off * NV); };
        const int dsh = gm->dshift;
        const uint32_t cmask = (1u << (dsh - 16)) - 1;
        auto inv_c = [&](uint32_t e) { return SP((int)((e >> 16) & cmask), A_IC); };
        auto bath_of = [&](uint32_t e) { return vec(BB, (int)(e >> dsh)); };
        constexpr int UM = 2, UL = 2;
        const uint4 nothing = make_uint4(0xFFFFu, 0, 0xFFFFu, 0);
        uint4 md[UM], lt[UL];
        int tm = R.mid0 + wave, tl = R.light0 + wave;
#pragma unroll
        for (int u = 0; u < UM; ++u) md[u] = tm + u * nwave < R.mid1 ? at4(gm->jm, (uint32_t)((tm + u * nwave) * 64 + lane)) : nothing;
        for (int t = R.heavy0 + wave; t < R.heavy1; t += nwave) {
            const Task k = hv;
            if (t + nwave < R.heavy1) hv = list_at(gm->jh, t + nwave);
            const int most = (int)(desc_x(k) & 0xFF), nm = (int)(desc_x(k) >> 8);
            const int lp = (int)((k.h.y >> 1 & 3) | (k.h.y >> 15 & 4));
            V w0 = 0.0, w1 = 0.0;
            auto words = [&](const uint32_t* x, auto nw) {
                constexpr int NW = decltype(nw)::value;
                V v[2 * NW];
#pragma unroll
                for (int c = 0; c < NW; ++c) {
                    const uint32_t m = x[c] & 0xFFF8FFF8u;
                    v[2 * c] = val(m & 0xFFFF);
                    v[2 * c + 1] = val(m >> 16);
                }
                PJ_READS_FIRST();
#pragma unroll
                for (int c = 0; c < NW; ++c) {
                    w0 += sign0(x[c]) * v[2 * c];
                    w1 += sign16(x[c]) * v[2 * c + 1];
                }
            };
            const uint32_t x[7] = {k.h.y, k.h.z, k.h.w, k.x.x, k.x.y, k.x.z, k.x.w};
            words(x, std::integral_constant<int, 7>());
            for (int c = 0; c < nm; ++c) {
                const uint4 y = at4(gm->jh.more, (desc_y(k) + c) * 64 + lane);
                const uint32_t z[4] = {y.x, y.y, y.z, y.w};
                words(z, std::integral_constant<int, 4>());
            }
            w0 += w1;
            w0 = vmap(w0, [&](double y) { return fold(y, most, lp); });
            if (k.h.x != 0xFFFFFFFFu)
                vec(buf, (int)(k.h.x & 0xFFFF)) = w0 * inv_c(k.h.x) - bath_of(k.h.x);
        }
#pragma unroll
        for (int u = 0; u < UL; ++u) lt[u] = tl + u * nwave < R.light1 ? at4(gm->jl, (uint32_t)((tl + u * nwave) * 64 + lane)) : nothing;
        for (; tm < R.mid1; tm += UM * nwave) {
#pragma unroll
            for (int u = 0; u < UM; ++u) {
                if (tm + u * nwave >= R.mid1) break;
                const uint4 h = md[u];
                const int t2 = tm + (UM + u) * nwave;
                if (t2 < R.mid1) md[u] = at4(gm->jm, (uint32_t)(t2 * 64 + lane));
                const uint32_t x[3] = {h.y, h.z, h.w};
                V v[6];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const uint32_t m = x[c] & 0xFFF8FFF8u;
                    v[2 * c] = val(m & 0xFFFF);
                    v[2 * c + 1] = val(m >> 16);
                }
                const V ic = inv_c(h.x), bb = bath_of(h.x);
                PJ_READS_FIRST();
                V w0 = 0.0, w1 = 0.0;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    w0 += sign0(x[c]) * v[2 * c];
                    w1 += sign16(x[c]) * v[2 * c + 1];
                }
                if ((h.x & 0xFFFF) != 0xFFFF) vec(buf, (int)(h.x & 0xFFFF)) = (w0 + w1) * ic - bb;
            }
        }
        for (; tl < R.light1; tl += UL * nwave) {
#pragma unroll
            for (int u = 0; u < UL; ++u) {
                if (tl + u * nwave >= R.light1) break;
                const uint4 h = lt[u];
                const int t2 = tl + (UL + u) * nwave;
                if (t2 < R.light1) lt[u] = at4(gm->jl, (uint32_t)(t2 * 64 + lane));
                const uint32_t x[2] = {h.y, h.w}, e[2] = {h.x, h.z};
                V v[4], ic[2], bb[2];
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const uint32_t m = x[c] & 0xFFF8FFF8u;
                    v[2 * c] = val(m & 0xFFFF);
                    v[2 * c + 1] = val(m >> 16);
                    ic[c] = inv_c(e[c]);
                    bb[c] = bath_of(e[c]);
                }
                PJ_READS_FIRST();
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const V w = sign0(x[c]) * v[2 * c] + sign16(x[c]) * v[2 * c + 1];
                    if ((e[c] & 0xFFFF) != 0xFFFF) vec(buf, (int)(e[c] & 0xFFFF)) = w * ic[c] - bb[c];
                }
            }
        }
        // the next round's first lists
        if (rd + 1 < n_rounds) {
            const JacRound Rn = uniform_load(gm->rounds, rd + 1);
            if (Rn.heavy0 + wave < Rn.heavy1) hv = list_at(gm->jh, Rn.heavy0 + wave);
        }
        // T and V/P columns of the species rows
        for (int k = row0 - 2 + tid; k < row1 - 2; k += nthr) {
            const int e = (int)at(gm->row_ptr, (uint32_t)(2 + k)) - e0;
            const V Vv = K(SC_V);
            vec(buf, e) = Vv * SP(k, A_VT);
            const V vs = Vv * vec(VS, k);
            vec(buf, e + 1) = FORM == PJ_CONP ? vs + SP(k, A_W) : vs;   // d(V wdot_k)/dV = wdot_k + V dwdot_k/dV
        }
        __syncthreads();
        // ---- (5) output
        const int nnz = gm->nnz;
        const long NN = (long)N * N;
        if (rd == 0) {
            write_source();
            if (st2 < n && g2 < N) {
                // T and V/P rows
                const double T2 = C_(SC_T), V2 = C_(SC_V), P2 = C_(SC_P);
                const double iT = C_(SC_INVT), iV = C_(SC_INVV), ct = C_(SC_CTOT);
                const double Dp = C_(SC_DP), Tdot = C_(SC_TDOT), Om = C_(SC_OM), Scw = C_(SC_SCW);
                const double cpb = A[fld(bath, A_CP) * NV + s2];
                const double dDdT = C_(SC_DDP) - cpb * ct * iT;
                const double dDdS = FORM == PJ_CONP ? -((Dp - cpb * C_(SC_CB)) - cpb * (C_(SC_NSUM) * iV)) * iV
                                                    : cpb / (RU * T2);
                const double RTP = RU * T2 / P2;
                const bool approx = gm->approx;
                const double tqb = approx ? 0.0 : TQ[bath * NV + s2], sqb = approx ? 0.0 : SQ[bath * NV + s2];
                const double cpb_n = approx ? 0.0 : cpb;
                for (int j = g2; j < N; j += G) {
                    double j0, j1;
                    if (j == 0) {
                        j0 = -(T2 * C_(SC_TT) + Scw + Tdot * dDdT) / Dp;
                        j1 = FORM == PJ_CONP
                                 ? V2 * iT * j0 - V2 * Tdot * iT * iT + V2 * (RU / P2) * Om + V2 * RTP * C_(SC_ST)
                                 : P2 * iT * j0 - P2 * Tdot * iT * iT + RU * Om + RU * T2 * C_(SC_ST);
                    } else if (j == 1) {
                        j0 = -(T2 * C_(SC_TS) + Tdot * dDdS) / Dp;
                        j1 = FORM == PJ_CONP ? Tdot * iT + V2 * iT * j0 + RTP * Om + V2 * RTP * C_(SC_SS)
                                             : Tdot * iT + P2 * iT * j0 + RU * T2 * C_(SC_SS);
                    } else {
                        const int k = (j - 2) * NV + s2;
                        j0 = -(T2 * (TQ[k] - tqb) + Tdot * (A[fld(j - 2, A_CP) * NV + s2] - cpb_n)) * iV / Dp;
                        j1 = FORM == PJ_CONP ? V2 * iT * j0 + RTP * (SQ[k] - sqb)
                                             : P2 * iT * j0 + RU * T2 * (SQ[k] - sqb) * iV;
                    }
                    if (dense) {
                        if (layout == PJ_LAYOUT_F) {
                            jac[st2 + n * ((long)N * j)] = j0;
                            jac[st2 + n * (1 + (long)N * j)] = j1;
                        } else {
                            jac[st2 * NN + j] = j0;
                            jac[st2 * NN + N + j] = j1;
                        }
                    } else {
                        const long o0 = gm->ccs_pos ? at(gm->ccs_pos, (uint32_t)j) : j;
                        const long o1 = gm->ccs_pos ? at(gm->ccs_pos, (uint32_t)(N + j)) : N + j;
                        if (layout == PJ_LAYOUT_F) {
                            jac[o0 * n + st2] = j0;
                            jac[o1 * n + st2] = j1;
                        } else {
                            jac[st2 * (long)nnz + o0] = j0;
                            jac[st2 * (long)nnz + o1] = j1;
                        }
                    }
                }
            }
        }
        if (st2 < n) {
            const double* bs = buf + s2;
            if (!dense) {
                if (gm->ccs_pos) {
                    double* out = layout == PJ_LAYOUT_F ? jac + st2 : jac + st2 * (long)nnz;
                    const long step = layout == PJ_LAYOUT_F ? n : 1;
                    for (int e = g2; e < ne; e += G) out[(long)at(gm->ccs_pos, (uint32_t)(e0 + e)) * step] = bs[e * NV];
                } else if (layout == PJ_LAYOUT_F) {
                    double* out = jac + st2 + (long)(e0 + g2) * n;
                    for (int e = g2; e < ne; e += G, out += (long)G * n) *out = bs[e * NV];
                } else {
                    double* out = jac + st2 * (long)nnz + e0;
#pragma unroll 4
                    for (int e = g2; e < ne; e += G) out[e] = bs[e * NV];
                }
            } else {
                // every entry of the round's rows through the (row, column) map,
                // several map reads in flight per lane
                constexpr int DU = 8;
                const int f1 = row1 * N;
                auto put = [&](int f, uint16_t e) {
                    const double v = e == NOSLOT ? 0.0 : bs[(e - e0) * NV];
                    if (layout == PJ_LAYOUT_F) {
                        const int i = f / N, j = f - i * N;
                        jac[st2 + n * (i + (long)N * j)] = v;
                    } else {
                        jac[st2 * NN + f] = v;
                    }
                };
                int f = row0 * N + g2;
                for (; f + (DU - 1) * G < f1; f += DU * G) {
                    uint16_t e[DU];
#pragma unroll
                    for (int u = 0; u < DU; ++u) e[u] = at(gm->dmap_rm, (uint32_t)(f + u * G));
#pragma unroll
                    for (int u = 0; u < DU; ++u) put(f + u * G, e[u]);
                }
                for (; f < f1; f += G) put(f, at(gm->dmap_rm, (uint32_t)f));
            }
        }
        if (rd + 1 < n_rounds) __syncthreads();
    }
    }
}

template <int FORM, int LAYOUT, int MODE, int NV, bool EXT>
__global__ void __launch_bounds__(MAX_THREADS) __attribute__((amdgpu_waves_per_eu(MODE == GM_SRC ? PJ_WPE_SRC : PJ_WPE_JAC)))
pj_gather_kernel(const GatherMech* const gmp, const long n, const long ngroups, const unsigned per,
                 const double* __restrict__ state, const double* __restrict__ param,
                 double* __restrict__ dstate, double* __restrict__ jac, const double* __restrict__ arr) {
    // workgroups are dealt to the 8 XCDs in turn: XCD x takes the contiguous
    // groups [x per, (x + 1) per), so that the partial cache lines of layout-F
    // arrays of neighbouring states meet in one L2
    const long qg = (long)(blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (qg >= ngroups) return;
    gather_group<FORM, LAYOUT, MODE, NV, EXT>((GatherPtr)gmp, n, state, param, dstate, jac, arr, qg);
}

// J^T v and the parameter sums, a state per workgroup.  With dE_i, dOmega_i and
// v known before the reactions, all that v^T J takes of reaction i is lambda_i
// grad q_i: the pool holds lambda_i F_i, lambda_i B_i and lambda_i T_ik, and a
// species column is one gathered sum, where the scatter kernels add every
// partial to three accumulators.  Persistent workgroups, which sum their
// states' parameter derivatives in LDS (each element has one lane) and add them
// to the output once.  111 species, 784 reactions, 65536 states: 1.47 ms
// against 1.80 (scatter, 4 states and 4 waves); 6,900 vector instructions a
// state, 52% of the issue slots at 12 waves a compute unit.  At 128 registers
// (16 waves) 66 spilled ones made it 2.46 ms.
template <int FORM, int LAYOUT, bool EXT>
__global__ void __launch_bounds__(MAX_THREADS) __attribute__((amdgpu_waves_per_eu(PJ_WPE_ADJ)))
pj_gather_adjoint(const GatherMech* const gmp, const long n, const int gr_offset,
                  const double* __restrict__ state, const double* __restrict__ param, const double* __restrict__ vin,
                  double* __restrict__ jtv, double* __restrict__ grad, const double* __restrict__ arr) {
    extern __shared__ double lds[];
    double* const GR = grad ? lds + gr_offset : nullptr;
    const int nr = gmp->nr;
    if (grad)
        for (int i = threadIdx.x; i < 3 * nr; i += blockDim.x) GR[i] = 0.0;
    __syncthreads();
    long q0, q1, qstep;
    group_range(n, q0, q1, qstep);
    for (long q = q0; q < q1; q += qstep) {
        gather_group<FORM, LAYOUT, GM_ADJ, 1, EXT>(fresh((GatherPtr)gmp), n, state, param, nullptr, jtv, arr, q, vin, GR);
        __syncthreads();
    }
    // (each workgroup from a place of its own, so that they don't meet at one
    // address)
    if (grad)
        for (int i = threadIdx.x; i < nr; i += blockDim.x) {
            int p = i + (int)(blockIdx.x * 61 % (unsigned)nr);
            if (p >= nr) p -= nr;
            const int o = gmp->orig[p];
            atomicAdd(&grad[o], GR[p]);
            atomicAdd(&grad[nr + o], GR[nr + p]);
            atomicAdd(&grad[2 * nr + o], GR[2 * nr + p]);
        }
}

template <int FORM, int LAYOUT, bool EXT>
static hipError_t launch_gather_adjoint_t(const GatherCall& c) {
    auto k = pj_gather_adjoint<FORM, LAYOUT, EXT>;
    const int64_t lds = gather_lds(*c.gm, GM_ADJ, 1), sums = 24 * (int64_t)c.gm->nr;
    if (lds > 65536) {
        static std::atomic<uint64_t> done{0};
        hipError_t e = allow_full_lds((const void*)k, done);
        if (e != hipSuccess) return e;
    }
    // as many workgroups as the chip holds at 4 * PJ_WPE_ADJ waves a compute unit
    const int64_t cap = 256 * std::max<int64_t>(1, 4 * PJ_WPE_ADJ / c.waves);
    int64_t grid = c.n < cap ? c.n : cap;
    if (grid >= 8) grid &= ~(int64_t)7;
    if (c.grad) {
        hipError_t e = zero_async(c.grad, 3 * (int64_t)c.gm->nr, c.stream);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(64 * c.waves), (size_t)lds, c.stream, c.d_gm, (long)c.n,
                       (int)((lds - sums) / 8), c.state, c.param, c.vin, c.jac, c.grad, c.arr);
    return hipGetLastError();
}

template <int FORM, int LAYOUT, int MODE, int NV, bool EXT>
static hipError_t launch_gather_t(const GatherCall& c) {
    auto k = pj_gather_kernel<FORM, LAYOUT, MODE, NV, EXT>;
    const int64_t lds = gather_lds(*c.gm, MODE, NV);
    if (lds > 65536) {
        static std::atomic<uint64_t> done{0};
        hipError_t e = allow_full_lds((const void*)k, done);
        if (e != hipSuccess) return e;
    }
    const int64_t groups = (c.n + NV - 1) / NV;
    const int64_t per = (groups + 7) / 8;
    if (per > (1 << 27)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, dim3((unsigned)(8 * per)), dim3(64 * c.waves), (size_t)lds, c.stream, c.d_gm, (long)c.n,
                       (long)groups, (unsigned)per, c.state, c.param, c.dstate, c.jac, c.arr);
    return hipGetLastError();
}

template <bool EXT>
hipError_t launch_gather_impl(const GatherCall& c) {
#define PJ_G(F, L, M, SS) \
    if (c.form == F && c.layout == L && c.gmode == M && c.S == SS) return launch_gather_t<F, L, M, SS, EXT>(c);
#define PJ_GA(F, L) \
    if (c.form == F && c.layout == L && c.gmode == GM_ADJ && c.S == 1) return launch_gather_adjoint_t<F, L, EXT>(c);
#define PJ_GS(F, L, M) PJ_G(F, L, M, 1) PJ_G(F, L, M, 2)
#define PJ_GL(F, L) PJ_GS(F, L, GM_SRC) PJ_GS(F, L, GM_JAC) PJ_GS(F, L, GM_DENSE) PJ_GA(F, L)
    PJ_GL(PJ_CONP, PJ_LAYOUT_C) PJ_GL(PJ_CONP, PJ_LAYOUT_F) PJ_GL(PJ_CONV, PJ_LAYOUT_C) PJ_GL(PJ_CONV, PJ_LAYOUT_F)
#undef PJ_GL
#undef PJ_GS
#undef PJ_G
#undef PJ_GA
    return hipErrorInvalidValue;
}

}  // namespace pj
