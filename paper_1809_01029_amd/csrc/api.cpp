// C-ABI entry points (declared in include/pjac.h): argument checking, launch
// shape, and dispatch to the kernels.  No call here synchronises the host
// except pj_mech_load, which uploads the tables.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <new>
#include <string>

#include "internal.h"

namespace {

thread_local std::string g_err;

pj_status fail(pj_status st, const std::string& msg) {
    g_err = msg;
    return st;
}

bool pow2_upto(int v, int mx) { return v >= 1 && v <= mx && (v & (v - 1)) == 0; }

constexpr int MAX_S = 64, MAX_WAVES = 8;

// The kernel that evaluates `mode` for a mechanism: the run-time slot search
// and the fixed-order additions have kernels of their own, and so has a call
// with its own Arrhenius parameters.
int kernel_mode(const pj::Mechanism& m, int mode, bool per_call_arrhenius) {
    if (per_call_arrhenius) return mode == pj::MODE_SRC ? pj::MODE_SRC_P : pj::MODE_ADJ_P;
    if (mode == pj::MODE_DENSE && m.dense_unroll == 16 && m.S[mode] <= 4) return pj::MODE_DENSE_U16;
    if (mode == pj::MODE_SPARSE && m.dm.lsearch) return pj::MODE_SPARSE_LS;
    if (m.dm.det && mode == pj::MODE_SRC) return pj::MODE_SRC_DET;
    if (m.dm.det && mode == pj::MODE_SPARSE) return pj::MODE_SPARSE_DET;
    return mode;
}

// the most states per workgroup a kernel mode is built for
int max_states(int kmode) {
    if (kmode == pj::MODE_SPARSE_LS || kmode == pj::MODE_SRC_DET || kmode == pj::MODE_SPARSE_DET) return 4;
    if (pj::base_mode(kmode) == pj::MODE_ADJ) return pj::MAX_S_ADJ;
    return MAX_S;
}

}  // namespace

namespace pj {

static int gather_mode(int mode) { return mode == MODE_SRC ? GM_SRC : mode == MODE_ADJ ? GM_ADJ : mode == MODE_DENSE ? GM_DENSE : GM_JAC; }

// A call with S states and w waves per workgroup runs on the gather kernels
// (gather_body.h) if they are built for it: at most two states (the adjoint
// one), each with a wave of its own or more, a wave's reactions in at most GATHER_BLOCKS blocks
// of 64 (adjoints in 2 GATHER_BLOCKS, source terms in 12: with more the scatter
// kernels are the faster; 360 species, 34 blocks, 6410 states, scatter -> gather, us:
// source terms 2x2 184 -> 285, 1x3 205 -> 180; adjoint 1x2 1090 -> 1370, 1x4
// 907 -> 803).  One wave per workgroup stays with the scatter kernels (their fixed
// order is documented), and so do the run-time slot search and the fixed-order
// option, whose results are theirs by definition.  A dense Jacobian in layout
// F is written by columns of single states at S = 1: 2993 us against the
// scatter kernels' 2760 for 2048 states of 360 species.  The grid's threads
// stay below 2^32.
static bool gather_takes(const Mechanism& m, int mode, pj_layout layout, int64_t n, int S, int w) {
    if (!m.gm.ok || m.dm.lsearch || m.dm.det) return false;
    if (S > (mode == MODE_ADJ ? 1 : 2) || w < 2 || w % S) return false;
    if (mode == MODE_DENSE && layout == PJ_LAYOUT_F && S == 1) return false;
    const int most = mode == MODE_SRC ? 12 * w : mode == MODE_ADJ ? 2 * GATHER_BLOCKS * w : GATHER_BLOCKS * (w / S);
    if ((m.nr + 63) / 64 > most) return false;
    if ((n / S + 8) * 64 * w >= (int64_t)1 << 32) return false;
    return gather_lds(m.gm, gather_mode(mode), S) <= m.lds_max;
}

// Source terms of 64 states per workgroup and at least 2 waves (pairs of them)
// run on the wide kernel (wide_body.h).
static bool wide_takes(const Mechanism& m, int mode, int S, int w) {
    return mode == MODE_SRC && m.gm.ok && !m.dm.det && S == 64 && w >= 2 && wide_fits(m.gm, w);
}

// The automatic choice of the wide kernel: two workgroups of 8 waves a compute
// unit (about 54 species; of 70, 131072 states 563 us against the gather kernels'
// 554), more than 8192 states.  A workgroup's time is nearly the same however many
// share its compute unit, so what counts is how full the last round of workgroups
// over the 256 compute units is: 53 species, 16390 states (1.002 rounds, two
// workgroups on some units) 94 us against 67 (gather), 26000 95 against 99, 33000
// 140 against 122, 40000 141 against 147, 65536 (four rounds) 179 against 237;
// 32 species (scatter) 24001 states 63 against 59, 26000 63 against 68, 36000
// 92 against 83, 40000 92 against 94.
static bool wide_choice(const Mechanism& m, int mode, int64_t n, int& S, int& w) {
    if (mode != MODE_SRC || n <= 8192 || !wide_takes(m, mode, 64, 4) || 2 * wide_lds(m.gm, 4) > m.lds_max) return false;
    const int blocks = (m.nr + 63) / 64;
    const int64_t round = 256 * 64, rounds = (n + round - 1) / round;
    const bool four = wide_takes(m, mode, 64, 2) && 4 * wide_lds(m.gm, 2) <= m.lds_max;     // of 4 waves
    // One round: the gather kernels up to 13000 states of more than 256 reactions,
    // the scatter kernels up to 12288 of 129 to 256 where their grid is a multiple of
    // 8 (only then do they map neighbouring workgroups to one XCD): 32 species, 12000
    // states 31 against 38 us, 36 species 38 against 40, but 12001 39 against 38 and
    // 47 against 40.
    if (rounds == 1 && blocks >= 3 && blocks <= 4 && n <= 12288 && (n + 3) / 4 % 8 == 0) return false;
    if (rounds == 1 ? blocks > 4 && n <= 13000 : rounds < 4 && blocks > 1 && 5 * n < 4 * rounds * round && !(rounds == 3 && four))
        return false;
    // while each workgroup has a compute unit of its own, many waves
    S = 64;
    w = rounds == 1 ? (blocks > 1 && wide_takes(m, mode, 64, 8) ? 8 : 4) : four ? 2 : 4;
    return true;
}

// The automatic choice between the gather and the scatter kernels for a call
// of n states, and the gather kernels' shape (false: scatter, in the shape of
// choose_launch, or wide).  Measured on MI355X over mechanisms of 13 to 360 species
// and 64 to 262144 states; scatter -> gather, us per call:
//   few states: a workgroup per state or two fills the chip sooner; 13 species,
//     1024 states, sparse 19.8 -> 14.5 (2048: 20.3 -> 18.8, 4096: 21.4 -> 35);
//     53 species, 100 states, source terms 57 -> 10, sparse 67 -> 16.5;
//     111 species, 4096 states, source terms 63 -> 35
//   more than 256 reactions, Jacobians: 53 species, 71199 states, sparse
//     1388 -> 1110, dense (17799) 408 -> 375; 111 species, 16232 states 752 -> 620;
//     360 species, 4096 states 767 -> 660 (F 1270 -> 848)
//   fewer: 20 species, 131072 states, sparse 996 -> 1159
static bool gather_choice(const Mechanism& m, int mode, pj_layout layout, int64_t n, bool grad, int& S, int& w) {
    const int blocks = (m.nr + 63) / 64;
    auto take = [&](int s, int v) {
        if (!gather_takes(m, mode, layout, n, s, v)) return false;
        S = s;
        w = v;
        return true;
    };
    if (mode == MODE_ADJ) {
        // Few states: a workgroup each (256: 53 species 51 -> 46, but 13 species 19.0
        // -> 21.1 and 220 species 70 -> 80).  Then the workgroups' additions of their
        // parameter sums to the output weigh (about 50 ps each, 256 of four
        // states send a quarter of them): 111 species, 1024 states 88 -> 120,
        // 4096 states 208 -> 178; 220 species (4 states a
        // workgroup), 512 states 86 -> 93, 1000 143 -> 114, 360 species (2) 256 86 -> 91, 512
        // 123 -> 111.
        // A wave holds 168 registers, a compute unit 12
        // waves: taken where the LDS lets in workgroups for all 12, or where a
        // state needs 8 waves (360 species, 8192 states 962 -> 640).  53 species,
        // 4096 states 161 -> 138 (4 waves; 2: 200), 16384 383 -> 297 (2: 303), without
        // a gradient 12000 143 -> 127 (2 waves; 4: 172),
        // 65536 1047 -> 779 (2 waves; 3: 849), 111 species, 54054 states
        // 1492 -> 1229 (4 waves; 3: 1744); 160 species, two workgroups:
        // 1319 -> 1654; 32 species, 208 reactions: 580 -> 651.
        if (n <= 128 || (n <= 256 && blocks > 1 && blocks <= 20)) return take(1, blocks <= 8 ? 4 : 8);
        if (blocks > 4 * GATHER_BLOCKS) return n >= 192 * m.auto_S[mode] && take(1, 8);
        if (n < 3072 || blocks <= 4) return false;
        const int v = grad && n < 16384 ? 4 : blocks <= 6 ? 2 : blocks <= 9 ? 3 : 4;
        return gather_lds(m.gm, GM_ADJ, 1) * (12 / v) <= m.lds_max && take(1, v);
    }
    if (mode == MODE_SRC) {
        // 20 species, 4096 states 19 -> 14, 8192 23 -> 27; 40 species, 6001 states
        // 49 -> 27, 8192 33 -> 34; 53 species, 12001 states 64 -> 51, 24001 93 -> 91;
        // 80 species, 262144 states 1410 -> 1220, 111 species 2430 -> 1723, 360
        // species, 65536 states 5413 -> 1563.  32 species, 20000 states: 52 -> 62.
        if (n <= 1024) return take(1, 4);
        int s, v;
        if (blocks < 2 || wide_choice(m, mode, n, s, v)) return false;
        if (n > 4096 && blocks <= 4) return false;
        return take(2, blocks <= 9 ? 2 : 4);
    }
    const bool few = n <= 2048;
    if (!few && blocks <= 4) return false;
    if (layout == PJ_LAYOUT_F) {
        // Two states write twice as long runs; one if two leave a compute unit a
        // single workgroup.  More waves for more reactions: 60 species, 24001 states,
        // sparse 543 -> 578 with 4, 499 with 8; 53 species 478 -> 441 with 4.
        // Where the rows of the output start a multiple of 4 kB apart, neighbouring
        // rows share a memory channel and short runs suffer (65536 states of 53
        // species 1200 -> 1545; 16384 of 80 species 571 -> 697, of 111 species
        // 839 -> 925; dense 8192 of 111 species 667 -> 793): large outputs stay with
        // the scatter kernels.
        if (n % 512 == 0) {
            if (mode == MODE_SPARSE && (n >= 16384 || n * blocks >= 90000)) return false;
            if (mode == MODE_DENSE && blocks <= 14 && (blocks >= 7 ? n * blocks >= 36000 : blocks == 6 && n >= 16384)) return false;
        }
        const int v = blocks <= 6 ? 4 : 8;
        if ((mode == MODE_DENSE || 2 * gather_lds(m.gm, GM_JAC, 2) <= m.lds_max) && take(2, v)) return true;
    } else if (blocks <= 6 && (!few || (n > 1536 && blocks >= 5 && (mode == MODE_SPARSE || blocks == 5)))) {
        // (40 species, 2048 states, sparse 37 -> 31, one state 40)
        if (take(2, 4)) return true;
    }
    return take(1, blocks <= 4 ? 2 : blocks <= 4 * GATHER_BLOCKS ? 4 : 8);
}

// the kernel set of a call of n states and its launch shape
Route route(const Mechanism& m, int mode, pj_layout layout, int64_t n, bool fused, bool grad) {
    int S = m.S[mode], w = m.waves[mode];
    bool automatic = m.automatic[mode];
    // A tuned shape is no measure for the other layout (111 species, 262144 states,
    // the gather kernels' shape of layout C in layout F: 18.7 ms, the automatic one
    // 13.1), except the wide kernel's, which stages either; nor is the gather
    // kernels' for a call that they don't take.
    if (m.tuned_layout[mode] >= 0) {
        if (m.tuned_kernel[mode] == KERNEL_WIDE && wide_takes(m, mode, S, w)) return {KERNEL_WIDE, S, w};
        if (m.tuned_layout[mode] == layout) {
            if (m.tuned_kernel[mode] == KERNEL_SCATTER) return {KERNEL_SCATTER, S, w};
            if (!fused && gather_takes(m, mode, layout, n, S, w)) return {KERNEL_GATHER, S, w};
        }
        automatic = true;
        S = m.auto_S[mode];
        w = m.auto_waves[mode];
    }
    int sS = S, sw = w;              // the scatter kernels' shape
    if (automatic && layout == PJ_LAYOUT_F) {
        if (n >= m.f_from[mode]) {
            sS = m.f_S[mode];
            sw = m.f_waves[mode];
        }
        // dense, a state per workgroup, rows a multiple of 4 kB apart: with 8 waves
        // they meet in the same channels (360 species, 1024 states 1143 us, 7 waves 773,
        // 2048 states 2788 and 2576; 1500 states 1259 and 1287)
        if (mode == MODE_DENSE && sS == 1 && sw == 8 && n % 512 == 0) sw = 7;
    }
    // (the adjoint with fused source terms: scatter kernels)
    if (!fused && (automatic ? gather_choice(m, mode, layout, n, grad, S, w) : gather_takes(m, mode, layout, n, S, w)))
        return {KERNEL_GATHER, S, w};
    if (automatic ? wide_choice(m, mode, n, S, w) : wide_takes(m, mode, S, w)) return {KERNEL_WIDE, S, w};
    return {KERNEL_SCATTER, sS, sw};
}

// the shape of a large call in layout C (as tuned, if it is)
static void nominal_shape(const Mechanism& m, int mode, int& S, int& w, int64_t& lds) {
    const pj_layout layout = m.tuned_layout[mode] >= 0 ? (pj_layout)m.tuned_layout[mode] : PJ_LAYOUT_C;
    const Route r = route(m, mode, layout, 1 << 20, false);
    S = r.kernel == KERNEL_SCATTER ? m.S[mode] : r.S;
    w = r.kernel == KERNEL_SCATTER ? m.waves[mode] : r.waves;
    lds = r.kernel == KERNEL_SCATTER ? m.lds[mode] : r.kernel == KERNEL_GATHER ? gather_lds(m.gm, gather_mode(mode), S) : wide_lds(m.gm, w);
}

// Waves per workgroup for S states per workgroup: enough that a compute unit
// holds about 8 resident waves given how many workgroups fit in its LDS, and
// at least S/64 so that every state has a lane.
static int default_waves(const Mechanism& m, int mode, int S, bool gr) {
    int w = S > 64 ? S / 64 : 1;
    while (w < MAX_WAVES) {
        const int64_t l = lds_bytes(m.dm, mode, S, w, gr);
        if (l > m.lds_max || (m.lds_max / l) * w >= 8) break;
        w *= 2;
    }
    return w;
}

// Launch shape of each mode.  States per workgroup S: the most (4, 2 or 1)
// whose interleaved working set fits the LDS of one workgroup; waves per
// workgroup as default_waves.  A user setting overrides either choice when it
// fits.  The adjoint keeps its per-reaction parameter sums in LDS when they
// fit beside one state's working set.
void choose_launch(Mechanism& m) {
    m.adj_grad_in_lds = lds_bytes(m.dm, MODE_ADJ, 1, 1, true) <= m.lds_max;
    for (int mode = 0; mode < N_MODES; ++mode) {
        const bool gr = mode == MODE_ADJ && m.adj_grad_in_lds;
        auto L = [&](int S, int w) { return lds_bytes(m.dm, mode, S, w, gr); };
        int S = 1;
        for (int c = 4; c >= 1; c >>= 1)
            if (L(c, 1) <= m.lds_max) { S = c; break; }
        m.auto_S[mode] = S;
        m.auto_waves[mode] = default_waves(m, mode, S, gr);
        m.tuned_layout[mode] = -1;
        // Jacobians in layout F: 8 states write 64 bytes of a value together, once
        // their workgroups fill the chip (f_from, at most 8 a unit) and where 4 states don't run on one
        // wave, whose additions have a fixed order, and 8 on more.  Sparse, 4 -> 8
        // states, us: 13 species, 12001 states 42 -> 60, 32768 88 -> 72, 131072 333 -> 271;
        // 32 species, 3000 states 77 -> 81, 20000 223 -> 222, 65536 710 -> 684; dense, 13
        // species, 32768 states 110 -> 80, 32 species 476 -> 405 (8 states have 8 map
        // reads in flight, the other kernels 16)
        m.f_S[mode] = m.auto_S[mode];
        m.f_waves[mode] = m.auto_waves[mode];
        m.f_from[mode] = 0;
        if ((mode == MODE_SPARSE || mode == MODE_DENSE) && !m.dm.det && !m.dm.lsearch) {
            const int w8 = default_waves(m, mode, 8, gr);
            if (S == 4 && L(8, w8) <= m.lds_max && (w8 == 1 || m.auto_waves[mode] > 1)) {
                m.f_S[mode] = 8;
                m.f_waves[mode] = w8;
                m.f_from[mode] = 256 * 8 * std::min<int64_t>(8, m.lds_max / L(8, w8));
            }
        }
        const int maxS = max_states(kernel_mode(m, mode, false));
        if (m.user_S && m.user_S <= maxS && L(m.user_S, m.user_waves ? m.user_waves : 1) <= m.lds_max)
            S = m.user_S;
        if (wide_takes(m, mode, m.user_S, m.user_waves)) {
            m.automatic[mode] = false;
            m.S[mode] = m.user_S;
            m.waves[mode] = m.user_waves;
            m.lds[mode] = wide_lds(m.gm, m.user_waves);
            continue;
        }
        int w = m.user_waves ? m.user_waves : default_waves(m, mode, S, gr);
        if (L(S, w) > m.lds_max) w = default_waves(m, mode, S, gr);
        m.S[mode] = S;
        m.waves[mode] = w;
        m.lds[mode] = L(S, w);
        m.automatic[mode] = !m.user_S && !m.user_waves;
    }
}

}  // namespace pj

namespace {

pj_status eval(const pj_mech* mech, int mode, pj_form form, pj_layout layout, int64_t n,
               const double* state, const double* param, double* dstate, double* jac,
               pj_stream stream, const double* vin = nullptr, double* grad = nullptr,
               const double* arr = nullptr) {
    if (!mech) return fail(PJ_E_INVALID, "NULL mechanism");
    if (form != PJ_CONP && form != PJ_CONV) return fail(PJ_E_INVALID, "bad form");
    if (layout != PJ_LAYOUT_F && layout != PJ_LAYOUT_C) return fail(PJ_E_INVALID, "bad layout");
    if (n < 0) return fail(PJ_E_INVALID, "negative n_states");
    if (n == 0) { g_err.clear(); return PJ_OK; }
    if (!state || !param) return fail(PJ_E_INVALID, "NULL state or parameter");
    if (mode == pj::MODE_SRC && !dstate) return fail(PJ_E_INVALID, "NULL output");
    if (mode != pj::MODE_SRC && !jac)
        return fail(PJ_E_INVALID, mode == pj::MODE_ADJ ? "NULL J^T v output" : "NULL Jacobian output");
    if (mode == pj::MODE_ADJ && !vin) return fail(PJ_E_INVALID, "NULL vector v");
    const pj::Mechanism& m = mech->m;
    if (!m.dbuf) return fail(PJ_E_INVALID, "mechanism not uploaded to a device");
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != m.device)
        return fail(PJ_E_INVALID, "the current HIP device is not the one the mechanism was loaded on");
    const int64_t lds = m.lds[mode];
    if (lds > m.lds_max)
        return fail(PJ_E_UNSUPPORTED, "per-state working set (" + std::to_string(lds) +
                                          " B) exceeds the LDS of one workgroup");
    const pj::Route r = pj::route(m, mode, layout, n, mode == pj::MODE_ADJ && dstate, grad != nullptr);
    if (r.kernel != pj::KERNEL_SCATTER) {
        const pj::GatherCall c{&m.gm, m.d_gm, m.dm.ext, pj::gather_mode(mode), form, layout, r.S, r.waves, n, state, param,
                               dstate, jac, arr, (hipStream_t)stream, vin, grad};
        hipError_t e = r.kernel == pj::KERNEL_GATHER ? pj::launch_gather(c) : pj::launch_wide(c);
        if (e != hipSuccess) return fail(PJ_E_DEVICE, std::string("kernel launch failed: ") + hipGetErrorString(e));
        g_err.clear();
        return PJ_OK;
    }
    // the hot loop of the static map carries no trace of the run-time search,
    // the fixed-order additions or per-call parameters: kernels of their own
    int kmode = kernel_mode(m, mode, arr != nullptr);
    if (kmode == pj::MODE_DENSE_U16 && r.S > 4) kmode = pj::MODE_DENSE;   // built for at most 4 states
    const int S = std::min(r.S, max_states(kmode));
    // a call with its own Arrhenius parameters runs on a copy of the device
    // description that points at them (the mechanism itself is not touched)
    pj::DevMech dm = m.dm;
    dm.arr = pj::gptr(arr);
    hipError_t e = pj::launch(dm, kmode, form, layout, S, n, state, param, dstate, jac, vin, grad,
                              m.adj_grad_in_lds ? 1 : 0, r.waves, pj::lds_bytes(m.dm, mode, S, r.waves, m.adj_grad_in_lds),
                              (hipStream_t)stream);
    if (e != hipSuccess) return fail(PJ_E_DEVICE, std::string("kernel launch failed: ") + hipGetErrorString(e));
    g_err.clear();
    return PJ_OK;
}

}  // namespace

extern "C" {

pj_status pj_mech_parse_ex(const char* desc_path, int options, pj_mech** out) {
    if (!out) return fail(PJ_E_INVALID, "NULL output handle");
    *out = nullptr;
    if (!desc_path) return fail(PJ_E_INVALID, "NULL path");
    if (options & ~(PJ_OPT_APPROX_JACOBIAN | PJ_OPT_CCS | PJ_OPT_LINEAR_SEARCH | PJ_OPT_DETERMINISTIC))
        return fail(PJ_E_INVALID, "unknown option bits");
    pj_mech* h = new (std::nothrow) pj_mech();
    if (!h) return fail(PJ_E_NOMEM, "out of host memory");
    h->m.opts = options;
    std::string err;
    pj_status st = pj::build_mechanism(desc_path, h->m, err);
    if (st != PJ_OK) {
        pj_mech_free(h);
        return fail(st, err);
    }
    *out = h;
    g_err.clear();
    return PJ_OK;
}

pj_status pj_mech_upload(pj_mech* mech) {
    if (!mech) return fail(PJ_E_INVALID, "NULL mechanism");
    if (mech->m.dbuf) return fail(PJ_E_INVALID, "mechanism already uploaded");
    std::string err;
    pj_status st = pj::upload_mechanism(mech->m, err);
    if (st != PJ_OK) {
        if (mech->m.dbuf) { (void)hipFree(mech->m.dbuf); mech->m.dbuf = nullptr; }
        return fail(st, err);
    }
    g_err.clear();
    return PJ_OK;
}

pj_status pj_mech_parse(const char* desc_path, pj_mech** out) { return pj_mech_parse_ex(desc_path, 0, out); }

int pj_mech_options(const pj_mech* mech) { return mech ? mech->m.opts : -1; }

pj_status pj_mech_load(const char* desc_path, pj_mech** out) { return pj_mech_load_ex(desc_path, 0, out); }

pj_status pj_mech_load_ex(const char* desc_path, int options, pj_mech** out) {
    pj_status st = pj_mech_parse_ex(desc_path, options, out);
    if (st != PJ_OK) return st;
    st = pj_mech_upload(*out);
    if (st != PJ_OK) {
        std::string keep = g_err;
        pj_mech_free(*out);
        *out = nullptr;
        return fail(st, keep);
    }
    return PJ_OK;
}

void pj_mech_free(pj_mech* mech) {
    if (!mech) return;
    if (mech->m.dbuf) {
        int cur = -1;
        (void)hipGetDevice(&cur);
        if (cur != mech->m.device) (void)hipSetDevice(mech->m.device);
        (void)hipFree(mech->m.dbuf);
        if (cur >= 0 && cur != mech->m.device) (void)hipSetDevice(cur);
    }
    delete mech;
}

int pj_mech_n_species(const pj_mech* mech) { return mech ? mech->m.ns : -1; }
int pj_mech_n_reactions(const pj_mech* mech) { return mech ? mech->m.nr : -1; }
int pj_mech_state_size(const pj_mech* mech) { return mech ? mech->m.ns + 1 : -1; }

pj_status pj_mech_jac_pattern(const pj_mech* mech, int64_t* nnz, const int32_t** row_ptr,
                              const int32_t** col_idx) {
    if (!mech || !nnz || !row_ptr || !col_idx) return fail(PJ_E_INVALID, "NULL argument");
    *nnz = mech->m.nnz;
    *row_ptr = mech->m.row_ptr.data();
    *col_idx = mech->m.col_idx.data();
    g_err.clear();
    return PJ_OK;
}

pj_status pj_mech_jac_pattern_ccs(const pj_mech* mech, int64_t* nnz, const int32_t** col_ptr,
                                  const int32_t** row_idx) {
    if (!mech || !nnz || !col_ptr || !row_idx) return fail(PJ_E_INVALID, "NULL argument");
    *nnz = mech->m.nnz;
    *col_ptr = mech->m.col_ptr.data();
    *row_idx = mech->m.row_idx.data();
    g_err.clear();
    return PJ_OK;
}

pj_status pj_eval_source(const pj_mech* mech, pj_form form, pj_layout layout, int64_t n_states,
                         const double* d_state, const double* d_param, double* d_dstate,
                         pj_stream stream) {
    return eval(mech, pj::MODE_SRC, form, layout, n_states, d_state, d_param, d_dstate, nullptr,
                stream);
}

pj_status pj_eval_jacobian_sparse(const pj_mech* mech, pj_form form, pj_layout layout,
                                  int64_t n_states, const double* d_state, const double* d_param,
                                  double* d_jac_vals, double* d_dstate_or_null, pj_stream stream) {
    return eval(mech, pj::MODE_SPARSE, form, layout, n_states, d_state, d_param, d_dstate_or_null,
                d_jac_vals, stream);
}

pj_status pj_eval_jacobian_dense(const pj_mech* mech, pj_form form, pj_layout layout,
                                 int64_t n_states, const double* d_state, const double* d_param,
                                 double* d_jac, double* d_dstate_or_null, pj_stream stream) {
    return eval(mech, pj::MODE_DENSE, form, layout, n_states, d_state, d_param, d_dstate_or_null,
                d_jac, stream);
}

pj_status pj_eval_adjoint(const pj_mech* mech, pj_form form, pj_layout layout, int64_t n_states,
                          const double* d_state, const double* d_param, const double* d_v,
                          double* d_jtv, double* d_grad_or_null, double* d_dstate_or_null,
                          pj_stream stream) {
    if (n_states == 0 && mech && d_grad_or_null && mech->m.dbuf) {
        // an empty batch still defines the gradient sums: zero
        hipError_t e = pj::zero_async(d_grad_or_null, 3 * (int64_t)mech->m.nr, (hipStream_t)stream);
        if (e != hipSuccess) return fail(PJ_E_DEVICE, std::string("zeroing the gradient failed: ") + hipGetErrorString(e));
    }
    return eval(mech, pj::MODE_ADJ, form, layout, n_states, d_state, d_param, d_dstate_or_null, d_jtv,
                stream, d_v, d_grad_or_null);
}

pj_status pj_eval_source_arrhenius(const pj_mech* mech, pj_form form, pj_layout layout, int64_t n_states,
                                   const double* d_state, const double* d_param, const double* d_arrhenius,
                                   double* d_dstate, pj_stream stream) {
    if (!d_arrhenius) return fail(PJ_E_INVALID, "NULL Arrhenius parameters");
    return eval(mech, pj::MODE_SRC, form, layout, n_states, d_state, d_param, d_dstate, nullptr, stream,
                nullptr, nullptr, d_arrhenius);
}

pj_status pj_eval_adjoint_arrhenius(const pj_mech* mech, pj_form form, pj_layout layout, int64_t n_states,
                                    const double* d_state, const double* d_param, const double* d_arrhenius,
                                    const double* d_v, double* d_jtv, double* d_grad_or_null,
                                    double* d_dstate_or_null, pj_stream stream) {
    if (!d_arrhenius) return fail(PJ_E_INVALID, "NULL Arrhenius parameters");
    if (n_states == 0 && mech && d_grad_or_null && mech->m.dbuf) {
        hipError_t e = pj::zero_async(d_grad_or_null, 3 * (int64_t)mech->m.nr, (hipStream_t)stream);
        if (e != hipSuccess) return fail(PJ_E_DEVICE, std::string("zeroing the gradient failed: ") + hipGetErrorString(e));
    }
    return eval(mech, pj::MODE_ADJ, form, layout, n_states, d_state, d_param, d_dstate_or_null, d_jtv,
                stream, d_v, d_grad_or_null, d_arrhenius);
}

pj_status pj_mech_set_arrhenius(pj_mech* mech, const double* lnA, const double* b, const double* theta) {
    if (!mech) return fail(PJ_E_INVALID, "NULL mechanism");
    pj::Mechanism& m = mech->m;
    for (int i = 0; i < m.nr; ++i) {
        if (lnA) m.rx[i].lnA = lnA[i];
        if (b) m.rx[i].b = b[i];
        if (theta) m.rx[i].theta = theta[i];
    }
    if (m.dbuf) {
        for (int p = 0; p < m.nr; ++p) {
            const auto& r = m.rx[m.order[p]];
            m.h_rec[p].lnA = r.lnA;
            m.h_rec[p].b = r.b;
            m.h_rec[p].theta = r.theta;
        }
        int cur = -1;
        (void)hipGetDevice(&cur);
        if (cur != m.device && hipSetDevice(m.device) != hipSuccess)
            return fail(PJ_E_DEVICE, "cannot select the mechanism's device");
        hipError_t e = hipMemcpy((unsigned char*)m.dbuf + m.off_rec, m.h_rec.data(),
                                 m.h_rec.size() * sizeof(pj::RxnRec), hipMemcpyHostToDevice);
        if (cur >= 0 && cur != m.device) (void)hipSetDevice(cur);
        if (e == hipSuccess && m.gm.ok) {
            for (int p = 0; p < m.nr; ++p) {
                const auto& r = m.rx[m.gorder[p]];
                m.h_frec[p].lnA = r.lnA;
                m.h_frec[p].b = r.b;
                m.h_frec[p].theta = r.theta;
            }
            if (cur != m.device) (void)hipSetDevice(m.device);
            e = hipMemcpy((unsigned char*)m.dbuf + m.off_frec, m.h_frec.data(), m.h_frec.size() * sizeof(pj::FastRec),
                          hipMemcpyHostToDevice);
            if (cur >= 0 && cur != m.device) (void)hipSetDevice(cur);
        }
        if (e != hipSuccess) return fail(PJ_E_DEVICE, std::string("update of the reaction table failed: ") + hipGetErrorString(e));
    }
    g_err.clear();
    return PJ_OK;
}

pj_status pj_mech_get_arrhenius(const pj_mech* mech, double* lnA, double* b, double* theta) {
    if (!mech) return fail(PJ_E_INVALID, "NULL mechanism");
    for (int i = 0; i < mech->m.nr; ++i) {
        if (lnA) lnA[i] = mech->m.rx[i].lnA;
        if (b) b[i] = mech->m.rx[i].b;
        if (theta) theta[i] = mech->m.rx[i].theta;
    }
    g_err.clear();
    return PJ_OK;
}

pj_status pj_mech_set_launch(pj_mech* mech, int states_per_group, int waves_per_group) {
    if (!mech) return fail(PJ_E_INVALID, "NULL mechanism");
    if (states_per_group && !pow2_upto(states_per_group, MAX_S))
        return fail(PJ_E_INVALID, "states_per_group must be 0 or a power of two up to 64");
    if (waves_per_group < 0 || waves_per_group > MAX_WAVES)
        return fail(PJ_E_INVALID, "waves_per_group must be 0 (automatic) or 1 to 8");
    mech->m.user_S = states_per_group;
    mech->m.user_waves = waves_per_group;
    if (mech->m.dbuf) {
        pj::choose_launch(mech->m);
    } else {
        // provisional until the upload measures the LDS the modes need
        for (int mode = 0; mode < pj::N_MODES; ++mode) {
            mech->m.S[mode] = states_per_group ? states_per_group : 1;
            if (mode == pj::MODE_ADJ && mech->m.S[mode] > pj::MAX_S_ADJ) mech->m.S[mode] = pj::MAX_S_ADJ;
            mech->m.waves[mode] = waves_per_group ? waves_per_group : 1;
        }
    }
    g_err.clear();
    return PJ_OK;
}

pj_status pj_mech_set_waves_per_state(pj_mech* mech, int waves_per_state) {
    if (waves_per_state != 0 && !pow2_upto(waves_per_state, 4))
        return fail(PJ_E_INVALID, "waves_per_state must be 0, 1, 2 or 4");
    return pj_mech_set_launch(mech, waves_per_state ? 1 : 0, waves_per_state);
}

int pj_mech_waves_per_state(const pj_mech* mech, int for_jacobian) {
    if (!mech) return -1;
    const int mode = for_jacobian ? pj::MODE_SPARSE : pj::MODE_SRC;
    int S, w;
    int64_t lds;
    pj::nominal_shape(mech->m, mode, S, w, lds);
    return S == 1 ? w : -1;
}

int pj_mech_kernel(const pj_mech* mech, int mode, pj_layout layout, int64_t n_states, int fused, int* states_per_group,
                   int* waves_per_group) {
    if (!mech || !mech->m.dbuf || mode < 0 || mode >= pj::N_MODES || n_states < 1 ||
        (layout != PJ_LAYOUT_F && layout != PJ_LAYOUT_C))
        return -1;
    const pj::Mechanism& m = mech->m;
    const pj::Route r = pj::route(m, mode, layout, n_states, mode == pj::MODE_ADJ && fused);
    if (states_per_group)
        *states_per_group = r.kernel == pj::KERNEL_SCATTER ? std::min(r.S, max_states(kernel_mode(m, mode, false))) : r.S;
    if (waves_per_group) *waves_per_group = r.waves;
    return r.kernel;
}

pj_status pj_mech_set_dense_unroll(pj_mech* mech, int entries) {
    if (!mech) return fail(PJ_E_INVALID, "NULL mechanism");
    if (entries != 0 && entries != 8 && entries != 16)
        return fail(PJ_E_INVALID, "entries must be 0 (default, 16), 8 or 16");
    mech->m.dense_unroll = entries == 8 ? 8 : 16;
    g_err.clear();
    return PJ_OK;
}

int pj_mech_dense_unroll(const pj_mech* mech) { return mech ? mech->m.dense_unroll : -1; }

int pj_mech_launch_shape(const pj_mech* mech, int mode, int* states_per_group, int* waves_per_group) {
    if (!mech || mode < 0 || mode >= pj::N_MODES) return -1;
    int S, w;
    int64_t lds;
    pj::nominal_shape(mech->m, mode, S, w, lds);
    if (states_per_group) *states_per_group = S;
    if (waves_per_group) *waves_per_group = w;
    return 0;
}

}  // extern "C"

namespace {

// time every launch shape that fits for `mode` and keep the fastest
pj_status autotune(pj_mech* mech, int mode, pj_form form, pj_layout layout, int64_t n_states,
                   const double* d_state, const double* d_param, double* dst, double* jac, const double* vin,
                   double* grad, int reps, pj_stream stream, int* states_per_group, int* waves_per_group,
                   float* ms) {
    if (reps < 1) return fail(PJ_E_INVALID, "reps must be at least 1");
    if (n_states < 1) return fail(PJ_E_INVALID, "autotuning needs at least one state");
    pj::Mechanism& m = mech->m;
    // validate the arguments once with the current shape
    pj_status st = eval(mech, mode, form, layout, n_states, d_state, d_param, dst, jac, stream, vin, grad);
    if (st != PJ_OK) return st;
    const bool gr = mode == pj::MODE_ADJ && m.adj_grad_in_lds;
    const int kmode0 = kernel_mode(m, mode, false);
    const int maxS = max_states(kmode0);
    // the dense output's unroll width is a dimension of the search (8, 16)
    const int n_du = mode == pj::MODE_DENSE ? 2 : 1;
    int best_du = m.dense_unroll;
    hipStream_t hs = (hipStream_t)stream;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
        if (e0) (void)hipEventDestroy(e0);
        return fail(PJ_E_DEVICE, "hipEventCreate failed");
    }
    int best_S = m.S[mode], best_w = m.waves[mode];
    float best = -1.0f, best_scatter = -1.0f;
    int scatter_S = m.auto_S[mode], scatter_w = m.auto_waves[mode];
    std::string err;
    for (int S = 1; S <= maxS && err.empty(); S *= 2) {
        for (int w = 1; w <= MAX_WAVES * n_du && err.empty(); ++w) {
            const int du = w > MAX_WAVES ? 8 : 16;
            const int wv = w > MAX_WAVES ? w - MAX_WAVES : w;
            const int kmode = n_du == 2 ? (du == 16 ? pj::MODE_DENSE_U16 : pj::MODE_DENSE) : kmode0;
            if (kmode == pj::MODE_DENSE_U16 && S > 4) continue;   // built for at most 4 states
            const int64_t l = pj::lds_bytes(m.dm, mode, S, wv, gr);
            // a shape that the gather kernels take is theirs (timed once)
            const bool gather = pj::gather_takes(m, mode, layout, n_states, S, wv);
            const bool wide = pj::wide_takes(m, mode, S, wv);
            if ((!wide && l > m.lds_max) || (gather && du != 16)) continue;
            auto go = [&]() {
                if (wide)
                    return pj::launch_wide({&m.gm, m.d_gm, m.dm.ext, pj::GM_SRC, form, layout, S, wv, n_states, d_state,
                                            d_param, dst, nullptr, nullptr, hs, nullptr, nullptr});
                if (gather)
                    return pj::launch_gather({&m.gm, m.d_gm, m.dm.ext, pj::gather_mode(mode), form, layout, S, wv, n_states,
                                              d_state, d_param, dst, jac, nullptr, hs, vin, grad});
                return pj::launch(m.dm, kmode, form, layout, S, n_states, d_state, d_param, dst, jac, vin, grad,
                                  gr ? 1 : 0, wv, l, hs);
            };
            hipError_t e = go();
            if (e == hipSuccess) e = hipEventRecord(e0, hs);
            for (int r = 0; r < reps && e == hipSuccess; ++r) e = go();
            if (e == hipSuccess) e = hipEventRecord(e1, hs);
            if (e == hipSuccess) e = hipEventSynchronize(e1);
            float t = 0.0f;
            if (e == hipSuccess) e = hipEventElapsedTime(&t, e0, e1);
            if (e != hipSuccess) {
                err = std::string("autotuning launch failed: ") + hipGetErrorString(e);
                break;
            }
            t /= (float)reps;
            if (!gather && !wide && (best_scatter < 0.0f || t < best_scatter)) {
                best_scatter = t;
                scatter_S = S;
                scatter_w = wv;
            }
            if (best < 0.0f || t < best) {
                best = t;
                best_S = S;
                best_w = wv;
                best_du = du;
            }
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (!err.empty()) return fail(PJ_E_DEVICE, err);
    m.automatic[mode] = false;
    m.tuned_layout[mode] = layout;
    m.tuned_kernel[mode] = pj::gather_takes(m, mode, layout, n_states, best_S, best_w) ? pj::KERNEL_GATHER
                           : pj::wide_takes(m, mode, best_S, best_w)                   ? pj::KERNEL_WIDE
                                                                                       : pj::KERNEL_SCATTER;
    if (mode == pj::MODE_ADJ) {
        // calls with fused source terms stay with the scatter kernels
        m.auto_S[mode] = scatter_S;
        m.auto_waves[mode] = scatter_w;
        m.f_S[mode] = scatter_S;
        m.f_waves[mode] = scatter_w;
        m.f_from[mode] = 0;
    }
    m.S[mode] = best_S;
    m.waves[mode] = best_w;
    m.lds[mode] = pj::wide_takes(m, mode, best_S, best_w) ? pj::wide_lds(m.gm, best_w)
                                                          : pj::lds_bytes(m.dm, mode, best_S, best_w, gr);
    if (mode == pj::MODE_DENSE) m.dense_unroll = best_du;
    if (states_per_group) *states_per_group = best_S;
    if (waves_per_group) *waves_per_group = best_w;
    if (ms) *ms = best;
    g_err.clear();
    return PJ_OK;
}

}  // namespace

extern "C" {

pj_status pj_mech_autotune(pj_mech* mech, int mode, pj_form form, pj_layout layout, int64_t n_states,
                           const double* d_state, const double* d_param, double* d_out,
                           double* d_dstate_or_null, int reps, pj_stream stream,
                           int* states_per_group, int* waves_per_group, float* ms) {
    if (!mech) return fail(PJ_E_INVALID, "NULL mechanism");
    if (mode < pj::MODE_SRC || mode > pj::MODE_DENSE) return fail(PJ_E_INVALID, "bad mode");
    double* dst = mode == pj::MODE_SRC ? d_out : d_dstate_or_null;
    double* jac = mode == pj::MODE_SRC ? nullptr : d_out;
    return autotune(mech, mode, form, layout, n_states, d_state, d_param, dst, jac, nullptr, nullptr, reps, stream,
                    states_per_group, waves_per_group, ms);
}

pj_status pj_mech_autotune_adjoint(pj_mech* mech, pj_form form, pj_layout layout, int64_t n_states,
                                   const double* d_state, const double* d_param, const double* d_v,
                                   double* d_jtv, double* d_grad_or_null, int reps, pj_stream stream,
                                   int* states_per_group, int* waves_per_group, float* ms) {
    if (!mech) return fail(PJ_E_INVALID, "NULL mechanism");
    return autotune(mech, pj::MODE_ADJ, form, layout, n_states, d_state, d_param, nullptr, d_jtv, d_v,
                    d_grad_or_null, reps, stream, states_per_group, waves_per_group, ms);
}

int64_t pj_mech_lds_bytes(const pj_mech* mech, int for_jacobian) {
    if (!mech) return -1;
    int S, w;
    int64_t lds;
    pj::nominal_shape(mech->m, for_jacobian ? pj::MODE_SPARSE : pj::MODE_SRC, S, w, lds);
    return lds;
}

const char* pj_last_error(void) { return g_err.c_str(); }

}  // extern "C"
