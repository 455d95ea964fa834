// Host side of the gather kernels: from a parsed mechanism, the reaction
// records with single-molecule slots and the static lists through which the
// kernels sum production rates, column sums and Jacobian entries (the sparse
// index lookup of the paper's Sec. 3.4 done once, from the side of the result).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstring>
#include <map>

#include "internal.h"

namespace pj {

namespace {


struct Sum {
    uint32_t meta;
    std::vector<uint32_t> c;
};

// Lanes of a sum of deg contributions whose lanes take at most len each.
int lanes_of(size_t deg, int len) {
    int p = 1;
    while (p < 64 && (int)((deg + p - 1) / p) > len) p *= 2;
    return p;
}

// Cut sums into groups of 64 lanes.  bits: 16 (two contributions a word) or
// 32; lp_in_word: the number of lanes (its logarithm) goes into spare bits of
// the first word, else into bits 28..30 of the entry word.
// Sums take 2^k neighbouring lanes, the widest first (so that each is
// aligned), then the longest, so that the lanes of a group end together.  The
// length at which a sum is spread over more lanes is the one with the least
// cost: the steps of all groups, a group's own cost counted as 8, and the
// largest share of four waves that take the groups in turn (the others wait for
// it: 111 species, 262144 states 8.49 ms without that term, 8.35 with it).
void cut(const std::vector<Sum>& sums, int bits, bool lp_in_word, uint32_t empty, GatherImage::Lists& out) {
    const int per_word = 32 / bits, head = 3 * per_word, chunk = 4 * per_word;
    int best = -1, full = head + chunk;
    struct Item {
        int sum, lanes, len;
    };
    std::vector<Item> items(sums.size());
    auto arrange = [&](int f) {
        for (size_t i = 0; i < sums.size(); ++i) {
            const int p = lanes_of(sums[i].c.size(), f);
            items[i] = {(int)i, p, (int)((sums[i].c.size() + p - 1) / p)};
        }
        std::stable_sort(items.begin(), items.end(), [](const Item& a, const Item& b) {
            return a.lanes != b.lanes ? a.lanes > b.lanes : a.len > b.len;
        });
        // first item, number of items and steps of each group
        std::vector<std::array<int, 3>> gr;
        for (size_t i = 0; i < items.size();) {
            size_t j = i;
            int used = 0, longest = 0;
            while (j < items.size() && used + items[j].lanes <= 64) {
                used += items[j].lanes;
                longest = std::max(longest, items[j++].len);
            }
            gr.push_back({(int)i, (int)(j - i), longest});
            i = j;
        }
        return gr;
    };
    for (int nc = 1; nc <= 6; ++nc) {
        int cost = 0, t = 0, load[4] = {0, 0, 0, 0};
        for (auto& q : arrange(head + nc * chunk)) {
            const int c = 8 + head + std::max(1, (q[2] - head + chunk - 1) / chunk) * chunk;
            cost += c;
            load[t++ & 3] += c;
        }
        cost += 4 * *std::max_element(load, load + 4);
        if (best < 0 || cost < best) {
            best = cost;
            full = head + nc * chunk;
        }
    }
    for (auto& q : arrange(full)) {
        const int nc = std::max(1, (q[2] - head + chunk - 1) / chunk);   // the first chunk is always there
        const size_t more0 = out.more.size() / 64, h0 = out.head.size();
        out.head.resize(h0 + 64, make_uint4(0xFFFFFFFFu, 0, 0, 0));
        out.ext.resize(h0 + 64);
        out.more.resize(out.more.size() + (size_t)(nc - 1) * 64);
        int lane = 0, widest = 0;
        std::vector<uint32_t> c;      // a lane's contributions
        auto fill = [&](int l, uint32_t meta, int lp) {
            c.resize((size_t)(head + nc * chunk), empty);
            auto word = [&](int k) { return bits == 32 ? c[k] : c[2 * k] | c[2 * k + 1] << 16; };
            uint32_t w0 = word(0);
            if (lp_in_word) w0 |= (uint32_t)(lp & 3) << 1 | (uint32_t)(lp >> 2) << 17;
            else if (meta != 0xFFFFFFFFu) meta |= (uint32_t)lp << 28;
            out.head[h0 + l] = make_uint4(meta, w0, word(1), word(2));
            for (int x = 0; x < nc; ++x)
                (x ? out.more[(more0 + x - 1) * 64 + l] : out.ext[h0 + l]) =
                    make_uint4(word(3 + 4 * x), word(4 + 4 * x), word(5 + 4 * x), word(6 + 4 * x));
            c.clear();
        };
        for (int k = q[0]; k < q[0] + q[1]; ++k) {
            const Sum& sum = sums[items[k].sum];
            const int P = items[k].lanes;
            int lp = 0;
            while ((1 << lp) < P) ++lp;
            widest = std::max(widest, lp);
            // contribution j to lane j mod P: neighbouring lanes then read
            // neighbouring reactions of a sum that many contribute to
            for (int l = 0; l < P; ++l) {
                for (size_t j = l; j < sum.c.size(); j += P) c.push_back(sum.c[j]);
                fill(lane + l, l ? 0xFFFFFFFFu : sum.meta, lp);
            }
            lane += P;
        }
        for (; lane < 64; ++lane) fill(lane, 0xFFFFFFFFu, 0);
        out.desc.push_back(make_uint2((uint32_t)widest | (uint32_t)(nc - 1) << 8, (uint32_t)more0));
    }
}

// The wide kernel's sums for 2 w waves.  All wait for the wave with the most words,
// so a list longer than a wave's share is dealt to parts (further parts go to rows
// of species, at most one for each but the bath gas), and the parts, the longest
// first, to the wave with the fewest words.
void deal(const std::vector<Sum>& sp, int w, GatherImage& g) {
    const int ns = (int)sp.size(), waves = 2 * w;
    size_t total = 0;
    for (auto& s : sp) total += s.c.size();
    size_t len = std::max<size_t>(1, (total + waves - 1) / waves);
    auto parts = [&](const Sum& s) { return std::max<size_t>(1, (s.c.size() + len - 1) / len); };
    for (;; ++len) {
        size_t more = 0;
        for (auto& s : sp) more += parts(s) - 1;
        if ((int)more < ns) break;
    }
    struct Part {
        int to;
        std::vector<uint32_t> c;
    };
    std::vector<Part> all;
    std::vector<int32_t> xs{0};
    for (auto& s : sp) {
        const size_t n = parts(s);
        for (size_t q = 0; q < n; ++q) {
            Part t{q ? ns + xs.back() + (int)q - 1 : (int)s.meta, {}};
            for (size_t j = q; j < s.c.size(); j += n) t.c.push_back(s.c[j]);
            all.push_back(std::move(t));
        }
        xs.push_back(xs.back() + (int)n - 1);
    }
    std::stable_sort(all.begin(), all.end(), [](const Part& a, const Part& b) { return a.c.size() > b.c.size(); });
    std::vector<std::vector<const Part*>> of(waves);
    std::vector<size_t> load(waves, 0);
    for (auto& t : all) {
        int best = -1;
        for (int v = 0; v < waves; ++v)
            if ((int)of[v].size() < WIDE_OWN && (best < 0 || load[v] < load[best])) best = v;
        if (best < 0) return;      // more than the waves hold
        of[best].push_back(&t);
        load[best] += t.c.size();
    }
    g.wt[w] = g.wide.size();
    for (auto& o : of) {
        for (auto* t : o) g.wide.push_back(t->to);
        g.wide.resize(g.wide.size() + WIDE_OWN - o.size(), -1);
        g.gm.own[w] = std::max(g.gm.own[w], (int)o.size());
    }
    g.wo[w] = g.wide.size();
    for (auto& o : of) {
        g.wide.push_back((int32_t)g.wl.size());
        const size_t first = g.wl.size();
        for (size_t q = 0; q < o.size(); ++q)
            for (uint32_t c : o[q]->c) g.wl.push_back((c & 0x7FFF) | (uint32_t)q << 16 | (c & 0x8000) << 16);
        std::stable_sort(g.wl.begin() + first, g.wl.end(), [](uint32_t a, uint32_t b) { return (a & 0x7FFF) < (b & 0x7FFF); });
    }
    g.wide.push_back((int32_t)g.wl.size());
    g.xs[w] = g.wide.size();
    g.wide.insert(g.wide.end(), xs.begin(), xs.end());
}

}  // namespace

void build_gather(const Mechanism& m, const std::vector<RxnRec>& rec, const std::vector<FallRec>& fall,
                  const std::vector<int32_t>& dense_rows, int64_t lds_max, GatherImage& g) {
    const int ns = m.ns, nr = m.nr, N = ns + 1, bath = ns - 1;
    g = GatherImage{};
    GatherMech& gm = g.gm;
    // single-molecule slots: at most three molecules a side
    for (const auto& r : m.rx) {
        int a = 0, b = 0;
        for (auto& e : r.reac) a += e.second;
        for (auto& e : r.prod) b += e.second;
        if (a > MAXSIDE || b > MAXSIDE) return;
    }
    // (8 waves of GATHER_BLOCKS blocks: 2560 reactions; the lists' 13 bits hold 8191)
    if (nr < 1 || (nr + 63) / 64 > 8 * GATHER_BLOCKS || ns >= 8192) return;
    const bool approx = (m.opts & PJ_OPT_APPROX_JACOBIAN) != 0;
    const int nr_pad = (int)rec.size();
    // The kernel order of rec by class and shape, its classes the costliest
    // first: a class then starts in the block where the costlier one ends, and
    // the block that is not full holds the cheapest reactions.
    std::vector<int> ord(nr);
    for (int p = 0; p < nr; ++p) ord[p] = p;
    auto cost = [&](int p) {
        const auto& r = m.rx[m.order[p]];
        return r.kind == K_ELEM ? (r.rev ? 1 : 0) : kind_falloff(r.kind) ? 10 + r.kind + (r.chemact ? 3 : 0)
               : r.kind == K_THREEBODY ? 2 : 3 + r.kind;
    };
    std::stable_sort(ord.begin(), ord.end(), [&](int a, int b) { return cost(a) > cost(b); });
    g.order.resize(nr);
    for (int p = 0; p < nr; ++p) g.order[p] = m.order[ord[p]];
    // falloff records: those reactions come first
    for (int p = 0; p < nr && kind_falloff(m.rx[g.order[p]].kind); ++p) g.fall.push_back(fall[ord[p]]);
    g.rec.resize(nr_pad);
    std::memset(g.rec.data(), 0, g.rec.size() * sizeof(FastRec));
    FastEff none;
    std::memset(&none, 0, sizeof(none));
    for (auto& s : none.sp) s = (uint16_t)ns;
    g.eff.assign(1, none);

    // species a rate depends on, with the pool element that carries it
    struct Dep {
        int species;
        uint32_t elem;
        bool minus;
    };
    std::vector<std::vector<Dep>> deps(nr);
    std::vector<std::vector<int>> slots(nr);      // unit slots: species, -1 empty
    int el = nr;
    for (int p = 0; p < nr_pad; ++p) {
        FastRec& R = g.rec[p];
        for (auto& s : R.sp) s = (uint16_t)ns;
        if (p >= nr) continue;
        const auto& r = m.rx[g.order[p]];
        const RxnRec& old = rec[ord[p]];
        std::vector<int> sl(NSLOT, -1);
        int mol[2] = {0, 0};
        for (int side = 0; side < 2; ++side)
            for (auto& e : side ? r.prod : r.reac)
                for (int u = 0; u < e.second; ++u) sl[3 * side + mol[side]++] = e.first;
        const bool bathdep = (old.info & INFO_BATH) != 0;
        uint32_t w = (uint32_t)r.kind | (r.rev ? GI_REV : 0) | (bathdep ? GI_BATH : 0) | (r.chemact ? GI_CHEMACT : 0);
        w |= (uint32_t)(mol[1] - mol[0] + 3) << 8 | (uint32_t)mol[0] << 12 | (uint32_t)mol[1] << 14;
        for (int a = 0; a < NSLOT; ++a) {
            if (sl[a] < 0) continue;
            R.sp[a] = (uint16_t)sl[a];
            if (sl[a] == bath) w |= 1u << (16 + a);
            if (a < 3) deps[p].push_back({sl[a], (uint32_t)p, false});
        }
        if (r.rev) {
            R.bpos = (uint16_t)el;
            for (int a = 3; a < NSLOT; ++a) if (sl[a] >= 0) deps[p].push_back({sl[a], (uint32_t)el, true});
            ++el;
        }
        slots[p] = sl;
        R.tab = old.tab;
        R.lnA = old.lnA;
        R.b = old.b;
        R.theta = old.theta;
        R.domega = old.domega;
        R.info = w;
        R.orig = (uint32_t)g.order[p];
    }
    // dOmega = sum nu (1 - W/W_Ns) is the change of moles, sum nu, when the
    // weights balance as the elements do (each term then carries only its
    // rounding); the column lists hold it as a whole number
    std::vector<int> dom(nr);
    for (int p = 0; p < nr; ++p) {
        double scale = 0;
        for (int k : slots[p]) if (k >= 0) scale += m.W[k] / m.W[bath] + 1.0;
        dom[p] = (int)((g.rec[p].info >> 8) & 7) - 3;
        if (std::fabs(g.rec[p].domega - dom[p]) > 4e-16 * scale) return;
    }
    // third-body terms: a record for every reaction that is not elementary
    // (they come first)
    for (int p = 0; p < nr; ++p) {
        const auto& r = m.rx[g.order[p]];
        if (r.kind == K_ELEM) break;      // none follows
        if (kind_table(r.kind)) {
            g.eff.push_back(none);
            continue;
        }
        std::map<int, double> al;
        for (auto& e : r.eff) al[e.first] = e.second;
        FastEff E = none;
        int ne = 0;
        g.rec[p].tpos = (uint16_t)el;
        for (auto& e : al) {
            if (e.second == 1.0) continue;
            E.sp[ne] = (uint16_t)e.first;
            E.am1[ne] = e.second - 1.0;
            if (e.first == bath) E.bam1 = e.second - 1.0;
            deps[p].push_back({e.first, (uint32_t)el, false});
            ++ne;
            if (++el >= 8190) return;
        }
        g.rec[p].info |= (uint32_t)ne << 24;
        g.eff.push_back(E);
    }
    // bath-gas partials of the dense rows
    std::vector<int> qb(nr, -1);
    if (!approx)
        for (int p = 0; p < nr; ++p)
            if (g.rec[p].info & GI_BATH) {
                qb[p] = el;
                g.rec[p].qbpos = (uint16_t)el;
                if (++el >= 8190) return;
            }
    if (el >= 8190) return;
    gm.neff = (int)g.eff.size() - 1;
    gm.nfall = (int)g.fall.size();
    gm.zero = el++;
    el += el & 1;
    gm.b3 = el;
    // per 64-reaction chunk: slot positions in use, any reversible, most third
    // bodies, the further types
    for (int c = 0; c < nr_pad; c += 64) {
        uint32_t cm = 0, most = 0;
        for (int p = c; p < std::min(nr, c + 64); ++p) {
            const FastRec& R = g.rec[p];
            for (int a = 0; a < NSLOT; ++a) if (R.sp[a] != ns) cm |= 1u << a;
            if (R.info & GI_REV) cm |= 1u << 6;
            const int kd = R.info & 7;
            if (kd != K_ELEM) cm |= CHUNK_PRESSURE;
            if (kind_table(kd)) cm |= CHUNK_TAB;
            if (kd == K_SRI) cm |= CHUNK_SRI;
            if (R.info & GI_CHEMACT) cm |= CHUNK_CHEMACT;
            most = std::max(most, (R.info >> 24) & 0xFu);
        }
        for (int p = c; p < c + 64; ++p) g.rec[p].chunk = cm | most << 8;
    }

    // ---- lists
    std::vector<Sum> sp(ns), col(ns), br;
    for (int k = 0; k < ns; ++k) sp[k].meta = col[k].meta = (uint32_t)k;
    std::vector<int> dense_of(ns, -1);
    for (size_t d = 0; d < dense_rows.size(); ++d)
        if (dense_rows[d] >= 0) {
            dense_of[dense_rows[d]] = (int)br.size();
            br.push_back({(uint32_t)d, {}});
        }
    std::vector<std::vector<uint32_t>> ent(m.nnz);
    for (int p = 0; p < nr; ++p) {
        for (auto& d : deps[p]) col[d.species].c.push_back((d.elem << 3 | (d.minus ? 1u : 0u)) | (uint32_t)p << 16 | (uint32_t)dom[p] << 29);
        for (int a = 0; a < NSLOT; ++a) {
            const int k = slots[p][a];
            if (k < 0) continue;
            const bool neg = a < 3;
            sp[k].c.push_back((uint32_t)p | (neg ? 0x8000u : 0u));
            if (k == bath) continue;
            if (qb[p] >= 0 && dense_of[k] >= 0) br[dense_of[k]].c.push_back((uint32_t)qb[p] << 3 | (neg ? 1u : 0u));
            const int r0 = m.row_ptr[2 + k], r1 = m.row_ptr[3 + k];
            for (auto& d : deps[p]) {
                if (d.species == bath) continue;
                const auto it = std::lower_bound(m.col_idx.begin() + r0, m.col_idx.begin() + r1, 2 + d.species);
                if (it == m.col_idx.begin() + r1 || *it != 2 + d.species) return;
                ent[it - m.col_idx.begin()].push_back(d.elem << 3 | (d.minus != neg ? 1u : 0u));
            }
        }
    }
    for (int w = 2; w <= 8; ++w) deal(sp, w, g);
    g.wl.insert(g.wl.end(), 64, 0);
    gm.lds_max = (int)lds_max;
    cut(sp, 16, false, (uint32_t)nr, g.sl);
    cut(br, 16, false, (uint32_t)gm.zero << 3, g.bl);
    cut(col, 32, false, (uint32_t)gm.zero << 3, g.cl);

    // the entry word holds the column and the dense row (1 + its index) in 16 bits
    int cb = 1;
    while ((1 << cb) < ns) ++cb;
    gm.dshift = 16 + cb;
    if (br.size() >= (size_t)1 << (16 - cb)) return;

    // rounds: all species rows at once if their entries need no more LDS than
    // the reactions' own values or if that costs no workgroup of a compute
    // unit; else as many rows as fit the values' space
    const int own = 2 * (nr + 1);
    const int all = m.nnz - 2 * N;
    int cap = std::max(own, all);
    auto lds_of = [&](int c) {
        GatherMech t = gm;
        t.ns = ns;
        t.nr = nr;
        t.n_dense_rows = (int)br.size();
        t.npool = (gm.b3 + c + 1) & ~1;
        return gather_lds(t, GM_JAC, 1);
    };
    if (all > own) {
        const int64_t a = lds_of(cap), b = lds_of(own);
        if (a > lds_max || lds_max / a < std::min<int64_t>(lds_max / b, 4)) cap = own;
    }
    // (at the same number of workgroups per compute unit, fewer rounds)
    if (cap == own) {
        const int64_t k = std::min<int64_t>(4, std::max<int64_t>(1, lds_max / lds_of(own)));
        while (cap < all && lds_of(cap + 64) <= lds_max / k) cap += 64;
        const int rounds = (all + cap - 1) / cap;
        cap = std::max(own, std::min(cap, all / rounds + 2 * N));
    }
    for (int k = 0; k < ns - 1; ++k)
        if (m.row_ptr[3 + k] - m.row_ptr[2 + k] > cap || m.row_ptr[3 + k] - m.row_ptr[2 + k] >= 65535) return;
    for (int row = 2; row < N;) {
        JacRound R{};
        R.row0 = row;
        R.e0 = m.row_ptr[row];
        while (row < N && m.row_ptr[row + 1] - R.e0 <= std::min(cap, 65000)) ++row;
        R.row1 = row;
        R.ne = m.row_ptr[row] - R.e0;
        std::vector<Sum> heavy, mid, light;
        for (int i = R.row0; i < R.row1; ++i)
            for (int e = m.row_ptr[i] + 2; e < m.row_ptr[i + 1]; ++e) {
                Sum s{(uint32_t)(e - R.e0) | (uint32_t)(m.col_idx[e] - 2) << 16 |
                          (uint32_t)(i - 2 < ns ? dense_of[i - 2] + 1 : 0) << gm.dshift, std::move(ent[e])};
                (s.c.size() > 6 ? heavy : s.c.size() > 2 ? mid : light).push_back(std::move(s));
            }
        auto longer = [](const Sum& a, const Sum& b) { return a.c.size() > b.c.size(); };
        std::stable_sort(mid.begin(), mid.end(), longer);
        std::stable_sort(light.begin(), light.end(), longer);
        R.heavy0 = (int)g.jh.desc.size();
        cut(heavy, 16, true, (uint32_t)gm.zero << 3, g.jh);
        R.heavy1 = (int)g.jh.desc.size();
        const uint32_t z = (uint32_t)gm.zero << 3;
        auto at = [&](const std::vector<Sum>& v, size_t q, size_t k) { return q < v.size() && k < v[q].c.size() ? v[q].c[k] : z; };
        auto meta = [&](const std::vector<Sum>& v, size_t q) { return q < v.size() ? v[q].meta : 0xFFFFu; };
        R.mid0 = (int)(g.jm.size() / 64);
        for (size_t q0 = 0; q0 < mid.size(); q0 += 64)
            for (size_t q = q0; q < q0 + 64; ++q)
                g.jm.push_back(make_uint4(meta(mid, q), at(mid, q, 0) | at(mid, q, 1) << 16, at(mid, q, 2) | at(mid, q, 3) << 16,
                                          at(mid, q, 4) | at(mid, q, 5) << 16));
        R.mid1 = (int)(g.jm.size() / 64);
        R.light0 = (int)(g.jl.size() / 64);
        for (size_t q0 = 0; q0 < light.size(); q0 += 128)
            for (size_t q = q0; q < q0 + 64; ++q)
                g.jl.push_back(make_uint4(meta(light, q), at(light, q, 0) | at(light, q, 1) << 16,
                                          meta(light, q + 64), at(light, q + 64, 0) | at(light, q + 64, 1) << 16));
        R.light1 = (int)(g.jl.size() / 64);
        g.rounds.push_back(R);
    }
    gm.npool = (gm.b3 + std::max(cap, own) + 1) & ~1;
    gm.ns = ns;
    gm.nr = nr;
    gm.N = N;
    gm.nnz = m.nnz;
    gm.bath = bath;
    gm.n_dense_rows = (int)br.size();
    gm.approx = approx ? 1 : 0;
    gm.n_rounds = (int)g.rounds.size();
    gm.ok = 1;
    g.ok = true;
}

}  // namespace pj
