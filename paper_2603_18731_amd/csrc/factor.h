// Whether an operator factors over the low and the high part of its strings (product.h), and what the
// lists of the parts need of it: the groups by class, the keys of their terms and the tables of
// coefficients.  It depends on the operator and the split qubit alone, so the operator keeps it for the
// split in halves, which a subspace of at most 32 qubits has by itself (94 320 terms: 1.3 ms, of 150 for
// the compilation; per binding it was half of what binding takes).
#pragma once

#include <algorithm>

#include "common.h"

namespace qsd {

constexpr uint32_t kMaxKeys = 16384;        // term keys of one part: 2 key + sign fits 15 bits
constexpr uint32_t kMaxTail = 200;          // terms after the table, counted in 8 bits
constexpr uint64_t kMaxTable = 1ull << 23;  // entries of a two-sided table

// Term kinds within a group's part-only segment.
constexpr uint32_t kOwn = 0;    // depends on the group's own part alone
constexpr uint32_t kOther = 1;  // wants one qubit of the other part (class A: its key's table row)
constexpr uint32_t kFirst = 2;  // class B: the own term that heads its key's table row

struct HostTerm {
    uint32_t care, want, sign;
};

// Everything the device lists need of the operator, or `ok` = false.
struct Classified {
    bool ok = false;
    int split = 0;
    std::vector<uint32_t> tinfo;                    // [T]
    std::vector<uint32_t> gflip[2], gt0[2], gnt[2]; // part-only groups (A, B)
    uint32_t n1[2] = {0, 0};
    std::vector<uint32_t> fflip[2], fcare[2], fkey0[2], fwant[2], fsign[2];
    std::vector<double> ctab, dep, whead, wdep;     // dep [high][nUa], wdep [nWb][low]
    uint32_t nUa = 0, nWb = 0, tail_len = 0, rmask = 0;
    bool full = true;
};

inline Classified classify(const qsd_op *op, int split) {
    Classified c;
    c.split = split;
    const int nhi = op->n_qubits - split;
    if (op->Wp != 1 || op->is_complex || split < 1 || split > 16 || nhi < 1 || nhi > 16) return c;
    const uint32_t lm = (1u << split) - 1u;
    const size_t G = op->g_info.size(), T = op->t_coef.size() / 2;
    c.tinfo.assign(T, 0u);
    auto term = [&](size_t t) {
        return HostTerm{(uint32_t)op->t_cws[3 * t], (uint32_t)op->t_cws[3 * t + 1], (uint32_t)op->t_cws[3 * t + 2]};
    };
    auto half = [&](uint32_t m, int high) { return high ? m >> split : m & lm; };
    // the classes in order: low part only, both, high part only
    int stage = 0;
    size_t ab0 = G, ab1 = 0;
    for (size_t g = 0; g < G; ++g) {
        const uint32_t m = (uint32_t)op->g_mask[g];
        const int cls = half(m, 0) ? (half(m, 1) ? 1 : 0) : 2;
        if (cls < stage) return c;
        stage = cls;
        if (cls == 1) {
            ab0 = std::min(ab0, g);
            ab1 = g + 1;
        }
    }
    if (ab0 == G) ab1 = G;
    // classes A and B: within the terms that one ladder pattern selects, own terms and terms
    // that want one qubit of the other part
    uint32_t seg_tail = 0;
    std::vector<std::pair<uint64_t, double>> dep;  // (key << 8 | qubit, coefficient)
    std::vector<uint32_t> pats;
    for (size_t g = 0; g < G; ++g) {
        if (g >= ab0 && g < ab1 && ab0 < G) continue;
        const uint32_t m = (uint32_t)op->g_mask[g];
        const int H = half(m, 0) ? 0 : 1;
        const size_t a = op->g_term0[g], e = a + op->g_nterm[g];
        bool byflip = true;
        for (size_t t = a; t < e; ++t) byflip &= (term(t).care & m) == m;
        bool anydep = false;
        uint32_t tails = 0;
        // patterns: at most 2^4 with a ladder group, found in stored order
        pats.clear();
        for (size_t t = a; t < e; ++t) {
            const uint32_t p = byflip ? term(t).want & m : 0u;
            if (std::find(pats.begin(), pats.end(), p) == pats.end()) {
                pats.push_back(p);
                if (pats.size() > 16) return c;
            }
        }
        for (const uint32_t p : pats) {
            uint32_t own_before = 0, own_after = 0, deps = 0, last_q = 0;
            HostTerm key{};
            size_t head_t = 0;  // the last own term before the others
            for (size_t t = a; t < e; ++t) {
                const HostTerm x = term(t);
                if (byflip && (x.want & m) != p) continue;
                const uint32_t oc = half(x.care, !H), ow = half(x.want, !H), os = half(x.sign, !H);
                const HostTerm k{half(x.care, H), half(x.want, H), half(x.sign, H)};
                if (!oc && !os) {
                    if (deps) {
                        if (H == 0) return c;  // class A: own terms come first
                        ++own_after;
                    } else {
                        ++own_before;
                        head_t = t;
                    }
                    continue;
                }
                if (os || oc != ow || (oc & (oc - 1u))) return c;
                const uint32_t q = (uint32_t)__builtin_ctz(oc);
                if (deps && q <= last_q) return c;
                last_q = q;
                if (!deps) {
                    // the terms' own part: one key for all of them; an own term with the key's
                    // projector bits makes the element exist whenever one of them matches (class
                    // B: that term alone comes before them, with the key's sign mask)
                    if (!own_before || (H == 1 && own_before != 1)) return c;
                    bool same = false;
                    for (size_t u = a; u < t; ++u) {
                        const HostTerm y = term(u);
                        if (byflip && (y.want & m) != p) continue;
                        same |= half(y.care, H) == k.care && half(y.want, H) == k.want &&
                                (H == 0 || half(y.sign, H) == k.sign);
                    }
                    if (!same) return c;
                    key = k;
                    const uint32_t id = H == 0 ? c.nUa++ : c.nWb++;
                    if (id + 1 >= kMaxKeys) return c;
                    if (H == 1) {
                        c.tinfo[head_t] = kFirst | id << 8;
                        c.whead.push_back(op->t_coef[2 * head_t]);
                    }
                } else if (key.care != k.care || key.want != k.want || key.sign != k.sign) {
                    return c;
                }
                ++deps;
                const uint32_t id = (H == 0 ? c.nUa : c.nWb) - 1u;
                c.tinfo[t] = kOther | id << 8;
                if (H == 0) {
                    dep.push_back({(uint64_t)id << 8 | q, op->t_coef[2 * t]});
                    c.rmask |= 1u << q;
                } else {
                    c.wdep.resize((size_t)c.nWb * split, 0.0);
                    c.wdep[(size_t)id * split + q] = op->t_coef[2 * t];
                }
            }
            anydep |= deps != 0;
            if (H == 1) tails = std::max(tails, deps ? own_after : own_before);
        }
        // (terms that follow the table in segment 1, which ends with the last group that has one)
        if (H == 1) {
            seg_tail = std::max(seg_tail, tails);
            if (anydep) c.tail_len = seg_tail;
        }
        c.gflip[H].push_back(half(m, H));
        c.gt0[H].push_back((uint32_t)a);
        c.gnt[H].push_back((uint32_t)(e - a));
        if (anydep) c.n1[H] = (uint32_t)c.gflip[H].size();
    }
    // (groups of segment 1 without such terms use a table row of zeros, the last one)
    ++c.nUa;
    ++c.nWb;
    c.whead.push_back(0.0);
    c.wdep.resize((size_t)c.nWb * split, 0.0);
    c.dep.assign((size_t)nhi * c.nUa, 0.0);
    for (auto &d : dep) c.dep[(size_t)(d.first & 255u) * c.nUa + (size_t)(d.first >> 8)] = d.second;
    if (c.tail_len > kMaxTail) return c;
    // class AB: per part, the flips and their keys.  A group is one flip of each part, so what the flips
    // know is looked up once per group (by the flip, in a table of 2^16); hash maps asked per term took
    // a millisecond for the 14 400 groups and 80 000 terms of a 16-orbital molecule.
    struct Flip {
        uint32_t mask, care, key0;
        std::vector<std::pair<uint32_t, uint32_t>> keys;  // want, sign
        // the key that wants `want`, or the number of keys
        uint32_t find(uint32_t want) const {
            uint32_t k = 0;
            while (k < keys.size() && keys[k].first != want) ++k;
            return k;
        }
    };
    std::vector<Flip> flips[2];
    std::vector<uint32_t> at[2];  // flip -> place in `flips` + 1
    if (ab0 < ab1)
        for (int H = 0; H < 2; ++H) at[H].assign(size_t(1) << (H ? nhi : split), 0u);
    uint32_t cur = 0, prev = 0;
    auto before = [](uint32_t x, uint32_t z) {
        const int px = __builtin_popcount(x), pz = __builtin_popcount(z);
        return px != pz ? px < pz : x < z;
    };
    for (size_t g = ab0; g < ab1; ++g) {
        const uint32_t m = (uint32_t)op->g_mask[g], ml = half(m, 0), mh = half(m, 1);
        const size_t t0 = op->g_term0[g], t1 = t0 + op->g_nterm[g];
        if (t0 == t1) return c;
        if (g == ab0 || mh != cur) {
            if (at[1][mh]) return c;  // the groups of one high flip are not together
            cur = mh;
        } else if (!before(prev, ml)) {
            return c;
        }
        prev = ml;
        Flip *f[2];
        for (int H = 0; H < 2; ++H) {
            const uint32_t mask = half(m, H);
            uint32_t &k = at[H][mask];
            if (!k) {
                flips[H].push_back({mask, half(term(t0).care, H), 0u, {}});
                k = (uint32_t)flips[H].size();
            }
            f[H] = &flips[H][k - 1];
        }
        for (size_t t = t0; t < t1; ++t) {
            const HostTerm x = term(t);
            if (op->t_coef[2 * t] == 0.0 || (float)op->t_coef[2 * t] == 0.0f) return c;  // 0 marks an absent pair
            for (int H = 0; H < 2; ++H) {
                if (f[H]->care != half(x.care, H)) return c;
                const uint32_t want = half(x.want, H), sign = half(x.sign, H), k = f[H]->find(want);
                if (k == f[H]->keys.size())
                    f[H]->keys.push_back({want, sign});
                else if (f[H]->keys[k].second != sign)
                    return c;
                if (f[H]->keys.size() > 16) return c;
            }
        }
    }
    // low flips in the order that every high flip's groups have them (high flips are in order already)
    std::sort(flips[0].begin(), flips[0].end(), [&](const Flip &x, const Flip &z) { return before(x.mask, z.mask); });
    for (int H = 0; H < 2; ++H) {
        for (size_t k = 0; k < flips[H].size(); ++k) {
            Flip &f = flips[H][k];
            at[H][f.mask] = (uint32_t)k + 1u;
            f.key0 = (uint32_t)c.fwant[H].size();
            c.fflip[H].push_back(f.mask);
            c.fcare[H].push_back(f.care);
            c.fkey0[H].push_back(f.key0);
            for (auto &q : f.keys) {
                c.fwant[H].push_back(q.first);
                c.fsign[H].push_back(q.second);
            }
        }
        c.fkey0[H].push_back((uint32_t)c.fwant[H].size());
        if (c.fwant[H].size() >= kMaxKeys) return c;
    }
    const size_t nU = c.fwant[0].size(), nW = c.fwant[1].size();
    if ((uint64_t)nU * nW > kMaxTable) return c;
    c.ctab.assign(nU * nW, 0.0);
    for (size_t g = ab0; g < ab1; ++g) {
        const uint32_t m = (uint32_t)op->g_mask[g];
        const Flip &fl = flips[0][at[0][half(m, 0)] - 1], &fh = flips[1][at[1][half(m, 1)] - 1];
        for (size_t t = op->g_term0[g], e = t + op->g_nterm[g]; t < e; ++t) {
            const HostTerm x = term(t);
            const uint32_t u = fl.key0 + fl.find(half(x.want, 0)), w = fh.key0 + fh.find(half(x.want, 1));
            double &v = c.ctab[(size_t)w * nU + u];
            if (v != 0.0) return c;  // two terms for one pair of keys
            v = op->t_coef[2 * t];
        }
    }
    for (double v : c.ctab) c.full &= v != 0.0;
    c.ok = true;
    return c;
}

}  // namespace qsd
