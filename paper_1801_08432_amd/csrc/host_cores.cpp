// Host tables of the core kernels: the proton-neutron part of H written with
// one particle of each species taken out and put back,
//   sum_{abcd} V[(a b),(c d)] (p+_a n+_b) (n_d p_c),
// so that x is gathered once per (proton core, neutron core) pair for all the
// pairs (c d) that fill it, one dense matrix V of the pair's (2m, parity)
// turns them into the pairs (a b), and the results are added to y.
#include <algorithm>
#include <array>
#include <map>

#include "fotci_internal.h"

namespace fotci {

namespace {

inline bool odd_below(uint32_t m, int i) { return __builtin_popcount(m & ((1u << i) - 1u)) & 1; }

constexpr int kCoreVjpTasks = 1536;   // three rounds of two workgroups a CU

struct Cores {
    std::vector<uint32_t> mask;              // grouped by (2M, parity), ascending inside a group
    std::vector<int32_t> group;
    std::map<std::pair<int, int>, int> group_of;
    std::vector<int> first, count;
};

Cores cores_of(const SpeciesBasis &sb, const std::vector<MState> &ms) {
    std::vector<uint32_t> all;
    for (uint32_t m : sb.sd)
        for (uint32_t r = m; r; r &= r - 1) all.push_back(m & ~(r & (0u - r)));
    std::sort(all.begin(), all.end());
    all.erase(std::unique(all.begin(), all.end()), all.end());
    std::map<std::pair<int, int>, std::vector<uint32_t>> by;
    for (uint32_t m : all) {
        int tm = 0, par = 1;
        for (size_t i = 0; i < ms.size(); ++i)
            if ((m >> i) & 1u) tm += ms[i].two_m, par *= ms[i].parity;
        by[{tm, par}].push_back(m);
    }
    Cores c;
    for (auto &g : by) {
        const int id = (int)c.group_of.size();
        c.group_of[g.first] = id;
        c.first.push_back((int)c.mask.size());
        c.count.push_back((int)g.second.size());
        for (uint32_t m : g.second) c.mask.push_back(m), c.group.push_back(id);
    }
    return c;
}

}  // namespace

void build_core_tables(fotci_ham *h) {
    const fotci_basis *b = h->j->b;
    const auto &ms = b->ms;
    const int ns = h->j->ns;
    HostCore &t = h->hc;
    t = HostCore();
    // rows and columns that do not exist are read past the end of a vector, at
    // 2^31 - 2^20 bytes and above
    if (b->p.n < 1 || b->n.n < 1 || !h->tt.ok || b->dim * 8 > 0x7ff00000) return;
    const Cores U = cores_of(b->p, ms), W = cores_of(b->n, ms);
    t.u_mask = U.mask;
    t.u_group = U.group;
    // kept SD by mask, per species
    auto index = [](const SpeciesBasis &sb) {
        std::vector<std::pair<uint32_t, int32_t>> v(sb.sd.size());
        for (size_t i = 0; i < sb.sd.size(); ++i) v[i] = {sb.sd[i], (int32_t)i};
        std::sort(v.begin(), v.end());
        return v;
    };
    auto find = [](const std::vector<std::pair<uint32_t, int32_t>> &v, uint32_t m) {
        auto it = std::lower_bound(v.begin(), v.end(), std::make_pair(m, (int32_t)0));
        return it != v.end() && it->first == m ? it->second : -1;
    };
    const auto pidx = index(b->p), nidx = index(b->n);
    t.u_nn.assign(U.mask.size() * (size_t)ns, 0);
    t.u_base.assign(U.mask.size() * (size_t)ns, kCoreNoRow);
    for (size_t u = 0; u < U.mask.size(); ++u)
        for (int a = 0; a < ns; ++a) {
            if ((U.mask[u] >> a) & 1u) continue;
            const int ip = find(pidx, U.mask[u] | (1u << a));
            if (ip < 0) continue;
            const uint32_t phase = odd_below(U.mask[u], a) ? 0x80000000u : 0u;
            t.u_nn[u * ns + a] = b->sectors[b->p_basis_sector[ip]].nn;
            t.u_base[u * ns + a] = (uint32_t)b->pstart[ip] | phase;
        }
    // neutron cores: groups, codes
    const int nw = (int)W.count.size();
    int64_t total = 0;
    for (int g = 0; g < nw; ++g) {
        t.w_n.push_back(W.count[g]);
        t.w_pad.push_back((W.count[g] + 15) & ~15);
        t.w_off.push_back((int32_t)total);
        total += (int64_t)t.w_pad.back() * ns;
    }
    t.w_null = (int)total;   // a run of null codes as long as the largest group
    total += *std::max_element(t.w_pad.begin(), t.w_pad.end());
    if (total * 4 >= ((int64_t)1 << 30)) return;
    for (int s = kCoreMinShift; s <= kCoreMaxShift; ++s) t.w_code[s - kCoreMinShift].assign((size_t)total, core_null(s));
    for (int g = 0; g < nw; ++g)
        for (int j = 0; j < W.count[g]; ++j) {
            const uint32_t m = W.mask[W.first[g] + j];
            for (int d = 0; d < ns; ++d) {
                if ((m >> d) & 1u) continue;
                const int jn = find(nidx, m | (1u << d));
                if (jn < 0) continue;
                const uint32_t code = (uint32_t)b->n.sd_local[jn] | (odd_below(m, d) ? 0x80000000u : 0u);
                for (auto &c : t.w_code) c[(size_t)t.w_off[g] + (size_t)d * t.w_pad[g] + j] = code;
            }
        }
    // a code's column shifted must stay below the null code's bit
    if (h->tt.max_nn >= (1 << (31 - kCoreMaxShift))) return;
    // pair classes
    std::map<std::pair<int, int>, std::vector<std::pair<int, int>>> pcs;
    for (int a = 0; a < ns; ++a)
        for (int c = 0; c < ns; ++c) pcs[{ms[a].two_m + ms[c].two_m, ms[a].parity * ms[c].parity}].push_back({a, c});
    const size_t ns2 = (size_t)ns * ns;
    std::vector<std::pair<int, int>> pc_q;   // most pairs first: the tasks of a workgroup are drawn in this order
    for (auto &pc : pcs) pc_q.push_back(pc.first);
    std::stable_sort(pc_q.begin(), pc_q.end(), [&](const auto &x, const auto &y) { return pcs[x].size() > pcs[y].size(); });
    for (auto &q : pc_q) {
        const auto &pr = pcs[q];   // by a, then b
        t.pc_n.push_back((int32_t)pr.size());
        t.pc_pair.push_back((int32_t)t.pair_ab.size());
        t.pc_v.push_back((int32_t)t.v_src.size());
        size_t k = 0;
        for (int a = 0; a <= ns; ++a) {
            while (k < pr.size() && pr[k].first < a) ++k;
            t.pc_first.push_back((int32_t)k);
        }
        for (auto &p : pr) t.pair_ab.push_back(p.first | (p.second << 8));
        for (auto &p : pr)
            for (auto &r : pr)
                t.v_src.push_back((int32_t)(((size_t)p.first * ns + p.second) * ns2 + (size_t)r.first * ns + r.second));
    }
    t.n_pc = (int)t.pc_n.size();
    const int nu = (int)U.count.size();
    t.w_of.assign((size_t)nu * t.n_pc, -1);
    for (auto &g : U.group_of)
        for (int k = 0; k < t.n_pc; ++k) {
            auto it = W.group_of.find({b->two_M - g.first.first - pc_q[k].first, b->parity * g.first.second * pc_q[k].second});
            if (it != W.group_of.end()) t.w_of[(size_t)g.second * t.n_pc + k] = it->second;
        }
    if (t.n_pc > kCoreMaxPc || t.v_src.size() * 8 >= (1u << 30)) return;
    // Work items: a core with as many of the states a as a workgroup takes
    // (rows in LDS); the costliest start first.
    int most = 0;   // positions of an item in a class
    struct It {
        int u;
        uint32_t amask;
        int64_t cost;
    };
    std::vector<It> its;
    for (int u = 0; u < (int)U.mask.size(); ++u) {
        std::vector<std::pair<int, int>> st;   // (state, row columns)
        int64_t all = 0;
        for (int a = 0; a < ns; ++a) {
            if (t.u_base[(size_t)u * ns + a] == kCoreNoRow) continue;
            st.push_back({a, t.u_nn[(size_t)u * ns + a]});
            all += st.back().second;
        }
        // as few items as fit, of about equal size
        const int64_t parts = std::max<int64_t>({1, (all + kCoreRowElems - 1) / kCoreRowElems,
                                                 ((int64_t)st.size() + kCoreStates - 1) / kCoreStates});
        const size_t aim = (st.size() + (size_t)parts - 1) / (size_t)parts;
        uint32_t am = 0;
        int64_t cols = 0;
        auto emit = [&] {
            if (!am) return;
            int64_t cost = 0;
            for (int p = 0; p < t.n_pc; ++p) {
                const int w = t.w_of[(size_t)U.group[u] * t.n_pc + p];
                if (w < 0) continue;
                cost += (int64_t)t.w_pad[w] * t.pc_n[p] + 4096;
                int pos = 0;
                for (int a = 0; a < ns; ++a)
                    if ((am >> a) & 1u)
                        pos += (t.pc_first[(size_t)p * (ns + 1) + a + 1] - t.pc_first[(size_t)p * (ns + 1) + a] + 3) / 4;
                most = std::max(most, pos);
            }
            its.push_back({u, am, cost * (4 + __builtin_popcount(am))});
            t.item_cols = std::max(t.item_cols, (int)cols);
            am = 0;
            cols = 0;
        };
        for (auto &s : st) {
            if (am && cols + s.second > kCoreRowElems) emit();
            am |= 1u << s.first;
            cols += s.second;
            if ((size_t)__builtin_popcount(am) >= aim) emit();
        }
        emit();
    }
    if (most > kCoreMaxPos) return;
    std::stable_sort(its.begin(), its.end(), [](const It &x, const It &y) { return x.cost > y.cost; });
    for (auto &i : its) t.items.push_back(i.u), t.items.push_back((int32_t)i.amask);
    // One-body densities: states by (2m, parity), a block of 4 x 4 of a class's
    // entries per task (b block | d block << 4).
    std::map<std::pair<int, int>, std::vector<int>> sps;
    for (int a = 0; a < ns; ++a) sps[{ms[a].two_m, ms[a].parity}].push_back(a);
    const int n_sp = (int)sps.size(), n_s = (int)b->sectors.size();
    t.sp_ptr.assign(1, 0);
    t.ow_of.assign((size_t)n_s * n_sp, -1);
    int cls = 0;
    for (auto &sp : sps) {
        for (int a : sp.second) t.sp_state.push_back(a);
        t.sp_ptr.push_back((int32_t)t.sp_state.size());
        const int nblk = ((int)sp.second.size() + 3) / 4;
        for (int s = 0; s < n_s; ++s) {
            auto it = W.group_of.find({b->two_M - b->sectors[s].two_mp - sp.first.first,
                                       b->parity * b->sectors[s].parity_p * sp.first.second});
            if (it != W.group_of.end()) t.ow_of[(size_t)s * n_sp + cls] = it->second;
        }
        for (int bb = 0; bb < nblk; ++bb)
            for (int db = 0; db < nblk; ++db) {
                const int blk = bb | (db << 4);
                for (int u = 0; u < (int)U.mask.size(); u += kObdCores) t.op_tasks.insert(t.op_tasks.end(), {cls, blk, u});
                for (int s = 0; s < n_s; ++s) {
                    const int w = t.ow_of[(size_t)s * n_sp + cls];
                    if (w < 0) continue;
                    for (int j = 0; j < t.w_n[w]; j += 64)
                        for (int r = 0; r < b->sectors[s].np; r += kObdRows)
                            t.on_tasks.insert(t.on_tasks.end(), {cls, blk, s, j, r});
                }
            }
        ++cls;
    }
    // Tasks of the label densities: about equal shares of the work, each of one
    // class, whose n x n sums a workgroup adds to the result once.
    std::vector<std::pair<int64_t, std::array<int32_t, 3>>> vt;
    int64_t all = 0;
    auto vcost = [&](int u, int p) -> int64_t {
        const int w = t.w_of[(size_t)U.group[u] * t.n_pc + p], nt = (t.pc_n[p] + 15) / 16;
        return w < 0 ? 0 : (int64_t)(t.w_pad[w] + 16) * nt * (nt + 2);
    };
    const int n_u = (int)U.mask.size();
    for (int p = 0; p < t.n_pc; ++p)
        for (int u = 0; u < n_u; ++u) all += vcost(u, p);
    const int64_t share = std::max<int64_t>(all / kCoreVjpTasks, 4096);
    for (int p = 0; p < t.n_pc; ++p) {
        if (t.pc_n[p] > 64) return;
        int64_t c = 0;
        int first = 0;
        for (int u = 0; u < n_u; ++u) {
            c += vcost(u, p);
            if (c >= share || (u + 1 == n_u && c > 0)) {
                vt.push_back({c, {p, first, u + 1}});
                first = u + 1;
                c = 0;
            }
        }
    }
    std::stable_sort(vt.begin(), vt.end(), [](const auto &x, const auto &y) { return x.first > y.first; });
    for (auto &v : vt) t.v_tasks.insert(t.v_tasks.end(), v.second.begin(), v.second.end());
    t.ok = true;
}

void build_pair_tables(fotci_ham *h) {
    const fotci_basis *b = h->j->b;
    const auto &ms = b->ms;
    const int ns = h->j->ns, npairs = h->j->npairs;
    HostPairs &t = h->hp;
    t = HostPairs();
    if (b->p.n < 2 || !h->tt.ok || b->dim * 8 > 0x7ff00000) return;
    std::map<std::pair<int, int>, std::vector<std::pair<int, int>>> cls;
    for (int a = 0; a < ns; ++a)
        for (int c = a + 1; c < ns; ++c) cls[{ms[a].two_m + ms[c].two_m, ms[a].parity * ms[c].parity}].push_back({a, c});
    std::vector<std::pair<int, int>> st;   // the states of every entry of pc_pair
    t.pc_first.assign(1, 0);
    for (auto &c : cls) {
        if ((int)c.second.size() > kPairsMost) return;
        for (auto &p : c.second) {
            t.pc_pair.push_back(pair_index(p.first, p.second, ns));
            t.cls_of.push_back(t.n_pc);
            st.push_back(p);
        }
        t.pc_first.push_back((int32_t)t.pc_pair.size());
        ++t.n_pc;
    }
    std::vector<uint32_t> ts;
    std::vector<std::pair<uint32_t, int32_t>> idx;
    for (size_t i = 0; i < b->p.sd.size(); ++i) {
        const uint32_t m = b->p.sd[i];
        idx.push_back({m, (int32_t)i});
        for (uint32_t r = m; r; r &= r - 1)
            for (uint32_t q = r & (r - 1); q; q &= q - 1) ts.push_back(m & ~(r & (0u - r)) & ~(q & (0u - q)));
    }
    std::sort(ts.begin(), ts.end());
    ts.erase(std::unique(ts.begin(), ts.end()), ts.end());
    std::sort(idx.begin(), idx.end());
    // Multiply-adds of the two forms (the sampled product's in tiles of 32): all
    // densities before and after at shares of 0.35 to 0.88: 8.5 / 7.1 ms (20 states, 5p5n,
    // 0.35), 0.73 / 0.61 (4p4n, 0.54), 4.3 / 4.0 (3p6n, 0.77), 8.1 / 5.9 (18 states, 8p4n, 0.79),
    // 19.0 / 18.7 (5p8n, 0.88). The table stays below 64 MiB.
    int64_t dense = 0, mine = 0;
    for (auto &s : b->sectors) dense += (int64_t)((s.np + 31) / 32 * 32) * ((s.np + 31) / 32 * 32) * s.nn;
    if ((int64_t)ts.size() * npairs * 4 > ((int64_t)64 << 20)) return;
    const int n_t = (int)ts.size();
    std::map<std::pair<int, int>, int> cols;   // columns of the rows of a proton (2M, parity)
    for (auto &s : b->sectors) cols[{s.two_mp, s.parity_p}] = s.nn;
    std::vector<int32_t> nn((size_t)n_t * t.n_pc, 0);
    for (int i = 0; i < n_t; ++i) {
        int tm = 0, par = 1, c = 0;
        for (uint32_t r = ts[i]; r; r &= r - 1) tm += ms[__builtin_ctz(r)].two_m, par *= ms[__builtin_ctz(r)].parity;
        for (auto &q : cls) {
            auto it = cols.find({tm + q.first.first, par * q.first.second});
            if (it != cols.end()) nn[(size_t)i * t.n_pc + c] = it->second;
            ++c;
        }
    }
    auto cost = [&](int i, int c) -> int64_t {
        const int nt = (t.pc_first[c + 1] - t.pc_first[c] + 15) / 16;
        return (int64_t)nn[(size_t)i * t.n_pc + c] * 256 * nt * nt;
    };
    for (int c = 0; c < t.n_pc; ++c)
        for (int i = 0; i < n_t; ++i) mine += cost(i, c);
    if (mine > dense) return;
    std::vector<uint32_t> base((size_t)n_t * npairs, kCoreNoRow);
    for (int i = 0; i < n_t; ++i)
        for (size_t e = 0; e < st.size(); ++e) {
            const uint32_t add = (1u << st[e].first) | (1u << st[e].second);
            if ((ts[i] & add) || nn[(size_t)i * t.n_pc + t.cls_of[e]] == 0) continue;
            auto it = std::lower_bound(idx.begin(), idx.end(), std::make_pair(ts[i] | add, (int32_t)0));
            if (it == idx.end() || it->first != (ts[i] | add)) continue;
            const bool odd = odd_below(ts[i], st[e].first) != odd_below(ts[i], st[e].second);
            base[(size_t)i * npairs + t.pc_pair[e]] = (uint32_t)b->pstart[it->second] | (odd ? 0x80000000u : 0u);
        }
    std::vector<std::pair<int64_t, std::array<int32_t, 3>>> vt;
    const int64_t share = std::max<int64_t>(mine / kPairsTasks, 1 << 16);
    for (int c = 0; c < t.n_pc; ++c) {
        int64_t sum = 0;
        int first = 0;
        for (int i = 0; i < n_t; ++i) {
            sum += cost(i, c);
            if (sum >= share || (i + 1 == n_t && sum > 0)) {
                vt.push_back({sum, {c, first, i + 1}});
                first = i + 1;
                sum = 0;
            }
        }
    }
    std::stable_sort(vt.begin(), vt.end(), [](const auto &x, const auto &y) { return x.first > y.first; });
    for (auto &v : vt) t.tasks.insert(t.tasks.end(), v.second.begin(), v.second.end());
    t.t_base = std::move(base);
    t.t_nn = std::move(nn);
}

void fill_core_values(fotci_ham *h) {
    HostCore &t = h->hc;
    t.v.resize(t.v_src.size());
    for (size_t i = 0; i < t.v.size(); ++i) t.v[i] = h->v_pn[t.v_src[i]];
}

}  // namespace fotci
