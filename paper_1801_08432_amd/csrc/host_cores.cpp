// Host tables of the core kernels: the proton-neutron part of H written with
// one particle of each species taken out and put back,
//   sum_{abcd} V[(a b),(c d)] (p+_a n+_b) (n_d p_c),
// so that x is gathered once per (proton core, neutron core) pair for all the
// pairs (c d) that fill it, one dense matrix V of the pair's (2m, parity)
// turns them into the pairs (a b), and the results are added to y.
#include <algorithm>
#include <array>
#include <cmath>
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

// Masks with a number each (open addressing; a quarter to half full).
class MaskIndex {
  public:
    explicit MaskIndex(size_t most) {
        while (((size_t)1 << bits_) < 2 * most) ++bits_;
        slot_.assign((size_t)1 << bits_, {0, -1});
    }
    // false if the mask is there already
    bool insert(uint32_t m, int32_t v) {
        Slot &s = slot_[at(m)];
        if (s.val >= 0) return false;
        s = {m, v};
        return true;
    }
    int32_t find(uint32_t m) const { return slot_[at(m)].val; }   // -1: none

  private:
    struct Slot {
        uint32_t key;
        int32_t val;
    };
    size_t at(uint32_t m) const {
        size_t i = (m * 0x9e3779b1u) >> (32 - bits_);
        while (slot_[i].val >= 0 && slot_[i].key != m) i = (i + 1) & (slot_.size() - 1);
        return i;
    }
    int bits_ = 4;
    std::vector<Slot> slot_;
};

MaskIndex index_of(const SpeciesBasis &sb) {
    MaskIndex ix(sb.sd.size());
    for (size_t i = 0; i < sb.sd.size(); ++i) ix.insert(sb.sd[i], (int32_t)i);
    return ix;
}

double binomial(int n, int k) {
    double v = 1.0;
    for (int i = 1; i <= k; ++i) v = v * (n - k + i) / i;
    return v;
}

// The SDs with `out` (1 or 2) particles taken out, ascending.
std::vector<uint32_t> taken_out(const SpeciesBasis &sb, int ns, int out) {
    const double each = out == 1 ? sb.n : 0.5 * sb.n * (sb.n - 1);
    MaskIndex seen((size_t)std::min(each * (double)sb.sd.size(), binomial(ns, sb.n - out)));
    std::vector<uint32_t> all;
    auto add = [&](uint32_t m) {
        if (seen.insert(m, 0)) all.push_back(m);
    };
    for (uint32_t m : sb.sd)
        for (uint32_t r = m; r; r &= r - 1) {
            const uint32_t one = m & ~(r & (0u - r));
            if (out == 1) add(one);
            else
                for (uint32_t q = r & (r - 1); q; q &= q - 1) add(one & ~(q & (0u - q)));
        }
    std::sort(all.begin(), all.end());
    return all;
}

std::pair<int, int> two_m_parity(uint32_t m, const std::vector<MState> &ms) {
    int tm = 0, par = 1;
    for (; m; m &= m - 1) tm += ms[__builtin_ctz(m)].two_m, par *= ms[__builtin_ctz(m)].parity;
    return {tm, par};
}

Cores cores_of(const SpeciesBasis &sb, const std::vector<MState> &ms) {
    std::map<std::pair<int, int>, std::vector<uint32_t>> by;
    for (uint32_t m : taken_out(sb, (int)ms.size(), 1)) by[two_m_parity(m, ms)].push_back(m);
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

// The code tables of the other vector sizes, and the work items of the products:
// a core with as many of the states a as a workgroup takes (rows in LDS); the
// costliest start first.
void build_items(HostCore &t, int nu, int ns) {
    const std::vector<uint32_t> &code = t.w_code[3 - kCoreMinShift];
    for (int s = kCoreMinShift; s <= kCoreMaxShift; ++s) {
        if (s == 3) continue;
        auto &c = t.w_code[s - kCoreMinShift];
        c = code;
        for (auto &v : c)
            if (v == core_null(3)) v = core_null(s);
    }
    // states of an item with up to kCoreMaxPairs states b between them, four a position
    static_assert(kCoreMaxPairs / 4 + kCoreStates <= kCoreMaxPos, "positions of an item in a class");
    std::vector<int64_t> cost((size_t)nu, 0);   // of a core's group, per state
    for (int g = 0; g < nu; ++g)
        for (int p = 0; p < t.n_pc; ++p) {
            const int w = t.w_of[(size_t)g * t.n_pc + p];
            if (w >= 0) cost[g] += (int64_t)t.w_pad[w] * t.pc_n[p] + 4096;
        }
    struct It {
        int u;
        uint32_t amask;
        int64_t cost;
    };
    std::vector<It> its;
    for (int u = 0; u < (int)t.u_mask.size(); ++u) {
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
            its.push_back({u, am, cost[t.u_group[u]] * (4 + __builtin_popcount(am))});
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
    std::stable_sort(its.begin(), its.end(), [](const It &x, const It &y) { return x.cost > y.cost; });
    for (auto &i : its) t.items.push_back(i.u), t.items.push_back((int32_t)i.amask);
}

// Tasks of the label densities: about equal shares of the work, each of one
// class, whose n x n sums a workgroup adds to the result once.
void build_label_tasks(HostCore &t, int nu) {
    const int n_u = (int)t.u_mask.size();
    std::vector<std::pair<int64_t, std::array<int32_t, 3>>> vt;
    std::vector<int64_t> cost((size_t)nu * t.n_pc, 0);   // of a core's group in a class
    int64_t all = 0;
    for (int g = 0; g < nu; ++g)
        for (int p = 0; p < t.n_pc; ++p) {
            const int w = t.w_of[(size_t)g * t.n_pc + p], nt = (t.pc_n[p] + 15) / 16;
            if (w >= 0) cost[(size_t)g * t.n_pc + p] = (int64_t)(t.w_pad[w] + 16) * nt * (nt + 2);
        }
    for (int u = 0; u < n_u; ++u)
        for (int p = 0; p < t.n_pc; ++p) all += cost[(size_t)t.u_group[u] * t.n_pc + p];
    const int64_t share = std::max<int64_t>(all / kCoreVjpTasks, 4096);
    for (int p = 0; p < t.n_pc; ++p) {
        int64_t c = 0;
        int first = 0;
        for (int u = 0; u < n_u; ++u) {
            c += cost[(size_t)t.u_group[u] * t.n_pc + p];
            if (c >= share || (u + 1 == n_u && c > 0)) {
                vt.push_back({c, {p, first, u + 1}});
                first = u + 1;
                c = 0;
            }
        }
    }
    std::stable_sort(vt.begin(), vt.end(), [](const auto &x, const auto &y) { return x.first > y.first; });
    for (auto &v : vt) t.v_tasks.insert(t.v_tasks.end(), v.second.begin(), v.second.end());
}

// Whether apply_H of nb vectors runs its pn part on the cores.
//
// The core kernels gather x, per element of y, for Z N pairs, of which a share
// (N_s - N + 1) / N_s of the lanes hits a free state d, once for every group of
// kCoreStates states a; the one-body-jump kernels gather N (N_s - N + 1) rows of
// their contracted tile. Measured times of the two pn parts against the ratio
// of these counts (jumps / cores): float32 2.84 / 1.65 ms at 1.28 (20 states,
// 5p5n), 0.77 / 0.60 at 1.25 (3p6n), 2.14 / 2.48 at 0.78 (18 states, 8p4n), 4.4 /
// 10.3 at 0.67 (5p8n); float64, whose row updates cost the jump kernel more,
// 6.9 / 2.4, 1.85 / 0.78, 3.7 / 2.9 and 10.9 / 12.6. Shells beyond the middle
// fall far below the line (20 states, 15p14n: 0.16). The float32 figure at 0.78 is from
// before the items' set-up was shortened: the whole product takes 2.60 / 2.34 ms
// there since, so that line could lie lower.
//
// With few states a task is a few subtiles and an item costs its set-up, whatever
// it gathers, while the jump kernel pays per row: float64 products also need the
// ratio, divided by the items per row and times the share of a last round of
// workgroups that is not idle, to reach 1.2 (12 / N_s)^3, unless all items run
// at once (the line from 2000 products in spaces of 8 to 20 states, timed both ways: 47 of
// them are left more than 3% slower than by jumps, where the ratio alone left 244;
// 15 lose as much). float32, three workgroups a CU and cheaper registers, goes by the
// ratio. us of a product, jumps / cores, by the quotient: 12 states: 49.8 / 68.6
// at 0.40 (8p4n, blocks of 2), 46.3 / 51.2 at 0.80 (6p5n), 69.8 / 72.1 at 1.0 (4p3n,
// blocks of 4), 80.1 / 72.2 at 1.26 (5p6n, blocks of 2), one round 38.3 / 32.7 (4p4n); 14
// states: 128 / 157 at 0.52 (9p5n), 97 / 114 at 0.63 (6p3n), 130 / 110 at 1.16 (4p5n, blocks
// of 2); 16 states: 503 / 401 at 0.80 (6p4n); 18 states: 4767 / 3821 at 0.54 (8p4n).
bool apply_on_cores(const fotci_ham *h, int mode, int nb) {
    const double ns = h->j->ns, Z = h->j->b->p.n, N = h->j->b->n.n, open = ns - N + 1;
    const double groups = std::ceil((ns - Z + 1) / kCoreStates);
    const double ratio = N * open / (Z * N * ns / open * groups);
    if (ratio < (mode == FOTCI_MODE_F64 ? 0.75 : 1.0)) return false;
    if (mode != FOTCI_MODE_F64) return true;
    const double items = (double)h->hc.u_mask.size() * groups, rows = (double)h->j->b->p.sd.size();
    const double rounds = items * nb / 512.0;   // of four-wave workgroups, two a CU
    return rounds <= 1.0 || ratio * rows / items * (rounds / std::ceil(rounds)) >= 1.2 * std::pow(12.0 / ns, 3);
}

// Per element of g the cores gather Z N pairs, of which a share (N_s - N + 1) /
// N_s of the lanes finds a free state, the jump kernel scatters N (N_s - N + 1)
// entries: measured, all densities, jumps against cores, by the ratio of the
// counts: 17.4 / 10.5 ms at 2.6 (20 states, 5p5n), 0.40 / 0.34 at 0.7 (12 states, 6p6n),
// 7.6 / 29.8 at 0.15 (18 states, 13p13n). Where a row and its tiles exceed the jump
// kernel's LDS, what is left is one LDS atomic per pair of jumps (177 / 23.7 ms, 18
// states, 5p8n).
bool vjp_on_cores(const fotci_ham *h) {
    const double ns = h->j->ns, Z = h->j->b->p.n, N = h->j->b->n.n, open = ns - N + 1;
    return !vjp_pn_jumps(h) || N * open >= 0.6 * (Z * N * ns / open);
}

}  // namespace

// Bytes of work memory: one slot of dim * nb elements per proton.
int64_t apply_work_bytes(const fotci_ham *h, int mode, int nb) {
    if ((mode != FOTCI_MODE_F64 && mode != FOTCI_MODE_F32) || !h->hc.ok || !apply_on_cores(h, mode, nb)) return 0;
    return h->j->b->dim * nb * (mode == FOTCI_MODE_F64 ? 8 : 4) * h->j->b->p.n;
}

// Tables of the proton and neutron cores and of the densities, which every basis
// uses, and those of the products and the label densities where these run on
// the cores (fotci_set_interaction at 14p18n in 20 states, which has neither: 350
// ms with all of them built and searched for in sorted lists, 165 ms so).
void build_core_tables(fotci_ham *h) {
    const fotci_basis *b = h->j->b;
    const auto &ms = b->ms;
    const int ns = h->j->ns;
    HostCore &t = h->hc;
    t = HostCore();
    // rows and columns that do not exist are read past the end of a vector, at
    // 2^31 - 2^20 bytes and above; a code's column shifted must stay below the
    // null code's bit
    if (b->p.n < 1 || b->n.n < 1 || !h->tt.ok || b->dim * 8 > 0x7ff00000 ||
        h->tt.max_nn >= (1 << (31 - kCoreMaxShift)))
        return;
    // pair classes
    std::map<std::pair<int, int>, std::vector<std::pair<int, int>>> pcs;
    for (int a = 0; a < ns; ++a)
        for (int c = 0; c < ns; ++c) pcs[{ms[a].two_m + ms[c].two_m, ms[a].parity * ms[c].parity}].push_back({a, c});
    if ((int)pcs.size() > kCoreMaxPc) return;
    for (auto &pc : pcs)
        if (pc.second.size() > kCoreMaxPairs) return;
    const Cores U = cores_of(b->p, ms), W = cores_of(b->n, ms);
    const int nw = (int)W.count.size(), nu = (int)U.count.size();
    int64_t total = 0;
    for (int g = 0; g < nw; ++g) {
        t.w_n.push_back(W.count[g]);
        t.w_pad.push_back((W.count[g] + 15) & ~15);
        t.w_off.push_back((int32_t)total);
        total += (int64_t)t.w_pad.back() * ns;
        if (total * 4 >= ((int64_t)1 << 30)) return;
    }
    t.w_null = (int)total;   // a run of null codes as long as the largest group
    total += *std::max_element(t.w_pad.begin(), t.w_pad.end());
    if (total * 4 >= ((int64_t)1 << 30)) return;
    t.u_mask = U.mask;
    t.u_group = U.group;
    const MaskIndex pidx = index_of(b->p), nidx = index_of(b->n);
    t.u_nn.assign(U.mask.size() * (size_t)ns, 0);
    t.u_base.assign(U.mask.size() * (size_t)ns, kCoreNoRow);
    for (size_t u = 0; u < U.mask.size(); ++u)
        for (int a = 0; a < ns; ++a) {
            if ((U.mask[u] >> a) & 1u) continue;
            const int ip = pidx.find(U.mask[u] | (1u << a));
            if (ip < 0) continue;
            const uint32_t phase = odd_below(U.mask[u], a) ? 0x80000000u : 0u;
            t.u_nn[u * ns + a] = b->sectors[b->p_basis_sector[ip]].nn;
            t.u_base[u * ns + a] = (uint32_t)b->pstart[ip] | phase;
        }
    // neutron cores: codes, for float64 vectors
    std::vector<uint32_t> &code = t.w_code[3 - kCoreMinShift];
    code.assign((size_t)total, core_null(3));
    for (int g = 0; g < nw; ++g)
        for (int j = 0; j < W.count[g]; ++j) {
            const uint32_t m = W.mask[W.first[g] + j];
            for (int d = 0; d < ns; ++d) {
                if ((m >> d) & 1u) continue;
                const int jn = nidx.find(m | (1u << d));
                if (jn >= 0)
                    code[(size_t)t.w_off[g] + (size_t)d * t.w_pad[g] + j] =
                        (uint32_t)b->n.sd_local[jn] | (odd_below(m, d) ? 0x80000000u : 0u);
            }
        }
    // One-body densities: states by (2m, parity), a block of 4 x 4 of a class's
    // entries per task (b block | d block << 4).
    std::map<std::pair<int, int>, std::vector<int>> sps;
    for (int a = 0; a < ns; ++a) sps[{ms[a].two_m, ms[a].parity}].push_back(a);
    const int n_sp = (int)sps.size(), n_s = (int)b->sectors.size(), n_u = (int)U.mask.size();
    // A wave takes its cores one after another, so one each where there are few; but every task adds to the same
    // entries. Densities in us with tasks of 32 cores, of n_u / 64, of n_u / 128: 68 / 47 / 47 (pf 3p4n, 190 cores), 36 / 35 / 40
    // (pf 4p1n, 1140), 79 / 72 / 71 (pf 4p4n, 1140), 22 / 19 / 19 (j = 7/2 4p4n, 56).
    const int per = std::min(kObdCores, std::max(4, n_u / 64));
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
                for (int u = 0; u < n_u; u += per) t.op_tasks.insert(t.op_tasks.end(), {cls, blk, u, std::min(u + per, n_u)});
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
    t.ok = true;
    for (int mode : {FOTCI_MODE_F32, FOTCI_MODE_F64})
        for (int nb : {1, 2, 4, 8}) t.apply = t.apply || apply_on_cores(h, mode, nb);
    const bool labels = vjp_on_cores(h);
    if (!t.apply && !labels) return;
    // the classes with most pairs first: the tasks of a workgroup are drawn in this order
    const size_t ns2 = (size_t)ns * ns;
    std::vector<std::pair<int, int>> pc_q;
    for (auto &pc : pcs) pc_q.push_back(pc.first);
    std::stable_sort(pc_q.begin(), pc_q.end(), [&](const auto &x, const auto &y) { return pcs[x].size() > pcs[y].size(); });
    for (auto &q : pc_q) {
        const auto &pr = pcs[q];   // by a, then b
        t.pc_n.push_back((int32_t)pr.size());
        t.pc_pair.push_back((int32_t)t.pair_ab.size());
        size_t k = 0;
        for (int a = 0; a <= ns; ++a) {
            while (k < pr.size() && pr[k].first < a) ++k;
            t.pc_first.push_back((int32_t)k);
        }
        for (auto &p : pr) t.pair_ab.push_back(p.first | (p.second << 8));
        if (!t.apply) continue;
        t.pc_v.push_back((int32_t)t.v_src.size());
        for (auto &p : pr)
            for (auto &r : pr)
                t.v_src.push_back((int32_t)(((size_t)p.first * ns + p.second) * ns2 + (size_t)r.first * ns + r.second));
    }
    t.n_pc = (int)t.pc_n.size();
    t.w_of.assign((size_t)nu * t.n_pc, -1);
    for (auto &g : U.group_of)
        for (int k = 0; k < t.n_pc; ++k) {
            auto it = W.group_of.find({b->two_M - g.first.first - pc_q[k].first, b->parity * g.first.second * pc_q[k].second});
            if (it != W.group_of.end()) t.w_of[(size_t)g.second * t.n_pc + k] = it->second;
        }
    if (t.apply) build_items(t, nu, ns);
    if (labels) build_label_tasks(t, nu);
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
    // Multiply-adds of the two forms (the sampled product's in tiles of 32): all
    // densities before and after at shares of 0.35 to 0.88: 8.5 / 7.1 ms (20 states, 5p5n,
    // 0.35), 0.73 / 0.61 (4p4n, 0.54), 4.3 / 4.0 (3p6n, 0.77), 8.1 / 5.9 (18 states, 8p4n, 0.79),
    // 19.0 / 18.7 (5p8n, 0.88).
    // What a t and a class cost is at least 16 per column and row that they have, and every row has (Z over 2)
    // of them: most bases past the middle of the shell end here, without the list of the t.
    int64_t dense = 0, mine = 0;
    for (auto &s : b->sectors) dense += (int64_t)((s.np + 31) / 32 * 32) * ((s.np + 31) / 32 * 32) * s.nn;
    if (16.0 * binomial(b->p.n, 2) * (double)b->dim > (double)dense) return;
    // The table stays below 64 MiB; an SD t is in at most (N_s - Z + 2 over 2) of the SDs that it comes from.
    constexpr int64_t kMost = (int64_t)64 << 20;
    const double least = (double)b->p.sd.size() * binomial(b->p.n, 2) / binomial(ns - b->p.n + 2, 2);
    if (least * npairs * 4 > (double)kMost) return;
    const std::vector<uint32_t> ts = taken_out(b->p, ns, 2);
    if ((int64_t)ts.size() * npairs * 4 > kMost) return;
    const int n_t = (int)ts.size();
    std::map<std::pair<int, int>, int> cols;   // columns of the rows of a proton (2M, parity)
    for (auto &s : b->sectors) cols[{s.two_mp, s.parity_p}] = s.nn;
    std::vector<int32_t> nn((size_t)n_t * t.n_pc, 0);
    std::map<std::pair<int, int>, std::vector<int32_t>> rows;   // of a t's (2M, parity)
    for (int i = 0; i < n_t; ++i) {
        const auto key = two_m_parity(ts[i], ms);
        auto &r = rows[key];
        if (r.empty())
            for (auto &q : cls) {
                auto it = cols.find({key.first + q.first.first, key.second * q.first.second});
                r.push_back(it != cols.end() ? it->second : 0);
            }
        std::copy(r.begin(), r.end(), nn.begin() + (size_t)i * t.n_pc);
    }
    auto cost = [&](int i, int c) -> int64_t {
        const int nt = (t.pc_first[c + 1] - t.pc_first[c] + 15) / 16;
        return (int64_t)nn[(size_t)i * t.n_pc + c] * 256 * nt * nt;
    };
    for (int c = 0; c < t.n_pc; ++c)
        for (int i = 0; i < n_t; ++i) mine += cost(i, c);
    if (mine > dense) return;
    const MaskIndex idx = index_of(b->p);
    std::vector<uint32_t> base((size_t)n_t * npairs, kCoreNoRow);
    for (int i = 0; i < n_t; ++i)
        for (size_t e = 0; e < st.size(); ++e) {
            const uint32_t add = (1u << st[e].first) | (1u << st[e].second);
            if ((ts[i] & add) || nn[(size_t)i * t.n_pc + t.cls_of[e]] == 0) continue;
            const int ip = idx.find(ts[i] | add);
            if (ip < 0) continue;
            const bool odd = odd_below(ts[i], st[e].first) != odd_below(ts[i], st[e].second);
            base[(size_t)i * npairs + t.pc_pair[e]] = (uint32_t)b->pstart[ip] | (odd ? 0x80000000u : 0u);
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
