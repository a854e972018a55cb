// Tables of the core kernels (host_cores.cpp) under AddressSanitizer and
// UndefinedBehaviorSanitizer, without device code: the sums that the kernels
// take over them, carried out here, against the operators applied determinant
// by determinant; every row in one work item, every task range in its table;
// and no tables where neither products nor label densities run on the cores.
// Build and run: tests/test_host_core_sanitizers.py.
#include <cmath>
#include <cstdio>
#include <map>
#include <random>
#include <set>

#include "fotci_internal.h"

namespace fotci {
struct Thrown {
    int code;
    std::string msg;
};
[[noreturn]] void fail(int code, const std::string &msg) { throw Thrown{code, msg}; }
void set_error(const std::string &) {}
}  // namespace fotci

extern "C" int fotci_build_basis_impl(int32_t, const int32_t *, const int32_t *, int32_t, int32_t, int32_t, int32_t,
                                      fotci_basis **);

using namespace fotci;

static int n_fail = 0;
#define CHECK(c)                                                                          \
    do {                                                                                  \
        if (!(c)) {                                                                       \
            std::fprintf(stderr, "CHECK failed line %d (%s): %s\n", __LINE__, label, #c); \
            if (++n_fail > 20) std::exit(1);                                              \
        }                                                                                 \
    } while (0)

static bool odd_below(uint32_t m, int i) { return __builtin_popcount(m & ((1u << i) - 1u)) & 1; }

// p+_a p_c m; the sign, 0 where it vanishes
static int hop(uint32_t m, int a, int c, uint32_t &out) {
    if (!((m >> c) & 1u)) return 0;
    const uint32_t r = m ^ (1u << c);
    if ((r >> a) & 1u) return 0;
    out = r | (1u << a);
    return odd_below(r, c) != odd_below(r, a) ? -1 : 1;
}

struct Shape {
    const char *label;
    std::vector<int32_t> two_j, parity;
    int Z, N, two_M;
    bool products, labels;   // on the cores
};

static void check(const Shape &sh) {
    const char *label = sh.label;
    fotci_basis *b = nullptr;
    fotci_build_basis_impl((int32_t)sh.two_j.size(), sh.two_j.data(), sh.parity.data(), sh.Z, sh.N, sh.two_M, 1, &b);
    fotci_jumps j;
    j.b = b;
    const int ns = j.ns = (int)b->ms.size();
    const int npairs = j.npairs = ns * (ns - 1) / 2;
    fotci_ham h;
    h.j = &j;
    for (auto &s : b->sectors) h.tt.max_nn = std::max(h.tt.max_nn, s.nn);
    h.tt.ok = true;
    std::mt19937_64 rng(7);
    std::normal_distribution<double> normal;
    const size_t ns2 = (size_t)ns * ns;
    h.v_pn.assign(ns2 * ns2, 0.0);
    auto cls = [&](size_t ab) {
        const auto &p = b->ms[ab / ns], &n = b->ms[ab % ns];
        return std::make_pair(p.two_m + n.two_m, p.parity * n.parity);
    };
    for (size_t r = 0; r < ns2; ++r)
        for (size_t c = 0; c <= r; ++c)
            if (cls(r) == cls(c)) h.v_pn[r * ns2 + c] = h.v_pn[c * ns2 + r] = normal(rng);
    build_core_tables(&h);
    build_pair_tables(&h);
    fill_core_values(&h);
    const HostCore &t = h.hc;
    CHECK(t.ok);
    CHECK(t.apply == sh.products && t.items.empty() == !sh.products && t.v_src.empty() == !sh.products);
    CHECK(t.v_tasks.empty() == !sh.labels);
    for (int s = kCoreMinShift; s <= kCoreMaxShift; ++s)
        CHECK(t.w_code[s - kCoreMinShift].empty() == (s != 3 && !sh.products));
    for (int mode : {FOTCI_MODE_F32, FOTCI_MODE_F64})
        for (int nb : {1, 2, 4, 8}) CHECK(apply_work_bytes(&h, mode, nb) == 0 || t.apply);

    std::map<uint32_t, int> pi, ni;
    for (size_t i = 0; i < b->p.sd.size(); ++i) pi[b->p.sd[i]] = (int)i;
    for (size_t i = 0; i < b->n.sd.size(); ++i) ni[b->n.sd[i]] = (int)i;
    std::map<int, int> sector_of;   // neutron species sector -> basis sector
    for (size_t s = 0; s < b->sectors.size(); ++s) sector_of[b->sectors[s].n_sector] = (int)s;
    auto at = [&](uint32_t pm, uint32_t nm) -> int64_t {   // -1: not in the basis
        auto p = pi.find(pm), n = ni.find(nm);
        if (p == pi.end() || n == ni.end()) return -1;
        auto s = sector_of.find(b->n.sd_sector[n->second]);
        if (s == sector_of.end() || s->second != b->p_basis_sector[p->second]) return -1;
        return b->pstart[p->second] + b->n.sd_local[n->second];
    };
    std::vector<double> x((size_t)b->dim), g((size_t)b->dim);
    for (auto &v : x) v = normal(rng);
    for (auto &v : g) v = normal(rng);
    std::vector<double> y((size_t)b->dim, 0.0), dv(ns2 * ns2, 0.0), rp(ns2, 0.0), rn(ns2, 0.0);
    std::vector<double> dpp((size_t)npairs * npairs, 0.0);
    for (uint32_t pm : b->p.sd)
        for (uint32_t nm : b->n.sd) {
            const int64_t i = at(pm, nm);
            if (i < 0) continue;
            for (int c = 0; c < ns; ++c)
                for (int a = 0; a < ns; ++a) {
                    uint32_t p2 = 0, n2 = 0;
                    const int sp = hop(pm, a, c, p2), sn = hop(nm, a, c, n2);
                    int64_t k;
                    if (sp && (k = at(p2, nm)) >= 0) rp[(size_t)a * ns + c] += sp * g[k] * x[i];
                    if (sn && (k = at(pm, n2)) >= 0) rn[(size_t)a * ns + c] += sn * g[k] * x[i];
                    if (!sp) continue;
                    for (int d = 0; d < ns; ++d)
                        for (int e = 0; e < ns; ++e) {
                            const int s2 = hop(nm, e, d, n2);
                            if (!s2 || (k = at(p2, n2)) < 0) continue;
                            const size_t r = (size_t)a * ns + e, q = (size_t)c * ns + d;
                            y[k] += sp * s2 * h.v_pn[r * ns2 + q] * x[i];
                            dv[r * ns2 + q] += sp * s2 * g[k] * x[i];
                        }
                }
            for (int c = 0; c < ns; ++c)
                for (int d = c + 1; d < ns; ++d) {
                    if (!((pm >> c) & 1u) || !((pm >> d) & 1u)) continue;
                    const uint32_t r = pm & ~(1u << c) & ~(1u << d);
                    for (int a = 0; a < ns; ++a)
                        for (int e = a + 1; e < ns; ++e) {
                            if (((r >> a) & 1u) || ((r >> e) & 1u)) continue;
                            const int64_t k = at(r | (1u << a) | (1u << e), nm);
                            const bool odd = (odd_below(r, c) != odd_below(r, d)) != (odd_below(r, a) != odd_below(r, e));
                            if (k >= 0)
                                dpp[(size_t)pair_index(a, e, ns) * npairs + pair_index(c, d, ns)] += (odd ? -1 : 1) * g[k] * x[i];
                        }
                }
        }
    auto close = [](const std::vector<double> &a, const std::vector<double> &r) {
        double e = 0.0, n = 0.0;
        for (size_t i = 0; i < a.size(); ++i) e += (a[i] - r[i]) * (a[i] - r[i]), n += r[i] * r[i];
        return std::sqrt(e) <= 1e-12 * std::max(std::sqrt(n), 1.0);
    };
    auto sgn = [](uint32_t c) { return c >> 31 ? -1.0 : 1.0; };
    // element u + a, w + core j + d of a vector as the kernels address it, in bytes of 8; 0 past its end
    const auto &code = t.w_code[3 - kCoreMinShift];
    auto load = [&](const std::vector<double> &v, int u, int a, uint32_t c) {
        const uint32_t rb = t.u_base[(size_t)u * ns + a];
        const uint32_t off = (rb == kCoreNoRow ? 0x7ff00000u : rb << 3) + (c << 3);
        return off < (uint64_t)b->dim * 8 ? v[off / 8] * (rb == kCoreNoRow ? 1.0 : sgn(rb)) * sgn(c) : 0.0;
    };
    const int n_u = (int)t.u_mask.size();
    if (sh.products) {
        std::set<std::pair<int, int>> seen;
        std::vector<double> got((size_t)b->dim, 0.0);
        for (size_t it = 0; it < t.items.size(); it += 2) {
            const int u = t.items[it];
            const uint32_t am = (uint32_t)t.items[it + 1];
            int cols = 0;
            for (int a = 0; a < ns; ++a)
                if ((am >> a) & 1u) {
                    CHECK(seen.insert({u, a}).second && t.u_base[(size_t)u * ns + a] != kCoreNoRow);
                    cols += t.u_nn[(size_t)u * ns + a];
                }
            CHECK(__builtin_popcount(am) <= kCoreStates && cols <= t.item_cols && cols <= kCoreRowElems);
            for (int p = 0; p < t.n_pc; ++p) {
                const int w = t.w_of[(size_t)t.u_group[u] * t.n_pc + p];
                if (w < 0) continue;
                const int n = t.pc_n[p], wpad = t.w_pad[w];
                for (int jn = 0; jn < wpad; ++jn)
                    for (int r = 0; r < n; ++r) {
                        const int ab = t.pair_ab[t.pc_pair[p] + r];
                        const uint32_t cb = code[(size_t)t.w_off[w] + (size_t)(ab >> 8) * wpad + jn];
                        if (!((am >> (ab & 255)) & 1u) || (cb & 0x7fffffffu) == core_null(3)) continue;
                        double e = 0.0;
                        for (int q = 0; q < n; ++q) {
                            const int cd = t.pair_ab[t.pc_pair[p] + q];
                            e += t.v[t.pc_v[p] + r * n + q] *
                                 load(x, u, cd & 255, code[(size_t)t.w_off[w] + (size_t)(cd >> 8) * wpad + jn]);
                        }
                        const uint32_t rb = t.u_base[(size_t)u * ns + (ab & 255)];
                        CHECK((int)(cb & 0x7fffffffu) < t.u_nn[(size_t)u * ns + (ab & 255)]);
                        got[(rb & 0x7fffffffu) + (cb & 0x7fffffffu)] += sgn(rb) * sgn(cb) * e;
                    }
            }
        }
        size_t rows = 0;
        for (uint32_t rb : t.u_base) rows += rb != kCoreNoRow;
        CHECK(rows == seen.size() && rows == b->p.sd.size() * (size_t)sh.Z);
        CHECK(close(got, y));
        for (int s = kCoreMinShift; s <= kCoreMaxShift; ++s)
            for (size_t i = 0; i < code.size(); ++i) {
                const uint32_t c = t.w_code[s - kCoreMinShift][i];
                CHECK((code[i] & 0x7fffffffu) == core_null(3) ? c << s == 0x80000000u : c == code[i]);
            }
        for (int i = t.w_null; i < (int)code.size(); ++i) CHECK(code[i] == core_null(3));
    }
    if (sh.labels) {
        std::vector<double> got(ns2 * ns2, 0.0);
        std::vector<int> last(t.n_pc, 0);
        for (size_t k = 0; k < t.v_tasks.size(); k += 3) {
            const int p = t.v_tasks[k], n = t.pc_n[p];
            CHECK(t.v_tasks[k + 1] >= 0 && t.v_tasks[k + 1] < t.v_tasks[k + 2] && t.v_tasks[k + 2] <= n_u);
            for (int u = t.v_tasks[k + 1]; u < t.v_tasks[k + 2]; ++u) {
                const int w = t.w_of[(size_t)t.u_group[u] * t.n_pc + p];
                if (w < 0) continue;
                for (int jn = 0; jn < t.w_pad[w]; ++jn)
                    for (int r = 0; r < n; ++r)
                        for (int q = 0; q < n; ++q) {
                            const int ab = t.pair_ab[t.pc_pair[p] + r], cd = t.pair_ab[t.pc_pair[p] + q];
                            auto c = [&](int st) { return code[(size_t)t.w_off[w] + (size_t)st * t.w_pad[w] + jn]; };
                            got[((size_t)(ab & 255) * ns + (ab >> 8)) * ns2 + (size_t)(cd & 255) * ns + (cd >> 8)] +=
                                load(g, u, ab & 255, c(ab >> 8)) * load(x, u, cd & 255, c(cd >> 8));
                        }
            }
        }
        CHECK(close(got, dv));
    }
    // one-body densities: every core once a class and block
    std::map<std::pair<int, int>, int> next;
    for (size_t k = 0; k < t.op_tasks.size(); k += 4) {
        int &from = next[{t.op_tasks[k], t.op_tasks[k + 1]}];
        CHECK(t.op_tasks[k + 2] == from && t.op_tasks[k + 3] > from && t.op_tasks[k + 3] - from <= kObdCores);
        from = t.op_tasks[k + 3];
    }
    for (auto &n : next) CHECK(n.second == n_u);
    std::vector<double> gp(ns2, 0.0), gn(ns2, 0.0);
    const int n_sp = (int)t.sp_ptr.size() - 1;
    auto state = [&](int c, int i) { return t.sp_ptr[c] + i < t.sp_ptr[c + 1] ? t.sp_state[t.sp_ptr[c] + i] : -1; };
    for (size_t k = 0; k < t.op_tasks.size(); k += 4)
        for (int u = t.op_tasks[k + 2]; u < t.op_tasks[k + 3]; ++u)
            for (int i = 0; i < 4; ++i)
                for (int jj = 0; jj < 4; ++jj) {
                    const int bb = state(t.op_tasks[k], 4 * (t.op_tasks[k + 1] & 15) + i);
                    const int dd = state(t.op_tasks[k], 4 * (t.op_tasks[k + 1] >> 4) + jj);
                    if (bb < 0 || dd < 0 || t.u_base[(size_t)u * ns + bb] == kCoreNoRow) continue;
                    for (int c = 0; c < t.u_nn[(size_t)u * ns + bb]; ++c)
                        gp[(size_t)bb * ns + dd] += load(g, u, bb, (uint32_t)c) * load(x, u, dd, (uint32_t)c);
                }
    for (size_t k = 0; k < t.on_tasks.size(); k += 5) {
        const int *tk = &t.on_tasks[k];
        const auto &s = b->sectors[tk[2]];
        const int w = t.ow_of[(size_t)tk[2] * n_sp + tk[0]];
        CHECK(w >= 0 && tk[3] < t.w_n[w] && tk[4] < s.np);
        for (int jn = tk[3]; jn < std::min(tk[3] + 64, t.w_pad[w]); ++jn)
            for (int i = 0; i < 4; ++i)
                for (int jj = 0; jj < 4; ++jj) {
                    const int bb = state(tk[0], 4 * (tk[1] & 15) + i), dd = state(tk[0], 4 * (tk[1] >> 4) + jj);
                    if (bb < 0 || dd < 0) continue;
                    const uint32_t cb = code[(size_t)t.w_off[w] + (size_t)bb * t.w_pad[w] + jn];
                    const uint32_t cd = code[(size_t)t.w_off[w] + (size_t)dd * t.w_pad[w] + jn];
                    if (((cb | cd) & 0x7fffffffu) >= core_null(3)) continue;
                    for (int r = tk[4]; r < std::min(tk[4] + kObdRows, s.np); ++r) {
                        const int64_t row = s.offset + (int64_t)r * s.nn;
                        gn[(size_t)bb * ns + dd] +=
                            sgn(cb ^ cd) * g[row + (cb & 0x7fffffffu)] * x[row + (cd & 0x7fffffffu)];
                    }
                }
    }
    for (size_t a = 0; a < ns2; ++a)   // only pairs of one (2m, parity)
        if (b->ms[a / ns].two_m != b->ms[a % ns].two_m || b->ms[a / ns].parity != b->ms[a % ns].parity) rp[a] = rn[a] = 0.0;
    CHECK(close(gp, rp) && close(gn, rn));
    // proton pairs
    const HostPairs &hp = h.hp;
    if (!hp.tasks.empty()) {
        std::vector<double> got((size_t)npairs * npairs, 0.0);
        for (size_t k = 0; k < hp.tasks.size(); k += 3)
            for (int i = hp.tasks[k + 1]; i < hp.tasks[k + 2]; ++i)
                for (int r = hp.pc_first[hp.tasks[k]]; r < hp.pc_first[hp.tasks[k] + 1]; ++r)
                    for (int q = hp.pc_first[hp.tasks[k]]; q < hp.pc_first[hp.tasks[k] + 1]; ++q) {
                        CHECK(hp.cls_of[r] == hp.tasks[k]);
                        const uint32_t rb = hp.t_base[(size_t)i * npairs + hp.pc_pair[r]];
                        const uint32_t rd = hp.t_base[(size_t)i * npairs + hp.pc_pair[q]];
                        if (rb == kCoreNoRow || rd == kCoreNoRow) continue;
                        for (int c = 0; c < hp.t_nn[(size_t)i * hp.n_pc + hp.tasks[k]]; ++c)
                            got[(size_t)hp.pc_pair[r] * npairs + hp.pc_pair[q]] +=
                                sgn(rb ^ rd) * g[(rb & 0x7fffffffu) + c] * x[(rd & 0x7fffffffu) + c];
                    }
        CHECK(close(got, dpp));
    }
    std::printf("%s: dim %lld, pairs %s\n", label, (long long)b->dim, hp.tasks.empty() ? "no" : "yes");
    delete b;
}

int main() {
    const Shape shapes[] = {
        {"sd 2p3n", {1, 3, 5}, {1, 1, 1}, 2, 3, 1, true, true},
        {"one proton", {1, 3, 5, 7}, {1, 1, 1, 1}, 1, 2, 1, true, true},
        {"one neutron", {1, 3, 5, 7}, {1, 1, 1, 1}, 2, 1, 1, true, true},
        {"two items a core", {1, 3, 5}, {1, 1, 1}, 3, 2, 1, true, true},
        {"two parities", {1, 3, 1, 5}, {-1, -1, 1, 1}, 3, 2, 1, true, true},
        {"five states of one m", {1, 1, 1, 1, 1}, {1, 1, 1, 1, 1}, 2, 2, 0, true, true},
        {"nearly full", {1, 3, 5}, {1, 1, 1}, 10, 10, 0, false, false},
        {"full", {1, 3, 5}, {1, 1, 1}, 12, 12, 0, false, false},
        {"labels alone", {9}, {1}, 2, 6, 0, false, true},
    };
    for (const Shape &s : shapes) check(s);
    std::printf("%d failed\n", n_fail);
    return n_fail != 0;
}
