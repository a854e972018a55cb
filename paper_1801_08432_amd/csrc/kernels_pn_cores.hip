// Proton-neutron part of apply_H through cores (SDs with one particle of a
// species taken out), for gfx950:
//
//   D[(c d)] = phase x[u + c, w + d]        proton core u, neutron core w
//   E[(a b)] = sum_(c d) V[(a b),(c d)] D[(c d)]
//   y[u + a, w + b] += phase E[(a b)]
//
// over the pairs (c d), (a b) of the one pair class whose (2m, parity) completes
// those of u and w. x is gathered Z N times per element of y where the
// one-body-jump form (k_pn, k_pn2) gathers its contracted tile N (N_s - N + 1)
// times, and the dense matrices cover the pairs of a class (1.8 to 2.4 times the
// useful multiply-adds in 20 states) instead of the labels of an operator class
// (6.2 times). pn part at 5p5n in 20 states, dim 18.6 M: float32 2.84 -> 1.57 ms,
// float64 6.90 -> 2.34 ms (4p4n: 0.377 -> 0.184 and 0.662 -> 0.260 ms). What bounds it (float32):
// 0.2 ms to set up and write out the items, one workgroup per CU, 0.3 ms to
// load the operands of the tasks, and subtiles that issue 31% of the time to the
// vector and 34% to the matrix units. With parts taken out, when the whole took
// 1.64 ms (0.25 of it set-up): 1.49 without the loads of x and its codes, 1.35
// without the matrix instructions.
#include "tiled_common.h"

namespace fotci {

namespace {

constexpr int kCoreTiles = 2;                  // 16-row tiles of (a b) pairs per pass
constexpr int kCorePos = 4 * kCoreTiles;       // positions (a with up to four of its b) per pass
constexpr int kCoreSlots = 56;                 // (c d) pairs per pass: 14 k-steps, three waves per SIMD
constexpr int kCoreRowShift = 3;               // bytes of an LDS row element, log2
constexpr int kCoreSub = 12;                   // 16-core subtiles per task

// Matrix row i of a tile: lane group g and accumulator element r that hold it.
template <typename T>
__device__ __forceinline__ int core_g(int i) { return sizeof(T) == 4 ? i >> 2 : i & 3; }
template <typename T>
__device__ __forceinline__ int core_r(int i) { return sizeof(T) == 4 ? i & 3 : i >> 2; }

// What a workgroup keeps in LDS about its item (dynamic LDS: rows, scratch
// words, then the lists).
struct CoreLds {
    double *yl;              // rows, then one scratch word per thread
    const uint32_t *kl;      // (c d) pairs whose row exists, by class: c | d << 5 | pair << 10
    const uint32_t *ml;      // [n_pc][kCoreMaxPos] positions: a | first pair << 5 | pairs << 20
    const uint32_t *xo;      // [32] byte offset of row u + c
    const uint32_t *ps;      // [32] bit 31: phase of the state added to u
    const int32_t *yo;       // [32] LDS row of u + a
};

// One pass of one wave: nm positions x nk pairs over the 16-core subtiles
// [s0, s1) of a neutron core group. x of the next subtile and the codes of the
// one after it are in flight while a subtile is worked on. Results are added to
// the rows with LDS float64 atomics (8 cycles a wave on gfx950, where a float32
// atomic takes 192 and a read and write 10), also in float32, where the waves'
// order shows in the last bit of the float64 sum at most, and only if a row
// element's addends span 29 binary orders or more: float32 products are the same
// bits from run to run almost always, but not by construction.
template <typename T, int KST>
__device__ __forceinline__ void core_pass(const CoreLds &S, const uint32_t *kl, const uint32_t *ml, int nk, int nm, int n,
                                          unsigned pv, const int32_t *pab, unsigned wbytes, int wpad, int s0,
                                          int s1, unsigned null_off, int shift, __amdgpu_buffer_rsrc_t xr,
                                          __amdgpu_buffer_rsrc_t cr, __amdgpu_buffer_rsrc_t dr,
                                          __amdgpu_buffer_rsrc_t vr, int lane, unsigned own) {
    typedef typename Mma<T>::acc_t acc_t;
    constexpr int TM = kCoreTiles;
    const int li = lane & 15, g = lane >> 4;
    unsigned xo[KST], co[KST];
    T cv[TM][KST];
    uint32_t mp[TM];   // the position of this lane's matrix row
#pragma unroll
    for (int t = 0; t < TM; ++t) {
        const int pos = 4 * t + core_g<T>(li), r = core_r<T>(li);
        const uint32_t m = ml[min(pos, nm - 1)];
        const bool live = pos < nm && r < (int)(m >> 20);
        // operand element's offset in a row of V, and its phase
        mp[t] = live ? (((m >> 5) & 0x7fffu) + r) | (S.ps[m & 31]) : 0x7fffu;
    }
#pragma unroll
    for (int ks = 0; ks < KST; ++ks) {
        const int k = 4 * ks + g;
        const bool ok = k < nk;
        const uint32_t e = kl[min(k, nk - 1)];
        xo[ks] = ok ? S.xo[e & 31] : kOutOfRange;
        co[ks] = wbytes + ((e >> 5) & 31) * (unsigned)(4 * wpad) + 4u * li;
        const unsigned row = pv + (e >> 10) * (unsigned)n;
        const uint32_t sg = S.ps[e & 31];
#pragma unroll
        for (int t = 0; t < TM; ++t) {
            // V is symmetric: the 16 lanes of a group read neighbouring elements of row (c d)
            const bool live = ok && (mp[t] & 0x7fffffffu) != 0x7fffu;
            const T v = buffer_load<T>(vr, live ? (row + (mp[t] & 0x7fffu)) * (unsigned)sizeof(T) : kOutOfRange, 0);
            cv[t][ks] = signed_by(v, sg ^ mp[t]);
        }
    }
    unsigned dco[TM][4], yo[TM];   // codes' offsets (null codes where the position has no pair), row's LDS byte address
#pragma unroll
    for (int t = 0; t < TM; ++t) {
        const int pos = 4 * t + g;
        const uint32_t m = ml[min(pos, nm - 1)];
        const int np = pos < nm ? (int)(m >> 20) : 0;
        yo[t] = (unsigned)S.yo[m & 31] * 8u;
        const int p0 = (m >> 5) & 0x7fff, last = p0 + (int)(m >> 20) - 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const unsigned b = (unsigned)(pab[min(p0 + r, last)] >> 8) * (unsigned)(4 * wpad);
            dco[t][r] = (r < np ? wbytes + b : null_off) + 4u * li;
        }
    }
    T xa[KST], xb[KST];
    auto loadc = [&](uint32_t (&c)[KST], int sub) {
        // up to two subtiles past the last: other codes of the table, whose x is not used
        const unsigned o = 64u * (unsigned)sub;
#pragma unroll
        for (int k = 0; k < KST; ++k) c[k] = buffer_load_u32(cr, co[k] + o);
    };
    auto update = [&](int sub, const uint32_t (&dc)[TM][4], const acc_t (&acc)[TM]) {
#pragma unroll
        for (int t = 0; t < TM; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // the shift drops the phase; a null code lands past every row
                const unsigned at = min(yo[t] + (dc[t][r] << 3), own);
                double *p = reinterpret_cast<double *>(reinterpret_cast<char *>(S.yl) + at);
                __hip_atomic_fetch_add(p, (double)signed_by(acc[t][r], dc[t][r]), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            }
    };
    auto loadd = [&](uint32_t (&dc)[TM][4], int sub) {
#pragma unroll
        for (int t = 0; t < TM; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                dc[t][r] = buffer_load_u32(dr, dco[t][r] + 64u * sub);
    };
    uint32_t ca[KST], cb[KST];
    auto loadx = [&](T (&v)[KST], const uint32_t (&c)[KST]) {
#pragma unroll
        for (int k = 0; k < KST; ++k) v[k] = buffer_load<T>(xr, xo[k] + (c[k] << shift), 0);
    };
    loadc(ca, s0);
    loadc(cb, s0 + 1);
    loadx(xa, ca);
    auto step = [&](int sub, uint32_t (&c0)[KST], T (&x0)[KST], uint32_t (&c1)[KST], T (&x1)[KST]) {
        uint32_t dc[TM][4];
        loadd(dc, sub);
        loadx(x1, c1);
        acc_t acc[TM];
#pragma unroll
        for (int t = 0; t < TM; ++t) acc[t] = Mma<T>::zero();
#pragma unroll
        for (int ks = 0; ks < KST; ++ks) {
            const T v = signed_by(x0[ks], c0[ks]);
#pragma unroll
            for (int t = 0; t < TM; ++t) acc[t] = Mma<T>::mma(cv[t][ks], v, acc[t]);
        }
        loadc(c0, sub + 2);
        update(sub, dc, acc);
    };
    for (int sub = s0;; sub += 2) {
        step(sub, ca, xa, cb, xb);
        if (sub + 1 >= s1) break;
        step(sub + 1, cb, xb, ca, xa);
        if (sub + 2 >= s1) break;
    }
}

template <typename T>
struct CoreV;
template <>
struct CoreV<float> {
    static __device__ __forceinline__ const float *v(const DevCore &c) { return c.v32; }
};
template <>
struct CoreV<double> {
    static __device__ __forceinline__ const double *v(const DevCore &c) { return c.v64; }
};

// As many waves as the registers of a CU hold (three or two per SIMD).
template <typename T>
constexpr int core_threads() { return sizeof(T) == 4 ? 768 : 512; }

// One workgroup per item: a proton core and up to kCoreStates states a that can
// be added to it, whose rows it sums in LDS. Its waves draw tasks (a pair class
// and up to kCoreSub subtiles of its neutron core group, costly classes first)
// from a counter in LDS and run free of each other. The item's contribution to
// row u + a goes to slot k of `slots` ([Z][dim * vectors]) when a is the row's
// k-th particle, so every slot row is written once and the sum over the slots
// (in the nn kernel) has a fixed order.
template <typename T>
__global__ __launch_bounds__(core_threads<T>()) void k_pn_core(DevHam P, DevCore C, const int32_t *__restrict__ items,
                                                          int n_items, int lognb, int ycols, const T *__restrict__ x,
                                                          T *__restrict__ slots) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ uint32_t s_xo[32], s_ps[32], s_base[32];
    __shared__ int32_t s_yo[32], s_nn[32], s_pp[kCoreMaxPc];
    __shared__ int s_task[kCoreMaxPc + 1], s_w[kCoreMaxPc];
    __shared__ int s_nk[kCoreMaxPc], s_np[kCoreMaxPc], s_next;
    const int NT = blockDim.x;
    const int nb = 1 << lognb;
    int slot = blockIdx.x, g0 = 0;
    if (lognb) {   // the workgroups of one item's vectors are consecutive slots of one XCD
        const int xcd = blockIdx.x & 7, s8 = blockIdx.x >> 3;
        slot = (s8 >> lognb) * 8 + xcd;
        g0 = s8 & (nb - 1);
        if (slot >= n_items) return;   // uniform
    }
    constexpr int es = sizeof(T) == 4 ? 2 : 3;
    const int shift = es + lognb;
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int u = items[2 * slot];
    const uint32_t amask = (uint32_t)items[2 * slot + 1];
    const int ns = C.ns, npc = C.n_pc;
    CoreLds S;
    S.yl = reinterpret_cast<double *>(smem_raw);
    uint32_t *kl = reinterpret_cast<uint32_t *>(S.yl + ycols + NT);   // [ns * ns]
    uint32_t *ml = kl + ns * ns;                                      // [npc * kCoreMaxPos]
    // the pair tables, so that the lists below are built without a load
    int32_t *s_pair = reinterpret_cast<int32_t *>(ml + npc * kCoreMaxPos);   // [ns * ns]
    int32_t *s_first = s_pair + ns * ns;                                     // [npc * (ns + 1)]
    for (int i = tid; i < ns * ns; i += NT) s_pair[i] = C.pair_ab[i];
    for (int i = tid; i < npc * (ns + 1); i += NT) s_first[i] = C.pc_first[i];
    for (int i = tid; i < npc; i += NT) s_pp[i] = C.pc_pair[i];
    S.kl = kl;
    S.ml = ml;
    S.xo = s_xo;
    S.ps = s_ps;
    S.yo = s_yo;
    if (wid == 0) {
        const int a = lane & 31;
        const uint32_t rb = a < ns ? C.u_base[(int64_t)u * ns + a] : kCoreNoRow;
        const int rn = a < ns ? C.u_nn[(int64_t)u * ns + a] : 0;
        const unsigned xo = (((rb & 0x7fffffffu) << lognb) + g0) << es;
        // rows of the item's states, one after another
        const int mine = (amask >> a) & 1u ? rn : 0;
        int nn = mine;
        for (int o = 1; o < 32; o <<= 1) {
            const int v = __shfl_up(nn, o, 32);
            if (a >= o) nn += v;
        }
        if (lane < 32) {
            s_base[a] = rb;
            s_ps[a] = rb & 0x80000000u;
            s_xo[a] = rb == kCoreNoRow ? kOutOfRange : xo;
            s_nn[a] = rn;
            s_yo[a] = nn - mine;
        }
    } else if (wid == 1) {
        // neutron core group of every class, and the running count of tasks
        const int32_t *w_of = C.w_of + (int64_t)C.u_group[u] * npc;
        int run = 0;
        for (int p0 = 0; p0 < npc; p0 += 64) {
            const int pc = p0 + lane;
            const int w = pc < npc ? w_of[pc] : -1;
            const int nt = w < 0 ? 0 : ((C.w_pad[max(w, 0)] >> 4) + kCoreSub - 1) / kCoreSub;
            int sum = nt;
            for (int o = 1; o < 64; o <<= 1) {
                const int v = __shfl_up(sum, o, 64);
                if (lane >= o) sum += v;
            }
            if (pc < npc) {
                s_w[pc] = w;
                s_task[pc] = run + sum - nt;
            }
            run += __shfl(sum, 63, 64);
        }
        if (lane == 0) {
            s_task[npc] = run;
            s_next = 0;
        }
    }
    for (int c = tid; c < ycols + NT; c += NT) S.yl[c] = 0.0;
    __syncthreads();
    const uint64_t below = (1ull << lane) - 1ull;
    for (int pc = wid; pc < npc; pc += NT / 64) {
        if (s_w[pc] < 0) continue;   // uniform per wave
        const int pp = s_pp[pc], n = s_first[pc * (ns + 1) + ns];
        int nk = 0;
        for (int p = lane; p - lane < n; p += 64) {
            const int ab = s_pair[pp + min(p, n - 1)];
            const int c = ab & 255;
            const bool ok = p < n && s_base[c] != kCoreNoRow;
            const uint64_t km = __ballot(ok);
            if (ok) kl[pp + nk + __popcll(km & below)] = (uint32_t)c | ((uint32_t)(ab >> 8) << 5) | ((uint32_t)p << 10);
            nk += __popcll(km);
        }
        // positions: every state a of the item with four of its states b at a time
        int f0 = 0, nba = 0;
        if (lane < ns && ((amask >> lane) & 1u)) {
            f0 = s_first[pc * (ns + 1) + lane];
            nba = s_first[pc * (ns + 1) + lane + 1] - f0;
        }
        int np = 0;
        for (int lev = 0;; ++lev) {
            const uint64_t am = __ballot(nba > 4 * lev);
            if (!am) break;
            if (nba > 4 * lev)
                ml[pc * kCoreMaxPos + np + __popcll(am & below)] =
                    (uint32_t)lane | ((uint32_t)(f0 + 4 * lev) << 5) | ((uint32_t)min(nba - 4 * lev, 4) << 20);
            np += __popcll(am);
        }
        if (lane == 0) {
            s_nk[pc] = nk;
            s_np[pc] = np;
        }
    }
    __syncthreads();
    const __amdgpu_buffer_rsrc_t xr =
        __builtin_amdgcn_make_buffer_rsrc((void *)x, (short)0, (int)(P.dim << shift), kBufFlags);
    const __amdgpu_buffer_rsrc_t cr = __builtin_amdgcn_make_buffer_rsrc((void *)C.w_code[shift - kCoreMinShift], (short)0,
                                                                        C.n_w_code * 4, kBufFlags);
    const __amdgpu_buffer_rsrc_t vr =
        __builtin_amdgcn_make_buffer_rsrc((void *)CoreV<T>::v(C), (short)0, C.n_v * (int)sizeof(T), kBufFlags);
    const __amdgpu_buffer_rsrc_t dr = __builtin_amdgcn_make_buffer_rsrc(
        (void *)C.w_code[kCoreRowShift - kCoreMinShift], (short)0, C.n_w_code * 4, kBufFlags);
    const unsigned null_off = (unsigned)C.w_null * 4u, own = (unsigned)(ycols + tid) * 8u;
    const int n_task = s_task[npc];
    for (;;) {
        int task = 0;
        if (lane == 0) task = atomicAdd(&s_next, 1);
        task = __builtin_amdgcn_readfirstlane(task);
        if (task >= n_task) break;   // the counter only grows: every wave gets here
        int pc = 0;
        for (int p0 = 0; p0 < npc; p0 += 64) {   // last class whose first task is not after this one
            const int p = p0 + lane;
            pc += __popcll(__ballot(p < npc && s_task[min(p, npc)] <= task));
        }
        pc = __builtin_amdgcn_readfirstlane(pc - 1);
        const int w = __builtin_amdgcn_readfirstlane(s_w[pc]);
        const int nk = __builtin_amdgcn_readfirstlane(s_nk[pc]), np = __builtin_amdgcn_readfirstlane(s_np[pc]);
        const int s0 = (task - __builtin_amdgcn_readfirstlane(s_task[pc])) * kCoreSub;
        const int pp = __builtin_amdgcn_readfirstlane(s_pp[pc]);
        const int wpad = C.w_pad[w], n = C.pc_n[pc];
        const unsigned wbytes = (unsigned)C.w_off[w] * 4u, pv = (unsigned)C.pc_v[pc];
        const int s1 = min(s0 + kCoreSub, wpad >> 4);
        const int32_t *pab = s_pair + pp;
        for (int m0 = 0; m0 < np; m0 += kCorePos)
            for (int k0 = 0; k0 < nk; k0 += kCoreSlots) {
                const int nm = min(np - m0, kCorePos), kk = min(nk - k0, kCoreSlots);
                const uint32_t *kp = kl + pp + k0, *mp = ml + pc * kCoreMaxPos + m0;
#define FOTCI_CORE_CASE(K)                                                                                            \
    case K:                                                                                                           \
        core_pass<T, 2 * K>(S, kp, mp, kk, nm, n, pv, pab, wbytes, wpad, s0, s1, null_off, shift, xr, cr, dr, vr, lane, \
                           own); \
        break;
                switch ((kk + 7) >> 3) {
                    FOTCI_CORE_CASE(1)
                    FOTCI_CORE_CASE(2)
                    FOTCI_CORE_CASE(3)
                    FOTCI_CORE_CASE(4)
                    FOTCI_CORE_CASE(5)
                    FOTCI_CORE_CASE(6)
                    default:
                    FOTCI_CORE_CASE(7)
                }
#undef FOTCI_CORE_CASE
            }
    }
    __syncthreads();
    const uint32_t um = C.u_mask[u];
    for (uint32_t m = amask; m; m &= m - 1) {
        const int a = __builtin_ctz(m);
        const int64_t base = s_base[a] & 0x7fffffffu;
        const int k = __builtin_popcount(um & ((1u << a) - 1u));
        T *out = slots + (((int64_t)k * P.dim + base) << lognb) + g0;
        const int nn = s_nn[a], o = s_yo[a];
        for (int c = tid; c < nn; c += NT) out[(int64_t)c << lognb] = (T)S.yl[o + c];
    }
}

template <typename T>
void launch_cores(const fotci_ham *h, int nb, const T *x, T *slots, hipStream_t st) {
    const HostCore &hc = h->hc;
    const int lognb = nb == 8 ? 3 : nb == 4 ? 2 : nb == 2 ? 1 : 0;
    const int n = (int)(hc.items.size() / 2);
    const unsigned grid = nb == 1 ? (unsigned)n : (unsigned)((n + 7) / 8 * 8 * nb);
    const int ns = h->j->ns;
    auto bytes = [&](int threads) {
        return ((size_t)hc.item_cols + threads) * 8 + ((size_t)2 * ns * ns + (size_t)hc.n_pc * (kCoreMaxPos + ns + 1)) * 4;
    };
    // Workgroups of four waves where their rows leave room for as many of them
    // as the registers do (three float32, two float64), else one of all the
    // waves a CU takes: small sectors have few tasks per item (pn part at 4p4n in
    // 20 states, four waves against all: float32 0.184 / 0.253 ms, float64 0.260 /
    // 0.310; 3p4n, float32 0.049 / 0.063).
    constexpr int kMost = core_threads<T>();
    const int threads = bytes(256) * (kMost / 256) <= 156 * 1024 ? 256 : kMost;
    hipLaunchKernelGGL(k_pn_core<T>, dim3(grid), dim3(threads), bytes(threads), st, h->dev, h->dev_core, h->dev_core.items,
                       n, lognb, hc.item_cols, x, slots);
}

}  // namespace

void launch_pn_cores(const fotci_ham *h, int mode, int nb, const void *x, void *slots, void *stream) {
    if (mode == FOTCI_MODE_F64)
        launch_cores<double>(h, nb, (const double *)x, (double *)slots, (hipStream_t)stream);
    else
        launch_cores<float>(h, nb, (const float *)x, (float *)slots, (hipStream_t)stream);
    hip_check(hipGetLastError(), "pn core launch");
}

}  // namespace fotci
