// Proton-neutron label densities through cores (see kernels_pn_cores.hip):
//   dV[(a b),(c d)] += sum over cores u, w of G[(a b)] D[(c d)],
//   G = phase g[u + a, w + b],  D = phase x[u + c, w + d],
// per pair class a product of two n x (cores) matrices on the float64 matrix
// cores with the neutron cores as the summed index. Lane l of a fragment holds
// pair l % 16 of its tile at core l / 16 of a step of four, gathered straight
// into the registers: G and D take the same row offsets and codes, and a step's
// 2 NT gathered fragments feed NT^2 products, whose sums stay in registers for
// all proton cores of a task.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "tiled_common.h"

namespace fotci {

namespace {

constexpr int kVcWaves = 4;

template <int NT>
struct VcStep {
    double g[NT], x[NT];
};

// Sums of the proton cores i0 + wid, i0 + wid + kVcWaves, ... < i1 in class pc.
template <int NT>
__device__ __forceinline__ void vc_task(const DevCore &C, int pc, int n, const int32_t *__restrict__ pab, int i0, int i1,
                                        __amdgpu_buffer_rsrc_t xr, __amdgpu_buffer_rsrc_t gr, __amdgpu_buffer_rsrc_t cr,
                                        int wid, int lane, double *__restrict__ red) {
    const int li = lane & 15, kq = lane >> 4;
    doublex4 acc[NT][NT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = Mma<double>::zero();
    int ps[NT], pd[NT];   // the lane's pair of every tile
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int ab = pab[min(16 * t + li, n - 1)];
        ps[t] = ab & 255;
        pd[t] = ab >> 8;
    }
    for (int u = i0 + wid; u < i1; u += kVcWaves) {
        const int w = C.w_of[(int64_t)C.u_group[u] * C.n_pc + pc];   // uniform
        if (w < 0) continue;
        const int wpad = C.w_pad[w], w0 = C.w_off[w];
        unsigned ro[NT], co[NT];
        uint32_t sg[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const uint32_t rb = C.u_base[(int64_t)u * C.ns + ps[t]];
            const bool ok = 16 * t + li < n && rb != kCoreNoRow;
            sg[t] = rb & 0x80000000u;
            ro[t] = ok ? rb << 3 : kOutOfRange;   // the shift drops the phase
            co[t] = (unsigned)(w0 + pd[t] * wpad + kq) * 4u;
        }
        const int steps = wpad >> 2;
        auto codes = [&](uint32_t (&c)[NT], int st) {
            const unsigned o = 16u * (unsigned)min(st, steps - 1);
#pragma unroll
            for (int t = 0; t < NT; ++t) c[t] = buffer_load_u32(cr, co[t] + o);
        };
        auto load = [&](VcStep<NT> &v, const uint32_t (&c)[NT]) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                v.g[t] = buffer_load<double>(gr, ro[t] + (c[t] << 3), 0);
                v.x[t] = buffer_load<double>(xr, ro[t] + (c[t] << 3), 0);
            }
        };
        uint32_t ca[NT], cb[NT];
        VcStep<NT> a, b;
        codes(ca, 0);
        codes(cb, 1);
        load(a, ca);
        auto step = [&](int st, uint32_t (&c0)[NT], VcStep<NT> &v0, uint32_t (&c1)[NT], VcStep<NT> &v1) {
            load(v1, c1);   // the next step's
            double gv[NT], xv[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                gv[t] = signed_by(v0.g[t], c0[t] ^ sg[t]);
                xv[t] = signed_by(v0.x[t], c0[t] ^ sg[t]);
            }
            codes(c0, st + 2);
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[i][j] = Mma<double>::mma(gv[i], xv[j], acc[i][j]);
        };
        for (int st = 0;; st += 2) {
            step(st, ca, a, cb, b);
            if (st + 1 >= steps) break;
            step(st + 1, cb, b, ca, a);
            if (st + 2 >= steps) break;
        }
    }
    // the waves' sums meet in LDS
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                __hip_atomic_fetch_add(&red[(16 * i + Mma<double>::row(lane, r)) * (16 * NT) + 16 * j + li], acc[i][j][r],
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// One workgroup per task {class, first and last proton core}; two waves per
// SIMD (128 of their registers hold the sums).
__global__ __launch_bounds__(64 * kVcWaves) __attribute__((amdgpu_waves_per_eu(2))) void k_vjp_pn_cores(
    DevHam P, DevCore C, const double *__restrict__ x, const double *__restrict__ g, double *d_v_pn) {
    __shared__ double red[64 * 64];
    const int32_t *task = C.v_tasks + 3 * (int64_t)blockIdx.x;
    const int pc = task[0], i0 = task[1], i1 = task[2];
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = C.pc_n[pc];
    const int32_t *pab = C.pair_ab + C.pc_pair[pc];
    for (int i = tid; i < 64 * 64; i += 64 * kVcWaves) red[i] = 0.0;
    __syncthreads();
    const int bytes = (int)(P.dim * (int64_t)sizeof(double));
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void *)x, (short)0, bytes, kBufFlags);
    const __amdgpu_buffer_rsrc_t gr = __builtin_amdgcn_make_buffer_rsrc((void *)g, (short)0, bytes, kBufFlags);
    const __amdgpu_buffer_rsrc_t cr =
        __builtin_amdgcn_make_buffer_rsrc((void *)C.w_code[3 - kCoreMinShift], (short)0, C.n_w_code * 4, kBufFlags);
    const int nt = (n + 15) >> 4;
    switch (nt) {
        case 1: vc_task<1>(C, pc, n, pab, i0, i1, xr, gr, cr, wid, lane, red); break;
        case 2: vc_task<2>(C, pc, n, pab, i0, i1, xr, gr, cr, wid, lane, red); break;
        case 3: vc_task<3>(C, pc, n, pab, i0, i1, xr, gr, cr, wid, lane, red); break;
        default: vc_task<4>(C, pc, n, pab, i0, i1, xr, gr, cr, wid, lane, red); break;
    }
    __syncthreads();
    const int ns = C.ns;
    const int64_t ns2 = (int64_t)ns * ns;
    auto at = [&](int r, int c) -> int64_t {
        return ((int64_t)(r & 255) * ns + (r >> 8)) * ns2 + (int64_t)(c & 255) * ns + (c >> 8);
    };
    bool again = false;
    for (int i = tid; i < n * n; i += 64 * kVcWaves) {
        const int p = i / n, q = i - p * n;
        const double v = red[p * (16 * nt) + q];
        if (v - v != 0.0) again = true;
        else if (v != 0.0) atomicAdd(&d_v_pn[at(pab[p], pab[q])], v);
    }
    // A state that does not fit its core is a zero above, and 0 times an
    // infinity or NaN is NaN: sums that are not finite are taken again, a wave
    // for each, over the cores that both pairs fit. (A loop of its own: within
    // the one above it took the adjoint at pf 2p2n from 98 to 103 us.)
    if (!__any(again)) return;
    for (int base = 64 * wid; base < n * n; base += 64 * kVcWaves) {
        const int i = min(base + lane, n * n - 1), p = i / n, q = i - p * n;
        const double v = red[p * (16 * nt) + q];
        const int ab = pab[p], cd = pab[q];
        for (uint64_t m = __ballot(v - v != 0.0 && base + lane < n * n); m; m &= m - 1) {
            const int l = __builtin_ctzll(m), r = __shfl(ab, l, 64), c = __shfl(cd, l, 64);
            double sum = 0.0;
            for (int u = i0; u < i1; ++u) {
                const int w = C.w_of[(int64_t)C.u_group[u] * C.n_pc + pc];
                const uint32_t rb = C.u_base[(int64_t)u * ns + (r & 255)], rd = C.u_base[(int64_t)u * ns + (c & 255)];
                if (w < 0 || rb == kCoreNoRow || rd == kCoreNoRow) continue;
                const int wpad = C.w_pad[w];
                const uint32_t *code = C.w_code[3 - kCoreMinShift] + C.w_off[w];
                for (int j = lane; j < wpad; j += 64) {
                    const uint32_t vb = code[(r >> 8) * wpad + j], vd = code[(c >> 8) * wpad + j];
                    if (max(vb & 0x7fffffffu, vd & 0x7fffffffu) >= core_null(3)) continue;
                    sum += signed_by(buffer_load<double>(gr, (rb << 3) + (vb << 3), 0), rb ^ vb) *
                           signed_by(buffer_load<double>(xr, (rd << 3) + (vd << 3), 0), rd ^ vd);
                }
            }
            for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
            if (lane == 0) atomicAdd(&d_v_pn[at(r, c)], sum);
        }
    }
}

}  // namespace

bool launch_vjp_cores(const fotci_ham *h, const double *x, const double *g, double *d_v_pn, void *stream) {
    const int n = (int)(h->hc.v_tasks.size() / 3);
    if (n == 0) return false;
    hipLaunchKernelGGL(k_vjp_pn_cores, dim3(n), dim3(64 * kVcWaves), 0, (hipStream_t)stream, h->dev, h->dev_core, x, g,
                       d_v_pn);
    return true;
}

}  // namespace fotci
