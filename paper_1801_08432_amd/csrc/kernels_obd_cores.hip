// One-body densities through cores (SDs with one particle taken out, see
// kernels_pn_cores.hip): with a and c of one (2m, parity),
//   rho_p[a, c] = sum_u phase <g[u + a, :], x[u + c, :]>,
//   rho_n[b, d] = sum_w phase sum_r g[r, w + b] x[r, w + d],
// so a block of 4 x 4 entries takes eight loads per element pair (u, column) or
// (row, w) and its sums stay in registers; a row dot per jump reads 2 for one.
// A state that does not fit a core loads zeros, and 0 times an infinity or NaN
// of its partner is NaN: a task whose sum is not finite takes it again over the
// cores that both states fit. (Leaving those products out of the loops
// themselves took 0.66 ms at pf 5p5n instead of 0.64.)
#include <hip/hip_runtime.h>

#include "tiled_common.h"

namespace fotci {

namespace {

constexpr int kOcThreads = 256, kOcWaves = kOcThreads / 64;

// Adds the workgroup's 4 x 4 sums to rho; b, d: states of this block's rows and
// columns (-1: none). each(b, d): one entry's sum over the cores that both
// states fit, a share per lane of one wave (the others are gone by then: a
// second barrier for them took 104 us at pf 4p4n, which is short workgroups,
// instead of 79).
template <typename F>
__device__ __forceinline__ void oc_finish(double (&acc)[4][4], const int (&b)[4], const int (&d)[4], int ns, int lane,
                                          int wid, double (*lds)[16], double *rho, F each) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            double v = acc[i][j];
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
            if (lane == 0) lds[wid][4 * i + j] = v;
        }
    __syncthreads();
    if (wid != 0) return;
    bool again = false;
    int at = 0;
    if (lane < 16) {
        double v = 0.0;
        for (int w = 0; w < kOcWaves; ++w) v += lds[w][lane];
        const int i = lane >> 2, j = lane & 3;
        const int bi = i == 0 ? b[0] : i == 1 ? b[1] : i == 2 ? b[2] : b[3];
        const int dj = j == 0 ? d[0] : j == 1 ? d[1] : j == 2 ? d[2] : d[3];
        if (bi >= 0 && dj >= 0) {
            at = bi * ns + dj;
            again = v - v != 0.0;
            if (!again) atomicAdd(&rho[at], v);
        }
    }
    for (uint64_t m = __ballot(again); m; m &= m - 1) {
        const int e = __shfl(at, __builtin_ctzll(m), 64);
        double v = each(e / ns, e % ns);
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if (lane == 0) atomicAdd(&rho[e], v);
    }
}

__device__ __forceinline__ void oc_states(const DevCore &C, int cls, int blk, int (&b)[4], int (&d)[4]) {
    const int s0 = C.sp_ptr[cls], s1 = C.sp_ptr[cls + 1];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int ib = s0 + 4 * (blk & 15) + i, id = s0 + 4 * (blk >> 4) + i;
        b[i] = ib < s1 ? C.sp_state[ib] : -1;
        d[i] = id < s1 ? C.sp_state[id] : -1;
    }
}

// task {class, block, first, end proton core}: the waves take the cores in turn
__global__ __launch_bounds__(kOcThreads) void k_obd_p(DevHam P, DevCore C, const double *__restrict__ x,
                                                      const double *__restrict__ g, double *rho) {
    __shared__ double lds[kOcWaves][16];
    const int32_t *t = C.op_tasks + 4 * (int64_t)blockIdx.x;
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int b[4], d[4];
    oc_states(C, t[0], t[1], b, d);
    const int bytes = (int)(P.dim * (int64_t)sizeof(double));
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void *)x, (short)0, bytes, kBufFlags);
    const __amdgpu_buffer_rsrc_t gr = __builtin_amdgcn_make_buffer_rsrc((void *)g, (short)0, bytes, kBufFlags);
    double acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = 0.0;
    const int u1 = t[3];
    for (int u = t[2] + wid; u < u1; u += kOcWaves) {
        // rows of the states, all in one sector: their common length
        uint32_t rb[4], rd[4];
        int nn = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            rb[i] = b[i] < 0 ? kCoreNoRow : C.u_base[(int64_t)u * C.ns + b[i]];
            rd[i] = d[i] < 0 ? kCoreNoRow : C.u_base[(int64_t)u * C.ns + d[i]];
            if (rb[i] != kCoreNoRow) nn = C.u_nn[(int64_t)u * C.ns + b[i]];
        }
        // the phases of u + a are the core's: the sign goes onto the loaded value
        unsigned ob[4], od[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ob[i] = rb[i] == kCoreNoRow ? kOutOfRange : rb[i] << 3;
            od[i] = rd[i] == kCoreNoRow ? kOutOfRange : rd[i] << 3;
        }
#pragma unroll 2
        for (int c = lane; c < nn; c += 64) {
            double gv[4], xv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                gv[i] = signed_by(buffer_load<double>(gr, ob[i] + 8u * c, 0), rb[i]);
                xv[i] = signed_by(buffer_load<double>(xr, od[i] + 8u * c, 0), rd[i]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] += gv[i] * xv[j];
        }
    }
    oc_finish(acc, b, d, C.ns, lane, wid, lds, rho, [&](int bi, int dj) {
        double sum = 0.0;
        for (int u = t[2]; u < u1; ++u) {
            const uint32_t rb = C.u_base[(int64_t)u * C.ns + bi], rd = C.u_base[(int64_t)u * C.ns + dj];
            if (rb == kCoreNoRow || rd == kCoreNoRow) continue;
            const int nn = C.u_nn[(int64_t)u * C.ns + bi];
            for (int c = lane; c < nn; c += 64)
                sum += signed_by(buffer_load<double>(gr, (rb << 3) + 8u * c, 0), rb) *
                       signed_by(buffer_load<double>(xr, (rd << 3) + 8u * c, 0), rd);
        }
        return sum;
    });
}

// task {class, block, basis sector, first core of the neutron group, first
// row}: a lane per core, kObdRows rows, a quarter to each wave
__global__ __launch_bounds__(kOcThreads) void k_obd_n(DevHam P, DevCore C, const double *__restrict__ x,
                                                      const double *__restrict__ g, double *rho) {
    __shared__ double lds[kOcWaves][16];
    const int32_t *t = C.on_tasks + 5 * (int64_t)blockIdx.x;
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cls = t[0], s = t[2], r0 = t[4];
    int b[4], d[4];
    oc_states(C, cls, t[1], b, d);
    const int w = C.ow_of[s * C.n_sp + cls];
    const int wpad = C.w_pad[w], j = t[3] + lane;
    const uint32_t *code = C.w_code[3 - kCoreMinShift] + C.w_off[w];
    const int np = P.sec_np[s], nn = P.sec_nn[s];
    const int64_t base = P.sec_off[s];
    const int bytes = (int)(P.dim * (int64_t)sizeof(double));
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void *)x, (short)0, bytes, kBufFlags);
    const __amdgpu_buffer_rsrc_t gr = __builtin_amdgcn_make_buffer_rsrc((void *)g, (short)0, bytes, kBufFlags);
    uint32_t cb[4], cd[4];
    double acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        cb[i] = b[i] >= 0 && j < wpad ? code[b[i] * wpad + j] : core_null(3);
        cd[i] = d[i] >= 0 && j < wpad ? code[d[i] * wpad + j] : core_null(3);
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[i][k] = 0.0;
    }
    const int ra = r0 + wid * (kObdRows / kOcWaves), re = min(ra + kObdRows / kOcWaves, np);
#pragma unroll 2
    for (int r = ra; r < re; ++r) {
        const unsigned ro = (unsigned)(base + (int64_t)r * nn) * 8u;
        double gv[4], xv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            gv[i] = buffer_load<double>(gr, ro + (cb[i] << 3), 0);
            xv[i] = buffer_load<double>(xr, ro + (cd[i] << 3), 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[i][k] += gv[i] * xv[k];
    }
    // a lane's phases are the same in every row
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[i][k] = signed_by(acc[i][k], cb[i] ^ cd[k]);
    oc_finish(acc, b, d, C.ns, lane, wid, lds, rho, [&](int bi, int dj) {
        double sum = 0.0;
        const uint32_t vb = j < wpad ? code[bi * wpad + j] : core_null(3), vd = j < wpad ? code[dj * wpad + j] : core_null(3);
        if (max(vb & 0x7fffffffu, vd & 0x7fffffffu) >= core_null(3)) return sum;
        for (int r = r0; r < min(r0 + kObdRows, np); ++r) {
            const unsigned ro = (unsigned)(base + (int64_t)r * nn) * 8u;
            sum += buffer_load<double>(gr, ro + (vb << 3), 0) * buffer_load<double>(xr, ro + (vd << 3), 0);
        }
        return signed_by(sum, vb ^ vd);
    });
}

}  // namespace

void launch_obd_cores(const fotci_ham *h, const double *g, const double *x, double *rho_p, double *rho_n, void *stream) {
    const int np = (int)(h->hc.op_tasks.size() / 4), nn = (int)(h->hc.on_tasks.size() / 5);
    if (rho_p && np)
        hipLaunchKernelGGL(k_obd_p, dim3(np), dim3(kOcThreads), 0, (hipStream_t)stream, h->dev, h->dev_core, x, g, rho_p);
    if (rho_n && nn)
        hipLaunchKernelGGL(k_obd_n, dim3(nn), dim3(kOcThreads), 0, (hipStream_t)stream, h->dev, h->dev_core, x, g, rho_n);
}

}  // namespace fotci
