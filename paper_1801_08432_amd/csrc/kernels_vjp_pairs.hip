// Proton two-body label densities through SDs t with two protons taken out:
//   dV[(a b),(c d)] += sum_t phase <g[t + a + b, :], x[t + c + d, :]>,
// a < b, c < d of one pair class (2m, parity). Per class and t the rows of the
// pairs form two n x nn matrices whose product (columns summed) is taken on the
// float64 matrix cores, its sums staying in registers over the t of a task. The dense product of
// a whole sector (k_vjp_sddmm) does np / n times the multiply-adds; the diagonal
// labels (a b) = (c d) come with the rest. 2.75 -> 1.26 ms at 5p5n in
// 20 states, a third of its matrix-core rate: a fragment's 16 rows are read in 32-byte pieces.
#include <hip/hip_runtime.h>

#include "tiled_common.h"

namespace fotci {

namespace {

constexpr int kVtWaves = 4;

template <int NT>
__device__ __forceinline__ void vt_task(const DevHam &P, const DevPairs &C, int n, int p0, int i0, int i1,
                                        __amdgpu_buffer_rsrc_t xr, __amdgpu_buffer_rsrc_t gr, int wid, int lane,
                                        double *__restrict__ red) {
    const int li = lane & 15, kq = lane >> 4;
    doublex4 acc[NT][NT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = Mma<double>::zero();
    for (int t = i0 + wid; t < i1; t += kVtWaves) {
        unsigned ro[NT];
        uint32_t sg[NT];
        int nn = 0;
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const int p = 16 * i + li;
            const uint32_t rb = p < n ? C.t_base[(int64_t)t * P.npairs + C.pc_pair[p0 + p]] : kCoreNoRow;
            sg[i] = rb & 0x80000000u;
            ro[i] = rb == kCoreNoRow ? kOutOfRange : (rb << 3) + 8u * kq;   // the shift drops the phase
        }
        nn = C.t_nn[(int64_t)t * C.n_pc + C.cls_of[p0]];   // uniform; 0: no row of the class
        auto load = [&](double (&gv)[NT], double (&xv)[NT], int st) {
            // past the row's end: zero
            const unsigned o = 4 * st + kq < nn ? 32u * (unsigned)st : kOutOfRange;
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                gv[i] = buffer_load<double>(gr, ro[i] + o, 0);
                xv[i] = buffer_load<double>(xr, ro[i] + o, 0);
            }
        };
        const int steps = (nn + 3) >> 2;
        if (steps == 0) continue;
        double ga[NT], xa[NT], gb[NT], xb[NT], gc[NT], xc[NT];
        load(ga, xa, 0);
        load(gb, xb, 1);
        auto step = [&](int st, double (&g0)[NT], double (&x0)[NT], double (&g2)[NT], double (&x2)[NT]) {
            load(g2, x2, st + 2);
            double u[NT], v[NT];
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                u[i] = signed_by(g0[i], sg[i]);
                v[i] = signed_by(x0[i], sg[i]);
            }
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[i][j] = Mma<double>::mma(u[i], v[j], acc[i][j]);
        };
        for (int st = 0;; st += 3) {
            step(st, ga, xa, gc, xc);
            if (st + 1 >= steps) break;
            step(st + 1, gb, xb, ga, xa);
            if (st + 2 >= steps) break;
            step(st + 2, gc, xc, gb, xb);
            if (st + 3 >= steps) break;
        }
    }
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                __hip_atomic_fetch_add(&red[(16 * i + Mma<double>::row(lane, r)) * (16 * NT) + 16 * j + li], acc[i][j][r],
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__global__ __launch_bounds__(64 * kVtWaves) void k_vjp_pairs(DevHam P, DevPairs C, const double *__restrict__ x,
                                                             const double *__restrict__ g, double *d_v) {
    __shared__ double red[48 * 48];
    const int32_t *task = C.tasks + 3 * (int64_t)blockIdx.x;
    const int pc = task[0], i0 = task[1], i1 = task[2];
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int p0 = C.pc_first[pc], n = C.pc_first[pc + 1] - p0, nt = (n + 15) >> 4;
    for (int i = tid; i < 48 * 48; i += 64 * kVtWaves) red[i] = 0.0;
    __syncthreads();
    const int bytes = (int)(P.dim * (int64_t)sizeof(double));
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void *)x, (short)0, bytes, kBufFlags);
    const __amdgpu_buffer_rsrc_t gr = __builtin_amdgcn_make_buffer_rsrc((void *)g, (short)0, bytes, kBufFlags);
    switch (nt) {
        case 1: vt_task<1>(P, C, n, p0, i0, i1, xr, gr, wid, lane, red); break;
        case 2: vt_task<2>(P, C, n, p0, i0, i1, xr, gr, wid, lane, red); break;
        default: vt_task<3>(P, C, n, p0, i0, i1, xr, gr, wid, lane, red); break;
    }
    __syncthreads();
    bool again = false;
    for (int i = tid; i < n * n; i += 64 * kVtWaves) {
        const int p = i / n, q = i - p * n;
        const double v = red[p * (16 * nt) + q];
        if (v - v != 0.0) again = true;
        else if (v != 0.0) atomicAdd(&d_v[(int64_t)C.pc_pair[p0 + p] * P.npairs + C.pc_pair[p0 + q]], v);
    }
    // A row that does not exist is a row of zeros above, and 0 times an infinity
    // or NaN is NaN: sums that are not finite are taken again, a wave for each,
    // over the t that both pairs fit.
    if (!__any(again)) return;
    for (int base = 64 * wid; base < n * n; base += 64 * kVtWaves) {
        const int i = min(base + lane, n * n - 1), p = i / n, q = i - p * n;
        const double v = red[p * (16 * nt) + q];
        const int pr = C.pc_pair[p0 + p], pq = C.pc_pair[p0 + q];
        for (uint64_t m = __ballot(v - v != 0.0 && base + lane < n * n); m; m &= m - 1) {
            const int l = __builtin_ctzll(m), rp = __shfl(pr, l, 64), rq = __shfl(pq, l, 64);
            double sum = 0.0;
            for (int t = i0; t < i1; ++t) {
                const uint32_t rb = C.t_base[(int64_t)t * P.npairs + rp], rd = C.t_base[(int64_t)t * P.npairs + rq];
                if (rb == kCoreNoRow || rd == kCoreNoRow) continue;
                const int nn = C.t_nn[(int64_t)t * C.n_pc + pc];
                for (int c = lane; c < nn; c += 64)
                    sum += signed_by(buffer_load<double>(gr, (rb << 3) + 8u * c, 0), rb) *
                           signed_by(buffer_load<double>(xr, (rd << 3) + 8u * c, 0), rd);
            }
            for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
            if (lane == 0) atomicAdd(&d_v[(int64_t)rp * P.npairs + rq], sum);
        }
    }
}

}  // namespace

bool launch_vjp_pairs(const fotci_ham *h, const double *x, const double *g, double *d_v_pp, void *stream) {
    const int n = (int)(h->hp.tasks.size() / 3);
    if (n == 0) return false;
    hipLaunchKernelGGL(k_vjp_pairs, dim3(n), dim3(64 * kVtWaves), 0, (hipStream_t)stream, h->dev, h->dev_pairs, x, g,
                       d_v_pp);
    return true;
}

}  // namespace fotci
