// pic_moments.hip -- node moments of one species (reading R27), on demand for pic_diag.
//
// Per node j the cloud-in-cell shares S_j of the particles give W_j = sum S_j,
// sum S_j v (three components) and sum S_j |v|^2, accumulated in FP64; a second kernel
// turns them into the number density n_j = w W_j / V_j, the mean velocity
// u_j = sum S_j v / W_j and the temperature T_j = (m/3)(sum S_j |v|^2 / W_j - |u_j|^2).
// These are the plasma profiles (density, flow, temperature per species) whose
// time-averaged output the paper's input table switches on and whose in-situ plots its
// results section shows.
//
// Accumulation: a block takes tiles of 2048 consecutive slots, eight to a thread as two runs
// of four.  Once sorted, a tile's particles sit in a few cells, so the block adds its shares
// into an LDS window over the tile's node span and flushes each touched node with one HBM
// FP64 atomic per quantity; a tile spanning more than the window (unsorted slots, a sparse
// region) adds straight to HBM.  FP64 atomics make the last bits order-dependent, which
// the moments' tolerance (rel 1e-4) does not see.
//
// What bounds it: LDS atomics of many lanes on the few nodes of a sorted tile, which the LDS
// takes one after another.  So a thread first merges its particles of equal cell, and the
// window holds one copy of a node per group of lanes: kMomWin slots shared out as copies x
// nodes, as many copies (a power of two, up to one per lane) as the tile's span leaves room
// for.  Lanes of one node then hit consecutive words.
#include <algorithm>

#include "pic_device.h"
#include "pic_kernels.h"
#include "pic_particle.h"

namespace pic {

constexpr int kMomThreads = 256;
constexpr int kMomRun = 4;    // consecutive slots per load
constexpr int kMomPpt = 8;
constexpr int kMomTile = kMomThreads * kMomPpt;
constexpr int kMomWin = 512;  // LDS window: nodes x copies
constexpr int kMomQ = 5;      // W, W vx, W vy, W vz, W |v|^2

// kMomRun consecutive slots from i (alive ones counted up to `end`).
template <bool F64>
__device__ __forceinline__ void mom_load(const Dev &d, const SegC &S, int b, int64_t i, int64_t end,
                                         int (&cell)[kMomRun], double (&f)[kMomRun], double (&v)[kMomRun][3])
{
    if constexpr (!F64) {
        int c[kMomRun];
        float o[kMomRun], w[3][kMomRun];
        if (i + kMomRun <= end) {
            // whole runs as 16-byte vectors: i is a multiple of kMomRun, the arrays are 256-byte aligned
            *(int4 *)c = *(const int4 *)(d.cell[b] + i);
            *(float4 *)o = *(const float4 *)(d.off[b] + i);
            *(float4 *)w[0] = *(const float4 *)(d.fvx[b] + i);
            *(float4 *)w[1] = *(const float4 *)(d.fvy[b] + i);
            *(float4 *)w[2] = *(const float4 *)(d.fvz[b] + i);
        } else {
#pragma unroll
            for (int k = 0; k < kMomRun; ++k) {
                const bool in = i + k < end;
                c[k] = in ? d.cell[b][i + k] : kDead;
                o[k] = in ? d.off[b][i + k] : 0.f;
                w[0][k] = in ? d.fvx[b][i + k] : 0.f;
                w[1][k] = in ? d.fvy[b][i + k] : 0.f;
                w[2][k] = in ? d.fvz[b][i + k] : 0.f;
            }
        }
#pragma unroll
        for (int k = 0; k < kMomRun; ++k) {
            cell[k] = c[k] == kDead ? -1 : c[k];
            f[k] = (double)o[k];
#pragma unroll
            for (int a = 0; a < 3; ++a) v[k][a] = (double)w[a][k];
        }
    } else {
        double x[kMomRun];
#pragma unroll
        for (int k = 0; k < kMomRun; ++k) {
            const bool in = i + k < end;
            x[k] = in ? d.x[b][i + k] : -1.0;
            v[k][0] = in ? d.dvx[b][i + k] : 0.0;
            v[k][1] = in ? d.dvy[b][i + k] : 0.0;
            v[k][2] = in ? d.dvz[b][i + k] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < kMomRun; ++k) {
            f[k] = 0.0;
            cell[k] = x[k] >= 0.0 ? (int)cell_of_x(S, x[k], f[k]) : -1;
        }
    }
}

// acc: [kMomQ][nn] of this segment's ensemble, zeroed by the caller.  On the sheath slab ten
// steps after its load (2e7 particles of a species, 1e5 cells) it takes 117 us, 3.4 TB/s of the
// 20 B a particle read; with one atomic per particle, node and quantity on a single copy of
// each node it took 711 us.
template <bool F64>
__global__ void __launch_bounds__(kMomThreads) k_moments(Dev d, int sg, double *acc, int64_t nn)
{
    __shared__ double s_acc[kMomQ][kMomWin];
    __shared__ int s_lo[kMomThreads / kWave], s_hi[kMomThreads / kWave];
    const SegC S = d.seg[sg];
    const int b = *d.cur;
    const int64_t end = S.base + d.n_slots[sg];
    const int lane = lane_id();
    for (int64_t t0 = S.base + (int64_t)blockIdx.x * kMomTile; t0 < end; t0 += (int64_t)gridDim.x * kMomTile) {
        int cell[kMomPpt / kMomRun][kMomRun];
        double f[kMomPpt / kMomRun][kMomRun], v[kMomPpt / kMomRun][kMomRun][3];
        int lo = INT32_MAX, hi = INT32_MIN;
#pragma unroll
        for (int g = 0; g < kMomPpt / kMomRun; ++g)
            mom_load<F64>(d, S, b, t0 + ((int64_t)g * kMomThreads + threadIdx.x) * kMomRun, end, cell[g], f[g], v[g]);
#pragma unroll
        for (int g = 0; g < kMomPpt / kMomRun; ++g)
#pragma unroll
            for (int k = 0; k < kMomRun; ++k)
                if (cell[g][k] >= 0) {
                    lo = min(lo, cell[g][k]);
                    hi = max(hi, cell[g][k]);
                }
        lo = wave_min_i32(lo);
        hi = wave_max_i32(hi);
        if (lane == 0) {
            s_lo[threadIdx.x / kWave] = lo;
            s_hi[threadIdx.x / kWave] = hi;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kMomThreads / kWave; ++w) {
            lo = min(lo, s_lo[w]);
            hi = max(hi, s_hi[w]);
        }
        // nodes lo .. hi + 1 of the tile (node N of a periodic grid is node 0)
        const int span = (lo <= hi) ? hi - lo + 2 : 0;
        const bool in_lds = span > 0 && span <= kMomWin;
        // copies of each node: the largest power of two that fits, at most one per lane
        const int ls = in_lds ? min(31 - __clz(kMomWin / span), 6) : 0;
        const int copies = 1 << ls, copy = lane & (copies - 1);
        if (in_lds) {
            for (int i = threadIdx.x; i < span * copies; i += kMomThreads)
#pragma unroll
                for (int q = 0; q < kMomQ; ++q) s_acc[q][i] = 0.0;
        }
        __syncthreads();
        // one run of equal cell: its shares of the left and the right node
        auto emit = [&](int c, const double (&L)[kMomQ], const double (&R)[kMomQ]) {
            if (in_lds) {
                const int i = ((c - lo) << ls) + copy;
#pragma unroll
                for (int q = 0; q < kMomQ; ++q) {
                    unsafeAtomicAdd(&s_acc[q][i], L[q]);
                    unsafeAtomicAdd(&s_acc[q][i + copies], R[q]);
                }
            } else {
                const int j1 = (S.periodic && c + 1 == S.ncells) ? 0 : c + 1;
#pragma unroll
                for (int q = 0; q < kMomQ; ++q) {
                    unsafeAtomicAdd(acc + (int64_t)q * nn + c, L[q]);
                    unsafeAtomicAdd(acc + (int64_t)q * nn + j1, R[q]);
                }
            }
        };
#pragma unroll
        for (int g = 0; g < kMomPpt / kMomRun; ++g) {
            int rc = -1;
            double L[kMomQ] = {0, 0, 0, 0, 0}, R[kMomQ] = {0, 0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k < kMomRun; ++k) {
                const int c = cell[g][k];
                if (c >= 0 && c != rc) {
                    if (rc >= 0) emit(rc, L, R);
                    rc = c;
#pragma unroll
                    for (int q = 0; q < kMomQ; ++q) L[q] = R[q] = 0.0;
                }
                const double *u = v[g][k];
                const double val[kMomQ] = {1.0, u[0], u[1], u[2], u[0] * u[0] + u[1] * u[1] + u[2] * u[2]};
                const double r = f[g][k], l = 1.0 - r;
                if (c >= 0) {
#pragma unroll
                    for (int q = 0; q < kMomQ; ++q) {
                        L[q] += l * val[q];
                        R[q] += r * val[q];
                    }
                }
            }
            if (rc >= 0) emit(rc, L, R);
        }
        __syncthreads();
        if (in_lds) {
            // one thread per node and quantity sums the copies, starting at its own offset so
            // that the lanes of a wave read different banks
            for (int i = threadIdx.x; i < span * kMomQ; i += kMomThreads) {
                const int q = i / span, n = i - q * span;
                double a = 0.0;
                for (int r = 0; r < copies; ++r) a += s_acc[q][(n << ls) + ((r + lane) & (copies - 1))];
                if (a == 0.0) continue;
                int j = lo + n;
                if (S.periodic && j == S.ncells) j = 0;
                unsafeAtomicAdd(acc + (int64_t)q * nn + j, a);
            }
        }
        __syncthreads();
    }
}

// Sums -> (n, ux, uy, uz, T) in place, node by node.
__global__ void k_moments_finish(Dev d, int sg, double *acc, int64_t nn)
{
    const SegC S = d.seg[sg];
    const EnsC e = d.ens[S.ens];
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < nn; j += (int64_t)gridDim.x * blockDim.x) {
        const double W = acc[j];
        double u[3] = {0.0, 0.0, 0.0}, T = 0.0;
        if (W > 0.0) {
#pragma unroll
            for (int k = 0; k < 3; ++k) u[k] = acc[(int64_t)(1 + k) * nn + j] / W;
            T = (S.m / 3.0) * (acc[4 * nn + j] / W - (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]));
        }
        const double V = (!e.periodic && (j == 0 || j == e.ncells)) ? 0.5 * e.dx : e.dx;
        acc[j] = S.w * W / V;
#pragma unroll
        for (int k = 0; k < 3; ++k) acc[(int64_t)(1 + k) * nn + j] = u[k];
        acc[4 * nn + j] = T;
    }
}

__global__ void k_fill_zero(double *p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.0;
}

hipError_t launch_moments(const Dev &d, bool f64, int sg, int64_t nn, double *out, hipStream_t s)
{
    const int64_t n5 = (int64_t)kMomQ * nn;
    hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)std::min<int64_t>((n5 + 255) / 256, 4096)), dim3(256), 0, s,
                       out, n5);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const unsigned grid = 4096;  // grid-stride over the segment's tiles
    if (f64)
        hipLaunchKernelGGL(k_moments<true>, dim3(grid), dim3(kMomThreads), 0, s, d, sg, out, nn);
    else
        hipLaunchKernelGGL(k_moments<false>, dim3(grid), dim3(kMomThreads), 0, s, d, sg, out, nn);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_moments_finish, dim3((unsigned)std::min<int64_t>((nn + 255) / 256, 4096)), dim3(256), 0,
                       s, d, sg, out, nn);
    return hipGetLastError();
}

}  // namespace pic
