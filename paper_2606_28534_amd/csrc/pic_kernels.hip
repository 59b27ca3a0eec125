// pic_kernels.hip -- gfx950 kernels of the electrostatic 1D3V PIC Monte Carlo step.
//
// This file holds the field solve, the birth ranking and placement, particle loading,
// diagnostics, the scans of the sort, and the FP64 sort scatter; the FP32 cell+offset pass
// and sort are in pic_pass32.hip, the FP64 (plain x, v) pass in pic_pass64.hip.
#include <type_traits>

#include "pic.h"
#include "pic_device.h"
#include "pic_kernels.h"
#include "pic_particle.h"
#include "pic_solve.h"

namespace pic {

// =======================================================================================
// Tile scheduling of the FP64 sort scatter: live tiles are enumerated over all segments and
// block b takes a contiguous run of them.  Blocks are dispatched round-robin over the 8 XCDs,
// so block b is mapped to run (b % 8) * (G / 8) + b / 8: each XCD gets one contiguous eighth
// of the particles (and of the cells, once sorted), which keeps its L2 working set to its
// own part of the grid.
// =======================================================================================
constexpr int kMaxSeg = 512;

__device__ __forceinline__ void sched_prefix(const Dev &d, int64_t tile, int64_t *s_tpre,
                                             int64_t *s_lim = nullptr)
{
    // s_tpre[i] = sum over segments < i of ceil(n_slots / tile); nseg <= kMaxSeg.  With
    // s_lim, also each segment's first slot and end of its slots in use, [2 i] and [2 i + 1].
    __shared__ int64_t s_tmp[kMaxSeg];
    for (int i = threadIdx.x; i < d.nseg; i += blockDim.x) {
        int64_t n = d.n_slots[i];
        s_tmp[i] = (n + tile - 1) / tile;
        if (s_lim) {
            const int64_t base = d.seg[i].base;
            s_lim[2 * i] = base;
            s_lim[2 * i + 1] = base + n;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t acc = 0;
        for (int i = 0; i < d.nseg; ++i) {
            s_tpre[i] = acc;
            acc += s_tmp[i];
        }
        s_tpre[d.nseg] = acc;
    }
    __syncthreads();
}

__device__ __forceinline__ int seg_of_tile(const int64_t *s_tpre, int nseg, int64_t t)
{
    int lo = 0, hi = nseg;  // s_tpre[lo] <= t < s_tpre[hi]
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (s_tpre[mid] <= t)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

__device__ __forceinline__ void block_run(int64_t T, int64_t &t0, int64_t &t1)
{
    const int64_t G = gridDim.x;
    int64_t vb = blockIdx.x;
    if ((G & 7) == 0) vb = (int64_t)(blockIdx.x & 7) * (G >> 3) + (blockIdx.x >> 3);
    t0 = vb * T / G;
    t1 = (vb + 1) * T / G;
}

// =======================================================================================
// Particle load.
// =======================================================================================
template <bool F64>
__global__ void k_init(Dev d, int sg, int64_t n, int64_t ppc, int init_mode, double vth,
                       double amp, int mode)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const SegC &S = d.seg[sg];
    const EnsC &e = d.ens[S.ens];
    const int s = S.species;
    const int64_t i = S.base + p;
    double x;
    int cell = 0;
    float off = 0.f;
    if (init_mode == 0) {
        cell = (int)(p / ppc);
        const uint4 w = draw(S.seed, s, (uint32_t)p, kInitTag, 0u);
        off = u01f(w.x);
        x = ((double)cell + (double)off) * S.dx;
    } else {
        const double L = e.L;
        const double k = 6.283185307179586476925286766559 * (double)mode / L;
        const double x0 = ((double)p + 0.5) * L / (double)n;
        x = x0 + (amp / k) * sin(k * x0);
        if (x < 0.0) x += L;
        if (x >= L) x -= L;
        if (!(x >= 0.0 && x < L)) x = 0.0;
        const double g = x / S.dx;
        double jf = floor(g);
        cell = (int)jf;
        off = (float)(g - jf);
        if (off >= 1.0f) {
            off = 0.0f;
            cell += 1;
            if (cell >= S.ncells) cell = 0;
        }
    }
    double z[3];
    three_normals<double>(draw(S.seed, s, (uint32_t)p, kInitTag, 1u), z);
    if constexpr (!F64) {
        d.cell[0][i] = cell;
        d.off[0][i] = off;
        d.fvx[0][i] = (float)(vth * z[0]);
        d.fvy[0][i] = (float)(vth * z[1]);
        d.fvz[0][i] = (float)(vth * z[2]);
    } else {
        d.x[0][i] = x;
        d.dvx[0][i] = vth * z[0];
        d.dvy[0][i] = vth * z[1];
        d.dvz[0][i] = vth * z[2];
    }
    d.id[0][i] = (uint32_t)p;
}

// Max |v|^2 of every segment into the current half of vmax2 (after a load or injection).
template <bool F64>
__global__ void k_vmax(Dev d)
{
    __shared__ double s_m[16];
    const int sg = blockIdx.y;
    const SegC &S = d.seg[sg];
    const int b = *d.cur;
    const int64_t n = d.n_slots[sg];
    double m = 0.0;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n;
         p += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = S.base + p;
        if constexpr (!F64) {
            if (d.cell[b][i] == kDead) continue;
            m = fmax(m, speed2_rn(d.fvx[b][i], d.fvy[b][i], d.fvz[b][i]));
        } else {
            if (!(d.x[b][i] >= 0.0)) continue;
            m = fmax(m, speed2_rn(d.dvx[b][i], d.dvy[b][i], d.dvz[b][i]));
        }
    }
    m = wave_max_f64(m);
    if (lane_id() == 0) s_m[threadIdx.x / kWave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < (int)(blockDim.x / kWave); ++i) m = fmax(m, s_m[i]);
        const int half = *d.vcur;
        if (m > 0.0)
            atomicMax(d.vmax2 + ((int64_t)half * kCntStripes + stripe_of_block()) * d.nseg + sg, dbits(m));
    }
}

// =======================================================================================
// Field solve.  With constant coefficients the three-point Poisson system on the interior
// nodes (phi_0 = phi_N = 0) factors into two prefix sums:
//   C_m = sum_{i=1..m} rho_i,  E_{m+1/2} = E_{1/2} + (dx/eps0) C_m,
//   phi_j = -dx (j E_{1/2} + (dx/eps0) sum_{m<j} C_m),
//   E_{1/2} = -(dx/eps0) sum_{m=0}^{N-1} C_m / N      (from phi_N = 0).
// This is the exact solution of the same tridiagonal system the Thomas algorithm solves,
// computed in two passes over the nodes: pass 1 reduces per-chunk aggregates, pass 2 has
// each chunk scan the aggregates of its ensemble and then its own nodes.  Node E is the
// centred difference, i.e. the mean of the two face fields, with the half-cell Gauss rule
// at bounded walls.  Periodic runs add the uniform background that cancels the deposited
// charge and shift phi to zero mean afterwards.
// =======================================================================================
// Block-wide inclusive scan of one double per thread (256 threads).
__device__ double block_incl_scan(double v, double *s_buf)
{
    const int lane = lane_id(), w = threadIdx.x / kWave;
    v = wave_incl_scan(v);
    if (lane == kWave - 1) s_buf[w] = v;
    __syncthreads();
    double add = 0.0;
    for (int i = 0; i < w; ++i) add += s_buf[i];
    __syncthreads();
    return v + add;
}

__device__ double block_sum(double v, double *s_buf)
{
    v = wave_sum_f64(v);
    const int w = threadIdx.x / kWave, nw = blockDim.x / kWave;
    if (lane_id() == 0) s_buf[w] = v;
    __syncthreads();
    double r = 0.0;
    for (int i = 0; i < nw; ++i) r += s_buf[i];
    __syncthreads();
    return r;
}

// N block-wide sums at once (one LDS round); same summation order as block_sum.
template <int N>
__device__ void block_sums(double (&v)[N], double *s /* N * 16 doubles */)
{
    const int w = threadIdx.x / kWave, nw = blockDim.x / kWave;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = wave_sum_f64(v[i]);
    if (lane_id() == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) s[i * 16 + w] = v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        double r = 0.0;
        for (int k = 0; k < nw; ++k) r += s[i * 16 + k];
        v[i] = r;
    }
    __syncthreads();
}

__device__ __forceinline__ int chunk_ens(const Dev &d, int64_t k)
{
    int lo = 0, hi = d.nens;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (d.ens[mid].chunk0 <= k)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// Blocks that place a step's births: the births grow with the particles (about 4.5e-4 of
// the electrons per step), so the block count does too, from 64 (enough for the 4e7-particle
// slab's ten thousand, under one per thread) to 256 from 5e8 slots on (64 batched
// ensembles: their solve kernel 61 -> 49 us; on the slab 256 blocks cost 1 us more).
__host__ __forceinline__ int place_blocks(const Dev &d)
{
    return (int)std::min<int64_t>(256, std::max<int64_t>(64, d.cap_tot >> 21));
}

// Birth ranking and placement, callable by a block of a kernel of their own or by extra
// blocks of the two solve kernels (defined with the births below).
__device__ void group_tile_scan_body(const Dev &d, int t);
template <bool F64, bool OWN = false>
__device__ void birth_place_body(const Dev &d, int deferred, int advance, int bid, int nblk, uint32_t *s_gp = nullptr);

// For the null-collision bound (R11) that the second solve kernel's last block computes: the
// largest |v|^2 of each segment over the stripes of the half the bound uses, one wave per
// segment (a block of kSolveThreads covers kSolveThreads / kWave segments), so that block
// reads one value per segment.  That half holds the previous step's maxima: the current
// one, or with the previous step's births still to be placed (`pending`), the other one,
// which their placement makes current.
__device__ void vmax_reduce_body(const Dev &d, int pending, int bid)
{
    const int half = pending ? 1 - *d.vcur : *d.vcur;
    const int sg = bid * (kSolveThreads / kWave) + (int)threadIdx.x / kWave;
    if (sg >= d.nseg) return;
    const double m2 = seg_vmax2(d, sg, half);
    if (lane_id() == 0) d.vmred[sg] = m2;
}

// Blocks [0, nchunks) solve; with `nscan` > 0, that many more blocks scan the group counts
// of the previous step's births (independent data; one tile each), so that scan costs no
// launch of its own; `nred` more blocks reduce the speed maxima for the null-collision bound
// (vmax_reduce_body).
template <bool F64>
__global__ void __launch_bounds__(kSolveThreads) k_solve1(Dev d, int nchunks, int nscan, int nred)
{
    if ((int)blockIdx.x >= nchunks) {
        const int r = (int)blockIdx.x - nchunks;
        if (r < nscan)
            group_tile_scan_body(d, r);
        else if (r - nscan < nred)
            vmax_reduce_body(d, nscan > 0, r - nscan);
        return;
    }
    __shared__ double s_buf[8];
    const int64_t k = blockIdx.x;
    const int ei = chunk_ens(d, k);
    const EnsC e = d.ens[ei];
    const int64_t N = e.ncells, nn = e.nnodes;
    const int64_t a = (k - e.chunk0) * kChunk;
    const int64_t j0 = a + (int64_t)threadIdx.x * kNodesPerThread;
    double loc = 0.0, sumpre = 0.0, totq = 0.0;
    // thread-local prefix of interior rho and its running sum
    double rho_loc[kNodesPerThread];
    double rho_first = 0.0;  // rho of the chunk's first node (thread 0), for the next chunk's solve
    // smoothing (R23): the chunk's raw densities and a halo of p nodes each side, folded
    // onto the grid, staged in LDS with coalesced loads; s_raw[i] is node a - p + i
    __shared__ double s_raw[kChunk + 2 * kMaxSmooth];
    const int p = e.smooth;
    double rq[kNodesPerThread];
    if (p > 0) {
        constexpr int kStage = (kChunk + 2 * kMaxSmooth + kSolveThreads - 1) / kSolveThreads;
        int64_t jm[kStage];
        bool ok[kStage];
        double rr[kStage];
#pragma unroll
        for (int u = 0; u < kStage; ++u) {
            const int i = threadIdx.x + u * kSolveThreads;
            const int64_t m = a - p + i;
            ok[u] = i < kChunk + 2 * p && m <= nn - 1 + p;
            jm[u] = ok[u] ? smooth_fold(e, m) : 0;
        }
        node_rho_raw<F64, kStage>(d, e, jm, ok, rr);
#pragma unroll
        for (int u = 0; u < kStage; ++u) {
            const int i = threadIdx.x + u * kSolveThreads;
            if (i < kChunk + 2 * p) s_raw[i] = rr[u];
        }
        __syncthreads();
        const double pscale = 1.0 / (double)(1 << (2 * p));
#pragma unroll
        for (int q = 0; q < kNodesPerThread; ++q) {
            double r = 0.0;
            double c = 1.0;  // C(2p, k), exact in binary64
            const int i0 = (int)(j0 + q - a);
            for (int k = 0; k <= 2 * p; ++k) {
                r += c * s_raw[i0 + k];
                c = c * (double)(2 * p - k) / (double)(k + 1);
            }
            rq[q] = r * pscale;
        }
    } else {
        int64_t jq[kNodesPerThread];
        bool ok[kNodesPerThread];
#pragma unroll
        for (int q = 0; q < kNodesPerThread; ++q) {
            jq[q] = j0 + q;
            ok[q] = jq[q] < nn;
        }
        node_rho_raw<F64, kNodesPerThread>(d, e, jq, ok, rq);
    }
#pragma unroll
    for (int q = 0; q < kNodesPerThread; ++q) {
        const int64_t j = j0 + q;
        double r = 0.0;
        if (j < nn) {
            r = rq[q];
            d.rho[e.gbase + j] = r;
            totq += r * node_vol(e, j);
        }
        if (q == 0) rho_first = r;
        rho_loc[q] = (j >= 1 && j <= N - 1) ? r : 0.0;
        loc += rho_loc[q];
    }
    const double excl = block_incl_scan(loc, s_buf) - loc;
    double run = excl;
#pragma unroll
    for (int q = 0; q < kNodesPerThread; ++q) {
        run += rho_loc[q];
        if (j0 + q < N) sumpre += run;  // m in [0, N-1]
    }
    // the ensemble's max |E| is accumulated by the second pass's blocks (atomic max)
    if (k == e.chunk0 && threadIdx.x == 0) d.emax[ei] = 0.0;
    __shared__ double s_red[3 * 16];
    double v[3] = {loc, sumpre, totq};
    block_sums<3>(v, s_red);
    if (threadIdx.x == 0) {
        double *g = d.agg + k * A_NAGG;
        g[A_SUMRHO] = v[0];
        g[A_SUMPRE] = v[1];
        g[A_TOTQ] = v[2];
        double n1, dd, cnt;
        chunk_counts(a, nn, N, n1, dd, cnt);
        g[A_N1] = n1;
        g[A_D] = dd;
        g[A_CNT] = cnt;
        g[A_RHO0] = rho_first;
    }
}

// Reading R11: per-segment null-collision bound from the current max speed and max field.
// One wave per segment (lanes read the striped speed maxima); every lane gets the result.
__device__ void compute_params(const Dev &d)
{
    const int nw = blockDim.x / kWave, w = threadIdx.x / kWave;
    const int half = *d.vcur;
    for (int sg = w; sg < d.nseg; sg += nw) {
        double numax, pnull;
        seg_params(d, sg, half, d.emax[d.seg[sg].ens], numax, pnull);
        if (lane_id() == 0) {
            d.numax[sg] = numax;
            d.pnull[sg] = pnull;
        }
    }
}

// The same bound in the last block of the second solve kernel, one thread per segment from
// the maxima the first kernel reduced: max |E| was accumulated by other blocks of the same
// launch, so it is read with an atomic, which sees every block's atomic update without a
// fence, and every segment's loads go out at once.
__device__ void compute_params_reduced(const Dev &d)
{
    for (int sg = threadIdx.x; sg < d.nseg; sg += blockDim.x) {
        const SegC &S = d.seg[sg];
        const double m2 = d.vmred[sg];
        const double emax =
            __longlong_as_double((long long)atomicMax((unsigned long long *)(d.emax + S.ens), 0ull));
        double numax, pnull;
        seg_bound(S, d.ens[S.ens], m2, emax, numax, pnull);
        d.numax[sg] = numax;
        d.pnull[sg] = pnull;
    }
}

__global__ void k_params(Dev d) { compute_params(d); }

template <bool F64>
__device__ void solve2_body(const Dev &d, int zero_q)
{
    __shared__ double s_buf[8];
    __shared__ double s_E[F64 ? 1 : kChunk + 1];  // the chunk's node E, for the gather table
    __shared__ double s_C0, s_F0, s_Eh, s_bg, s_Ctot;
    const int64_t k = blockIdx.x;
    const int ei = chunk_ens(d, k);
    const EnsC e = d.ens[ei];
    const int64_t N = e.ncells, nn = e.nnodes;
    const int64_t a = (k - e.chunk0) * kChunk;
    const double dx = e.dx, ce = e.dx / e.eps0;
    const int64_t j0 = a + (int64_t)threadIdx.x * kNodesPerThread;
    // this thread's densities (written by the first pass), loaded before the chunk scan so
    // the two round trips overlap
    double rv[kNodesPerThread];
#pragma unroll
    for (int q = 0; q < kNodesPerThread; ++q) {
        const bool in = j0 + q < nn;
        const double v = d.rho[e.gbase + (in ? j0 + q : 0)];
        rv[q] = in ? v : 0.0;
    }
    // Scan of the ensemble's chunk aggregates by the first wave, in parallel: lane l owns
    // the contiguous chunk range [l R, (l+1) R).  C_pre(c) = sum_{c'<c} A'(c') and
    // F_pre(c) = sum_{c'<c} (cnt(c') C_pre(c') + B'(c')) are two nested exclusive scans.
    // (Wave shuffles only: no block barrier inside the scan.)
    if (threadIdx.x < kWave) {
        const int lane = (int)threadIdx.x;
        const int64_t nc = e.nchunks;
        const int64_t R = (nc + kWave - 1) / kWave;
        const int64_t c0 = (int64_t)lane * R, c1 = min(c0 + R, nc);
        // floating walls (R22): the particles absorbed so far at the left wall, per
        // species, from the exact striped wall counts (sums < 2^53: exact in binary64)
        // (species loops run over the two array entries with constant indices, so that the
        // local copy of the ensemble stays in registers)
        double nabs[2] = {0.0, 0.0};
        if (e.floating)
            for (int st = lane; st < kCntStripes; st += kWave) {
#pragma unroll
                for (int s = 0; s < 2; ++s)
                    if (s < e.nspecies)
                        nabs[s] += (double)d.cnt[((int64_t)st * d.nseg + e.seg[s]) * C_NCNT + C_WALL_L];
            }
        double tq = 0.0;
        for (int64_t c = c0; c < c1; ++c) tq += d.agg[(e.chunk0 + c) * A_NAGG + A_TOTQ];
        const double tqs = wave_sum_f64(tq);
        const double bg = e.periodic ? -tqs / e.L : 0.0;
        double a = 0.0, g = 0.0, n = 0.0;  // local A sum, local sum of cnt*Cpre_local + B, cnt sum
        for (int64_t c = c0; c < c1; ++c) {
            const double *gg = d.agg + (e.chunk0 + c) * A_NAGG;
            const double A = gg[A_SUMRHO] + bg * gg[A_N1];
            const double B = gg[A_SUMPRE] + bg * gg[A_D];
            g += gg[A_CNT] * a + B;
            n += gg[A_CNT];
            a += A;
        }
        const double apre = wave_incl_scan(a) - a;  // C_pre at c0
        const double fin = n * apre + g;                // this range's sum of C over m
        const double fpre = wave_incl_scan(fin) - fin;
        const double Stot = wave_sum_f64(fin), Ctot = wave_sum_f64(a);
        const double nab0 = wave_sum_f64(nabs[0]), nab1 = wave_sum_f64(nabs[1]);
        const int64_t me = k - e.chunk0;
        if (me >= c0 && me < c1) {
            double ca = apre, fa = fpre;
            for (int64_t c = c0; c < me; ++c) {
                const double *gg = d.agg + (e.chunk0 + c) * A_NAGG;
                const double A = gg[A_SUMRHO] + bg * gg[A_N1];
                const double B = gg[A_SUMPRE] + bg * gg[A_D];
                fa += gg[A_CNT] * ca + B;
                ca += A;
            }
            s_C0 = ca;
            s_F0 = fa;
        }
        // Reading R22: floating walls fix E_{1/2} by Gauss's law over the left wall (the
        // charge absorbed there, q w per particle) and the half cell in front of it;
        // otherwise phi_N = 0 (or periodicity) fixes it.
        const double sigL = e.qw[0] * nab0 + (e.nspecies > 1 ? e.qw[1] * nab1 : 0.0);
        if (lane == 0) {
            s_bg = bg;
            s_Ctot = Ctot;
            if (e.floating)
                s_Eh = (sigL + d.agg[e.chunk0 * A_NAGG + A_RHO0] * node_vol(e, 0)) / e.eps0;
            else
                s_Eh = -ce * Stot / (double)N;
        }
    }
    __syncthreads();
    const double bg = s_bg, Eh = s_Eh;
    // local inclusive prefix of interior rho' (with background) -> C_j
    double rl[kNodesPerThread + 1];
    double loc = 0.0;
#pragma unroll
    for (int q = 0; q < kNodesPerThread; ++q) {
        const int64_t j = j0 + q;
        double r = 0.0;
        if (j < nn) {
            const double rj = rv[q] + bg;
            if (e.periodic) d.rho[e.gbase + j] = rj;  // report rho with the background
            if (j >= 1 && j <= N - 1) r = rj;
        }
        rl[q] = r;
        loc += r;
    }
    const double cex = block_incl_scan(loc, s_buf) - loc;
    double Cj[kNodesPerThread];
    double c = s_C0 + cex;
    double csum = 0.0;
#pragma unroll
    for (int q = 0; q < kNodesPerThread; ++q) {
        c += rl[q];
        Cj[q] = c;
        csum += (j0 + q < N) ? c : 0.0;
    }
    // exclusive prefix of C over m < j (m in [0, N-1])
    const double fex = block_incl_scan(csum, s_buf) - csum;
    double F = s_F0 + fex;
    double emax = 0.0, phisum = 0.0, fe = 0.0;
    int nonfin = 0;
    // C_{j-1} for the first node of the thread
    double Cprev = (j0 == 0) ? 0.0 : (Cj[0] - rl[0]);
#pragma unroll
    for (int q = 0; q < kNodesPerThread; ++q) {
        const int64_t j = j0 + q;
        if (j >= nn) break;
        double phi = -dx * ((double)j * Eh + ce * F);
        if (!e.periodic && !e.floating && j == N) phi = 0.0;
        if (j == 0) phi = 0.0;
        d.phi[e.gbase + j] = phi;
        phisum += phi;
        // face fields around node j
        const double Em = Eh + ce * Cprev;  // E_{j-1/2} (j >= 1)
        const double Ep = Eh + ce * Cj[q];  // E_{j+1/2} (j <= N-1)
        double Ej;
        if (e.periodic) {
            if (j == 0) {
                const double Elast = Eh + ce * s_Ctot;  // E_{N-1/2}
                Ej = 0.5 * (Elast + Ep);
            } else {
                Ej = 0.5 * (Em + Ep);
            }
        } else if (j == 0) {
            Ej = Eh - d.rho[e.gbase] * node_vol(e, 0) / e.eps0;
        } else if (j == N) {
            Ej = Em + d.rho[e.gbase + N] * node_vol(e, N) / e.eps0;
        } else {
            Ej = 0.5 * (Em + Ep);
        }
        d.E[e.gbase + j] = Ej;
        if constexpr (!F64) s_E[j - a] = Ej;
        if (!isfinite(Ej)) nonfin = 1;
        emax = fmax(emax, fabs(Ej));
        fe += Ej * Ej * node_vol(e, j);
        if (j < N) F += Cj[q];
        Cprev = Cj[q];
    }
    if constexpr (!F64) {
        // Gather table of the chunk's cells, (E_j, E_{j+1} - E_j) in binary32.  The node
        // after the chunk's last cell is the periodic wrap E_0, or the next chunk's first
        // node, computed here from this chunk's last C and that node's rho (kept by the
        // first solve pass, since the next chunk rewrites it with the background).
        const int64_t L = min((int64_t)kChunk, N - a);
        if (L > 0) {
            if (e.periodic && a + L == N) {
                if (threadIdx.x == 0) s_E[L] = 0.5 * ((Eh + ce * s_Ctot) + (Eh + ce * 0.0));
            } else if (L == kChunk && threadIdx.x == blockDim.x - 1) {
                const int64_t jn = a + kChunk;
                const double rn = d.agg[(k + 1) * A_NAGG + A_RHO0];
                const double Cl = Cj[kNodesPerThread - 1];  // C_{jn-1}
                const double Em = Eh + ce * Cl;
                if (!e.periodic && jn == N) {
                    s_E[L] = Em + rn * node_vol(e, N) / e.eps0;
                } else {
                    const double Cn = Cl + (rn + bg);
                    s_E[L] = 0.5 * (Em + (Eh + ce * Cn));
                }
            }
        }
        __syncthreads();
        for (int64_t j = a + threadIdx.x; j < a + L; j += blockDim.x) {
            const double E0 = s_E[j - a], E1 = s_E[j - a + 1];
            d.Ecell[e.gbase + j] = make_float2((float)E0, (float)(E1 - E0));
        }
    }
    // zero the deposit for the next pass when asked (fused step)
    if (zero_q) {
        for (int q = 0; q < kNodesPerThread; ++q) {
            const int64_t j = j0 + q;
            if (j >= nn) break;
            for (int s = 0; s < e.nspecies; ++s) {
                if constexpr (!F64)
                    d.Qi[(int64_t)s * d.nodes_tot + e.gbase + j] = 0ull;
                else
                    d.Qd[(int64_t)s * d.nodes_tot + e.gbase + j] = 0.0;
            }
        }
    }
    // chunk partials
    {
        double em = wave_max_f64(emax);
        __shared__ double s_em[8];
        if (lane_id() == 0) s_em[threadIdx.x / kWave] = em;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int i = 1; i < (int)(blockDim.x / kWave); ++i) em = fmax(em, s_em[i]);
            s_em[0] = em;
        }
        __syncthreads();
        em = s_em[0];
        __shared__ double s_red3[3 * 16];
        double fv[3] = {phisum, (double)nonfin, fe};
        block_sums<3>(fv, s_red3);
        if (threadIdx.x == 0) {
            d.part[k * P_NPART + P_PHISUM] = fv[0];
            d.part[k * P_NPART + P_FE] = 0.5 * e.eps0 * fv[2];  // this chunk's field energy
            // |E| >= 0: its bit pattern orders as an unsigned integer
            atomicMax((unsigned long long *)(d.emax + ei), dbits(em));
            if (fv[1] > 0.0) atomicOr(d.err, (int)E_NONFINITE);
        }
    }
}

// Blocks [0, nchunks) solve; blocks beyond place the previous step's births (they touch
// particle slots beyond the ones in use, the id and slot counters, the birth lists, the
// speed-maximum halves and the step counter, none of which the solve reads or writes).
// With `params`, the last block to finish computes the next pass's null-collision bound
// (R11) from this solve's max |E| and the speed maxima the first kernel reduced, in place of
// a kernel of its own; it reads max |E|, which other blocks of this launch updated, through
// an atomic, which needs no fence.
template <bool F64>
__global__ void __launch_bounds__(kSolveThreads) k_solve2(Dev d, int zero_q, int nchunks, int params, int advance)
{
    // (without births nothing else in this launch reads the step counter)
    if (advance && blockIdx.x == 0 && threadIdx.x == 0) *d.step += 1;
    if ((int)blockIdx.x >= nchunks)
        birth_place_body<F64>(d, 1, 1, (int)blockIdx.x - nchunks, (int)gridDim.x - nchunks);
    else
        solve2_body<F64>(d, zero_q);
    if (!params) return;
    __shared__ bool s_last;
    __syncthreads();
    if (threadIdx.x == 0) s_last = (atomicAdd(d.ticket + 6, 1u) == gridDim.x - 1);
    __syncthreads();
    if (!s_last) return;
    compute_params_reduced(d);
    if (threadIdx.x == 0) d.ticket[6] = 0u;
}

// Periodic only: subtract the mean of phi and build the gather table.
__global__ void __launch_bounds__(kSolveThreads) k_phi_shift(Dev d)
{
    const int64_t k = blockIdx.x;
    const int ei = chunk_ens(d, k);
    const EnsC e = d.ens[ei];
    __shared__ double s_mean;
    if (threadIdx.x < kWave) {
        double ps = 0.0;
        for (int64_t c = threadIdx.x; c < e.nchunks; c += kWave) ps += d.part[(e.chunk0 + c) * P_NPART + P_PHISUM];
        ps = wave_sum_f64(ps);
        if (threadIdx.x == 0) s_mean = ps / (double)e.ncells;
    }
    __syncthreads();
    const int64_t a = (k - e.chunk0) * kChunk;
    for (int64_t j = a + threadIdx.x; j < min(a + kChunk, e.nnodes); j += blockDim.x)
        d.phi[e.gbase + j] -= s_mean;
}

// Gather table: per cell (E_j, E_{j+1} - E_j) in float.
__global__ void k_ecell(Dev d)
{
    const int64_t k = blockIdx.x;
    const int ei = chunk_ens(d, k);
    const EnsC e = d.ens[ei];
    const int64_t a = (k - e.chunk0) * kChunk;
    for (int64_t j = a + threadIdx.x; j < min(a + kChunk, e.ncells); j += blockDim.x) {
        const int64_t j1 = (e.periodic && j + 1 == e.ncells) ? 0 : j + 1;
        const double E0 = d.E[e.gbase + j], E1 = d.E[e.gbase + j1];
        d.Ecell[e.gbase + j] = make_float2((float)E0, (float)(E1 - E0));
    }
}

// Field energy 1/2 eps0 sum_j E_j^2 V_j of every ensemble (for the diagnostics and the
// adjoint objective; one wave per ensemble).
__global__ void __launch_bounds__(1024) k_field_energy(Dev d)
{
    __shared__ double s_buf[16];
    const EnsC e = d.ens[blockIdx.x];  // one block per ensemble
    double f = 0.0;
    for (int64_t j = threadIdx.x; j < e.nnodes; j += blockDim.x) {
        const double E = d.E[e.gbase + j];
        f += E * E * node_vol(e, j);
    }
    double v[1] = {f};
    block_sums<1>(v, s_buf);
    if (threadIdx.x == 0) d.fe[blockIdx.x] = 0.5 * e.eps0 * v[0];
}

// Max |E| and field energy of a field set from the host (test hook).
__global__ void __launch_bounds__(kSolveThreads) k_field_stats(Dev d)
{
    __shared__ double s_buf[8];
    for (int en = 0; en < d.nens; ++en) {
        const EnsC &e = d.ens[en];
        double em = 0.0, fe = 0.0;
        for (int64_t j = threadIdx.x; j < e.nnodes; j += blockDim.x) {
            const double E = d.E[e.gbase + j];
            em = fmax(em, fabs(E));
            fe += E * E * node_vol(e, j);
        }
        em = wave_max_f64(em);
        __shared__ double s_em[8];
        if (lane_id() == 0) s_em[threadIdx.x / kWave] = em;
        __syncthreads();
        const double f = block_sum(fe, s_buf);
        if (threadIdx.x == 0) {
            for (int i = 1; i < (int)(blockDim.x / kWave); ++i) em = fmax(em, s_em[i]);
            d.emax[en] = em;
            d.fe[en] = 0.5 * e.eps0 * f;
        }
        __syncthreads();
    }
}

template <bool F64>
__global__ void k_zero_q(Dev d)
{
    const int64_t n = 2 * d.nodes_tot;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        if constexpr (!F64)
            d.Qi[i] = 0ull;
        else
            d.Qd[i] = 0.0;
    }
}

// =======================================================================================
// Generic exclusive scan of u32 (tile sums, down-sweep; a scan of the sums in between when they
// are many).
// =======================================================================================
constexpr int kScanTile = kScanBlock * kScanItems;

__device__ uint32_t block_excl_scan_u32(uint32_t v, uint32_t *s_buf, uint32_t &total)
{
    const int lane = lane_id(), w = threadIdx.x / kWave, nw = blockDim.x / kWave;
    uint32_t x = v;
    x = wave_incl_scan(x);
    if (lane == kWave - 1) s_buf[w] = x;
    __syncthreads();
    uint32_t add = 0, tot = 0;
    for (int i = 0; i < nw; ++i) {
        if (i < w) add += s_buf[i];
        tot += s_buf[i];
    }
    __syncthreads();
    total = tot;
    return x - v + add;
}

__global__ void __launch_bounds__(kScanBlock) k_scan_sums(const uint32_t *in, int64_t n, uint32_t *part,
                                                          const int64_t *parity_step)
{
    if (parity_step) in += (int64_t)(*parity_step & 1) * n;
    __shared__ uint32_t s_buf[16];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    uint32_t s = 0;
    for (int q = 0; q < kScanItems; ++q) {
        const int64_t i = base + (int64_t)q * kScanBlock + threadIdx.x;
        if (i < n) s += in[i];
    }
    uint32_t tot;
    block_excl_scan_u32(s, s_buf, tot);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

__global__ void __launch_bounds__(1024) k_scan_part(uint32_t *part, int64_t nb)
{
    __shared__ uint32_t s_buf[16];
    __shared__ uint32_t s_carry;
    if (threadIdx.x == 0) s_carry = 0;
    __syncthreads();
    for (int64_t c = 0; c < nb; c += blockDim.x) {
        const int64_t i = c + threadIdx.x;
        const uint32_t v = i < nb ? part[i] : 0u;
        uint32_t tot;
        const uint32_t ex = block_excl_scan_u32(v, s_buf, tot);
        if (i < nb) part[i] = ex + s_carry;
        __syncthreads();
        if (threadIdx.x == 0) s_carry += tot;
        __syncthreads();
    }
}

// With OWN each block adds up the tiles before its own from the tile sums (part unscanned);
// otherwise part holds their scan.
template <bool OWN>
__global__ void __launch_bounds__(kScanBlock) k_scan_down(uint32_t *in, uint32_t *out, int64_t n,
                                                          const uint32_t *part, int zero_in,
                                                          const int64_t *parity_step)
{
    if (parity_step) in += (int64_t)(*parity_step & 1) * n;
    __shared__ uint32_t s_buf[16];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    // each thread owns kScanItems consecutive elements
    const int64_t i0 = base + (int64_t)threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    uint32_t s = 0, before = 0;
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        v[q] = (i0 + q < n) ? in[i0 + q] : 0u;
        s += v[q];
    }
    uint32_t tot;
    if constexpr (OWN) {
        uint32_t mine = 0;
        for (uint32_t i = threadIdx.x; i < blockIdx.x; i += kScanBlock) mine += part[i];
        block_excl_scan_u32(mine, s_buf, before);
    } else {
        before = part[blockIdx.x];
    }
    uint32_t ex = block_excl_scan_u32(s, s_buf, tot) + before;
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        if (i0 + q < n) {
            out[i0 + q] = ex;
            if (zero_in) in[i0 + q] = 0u;
        }
        ex += v[q];
    }
}

// The sort's scan of a small run's cell counts into run cursors, and the segments' first
// positions, by one block: a thread owns kScanItems consecutive cells of every 16384 (its loads
// whole 16-byte vectors), the running total carried between rounds.  4096 cells take 3.7 us
// and 20014 take 10.5, where the scan's three kernels and k_segstart took 18 and 23; 40022 would
// take 18.5, more than the two kernels of the general scan and k_segstart.
constexpr int kOneThreads = 1024;
constexpr int64_t kOneScanMax = 2 * kOneThreads * kScanItems;
__global__ void __launch_bounds__(kOneThreads) k_sort_scan(Dev d)
{
    __shared__ uint32_t s_buf[16];
    const int64_t n = d.cells_tot;
    uint32_t carry = 0;
    for (int64_t base = 0; base < n; base += kOneThreads * kScanItems) {
        const int64_t i0 = base + (int64_t)threadIdx.x * kScanItems;
        uint32_t v[kScanItems], s = 0, tot;
        const bool full = i0 + kScanItems <= n;
        if (full) {
#pragma unroll
            for (int q = 0; q < kScanItems; q += 4) *(uint4 *)(v + q) = *(const uint4 *)(d.cellcnt + i0 + q);
        } else {
#pragma unroll
            for (int q = 0; q < kScanItems; ++q) v[q] = i0 + q < n ? d.cellcnt[i0 + q] : 0u;
        }
#pragma unroll
        for (int q = 0; q < kScanItems; ++q) s += v[q];
        uint32_t ex = block_excl_scan_u32(s, s_buf, tot) + carry;
        carry += tot;
#pragma unroll
        for (int q = 0; q < kScanItems; ++q) {
            const uint32_t c = v[q];
            v[q] = ex;
            ex += c;
        }
        if (full) {
#pragma unroll
            for (int q = 0; q < kScanItems; q += 4) {
                *(uint4 *)(d.cursor + i0 + q) = *(const uint4 *)(v + q);
                *(uint4 *)(d.cellcnt + i0 + q) = make_uint4(0u, 0u, 0u, 0u);
            }
        } else {
#pragma unroll
            for (int q = 0; q < kScanItems; ++q)
                if (i0 + q < n) {
                    d.cursor[i0 + q] = v[q];
                    d.cellcnt[i0 + q] = 0u;
                }
        }
    }
    __threadfence_block();
    __syncthreads();  // the cursors are written
    for (int sg = threadIdx.x; sg < d.nseg; sg += kOneThreads) d.segstart[sg] = d.cursor[d.seg[sg].cbase];
}

// =======================================================================================
// Births: a birth's rank among its ensemble's births of the step is the scanned count of
// the id groups below its own plus the bits below it in its group's 128 bitmap words.  The
// new electron and ion go to slot n_slots + rank with id next_id + rank.  The last block
// updates the counters.
// =======================================================================================
__device__ __forceinline__ void birth_locate(const Dev &d, int64_t k, int &st, uint32_t &idx,
                                             const uint32_t *s_pre)
{
    int lo = 0, hi = kStripes;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((int64_t)s_pre[mid] <= k)
            lo = mid;
        else
            hi = mid;
    }
    st = lo;
    idx = (uint32_t)(k - s_pre[lo]);
}

// Exclusive prefix of the per-stripe birth counts (clamped to the stripe capacity), with the
// total in s_pre[kStripes].  Called by the first wave of the block.
__device__ __forceinline__ void stripe_prefix(const BirthBuf &bb, int64_t cap, uint32_t *s_pre)
{
    const int lane = lane_id();
    const uint32_t v = lane < kStripes ? (uint32_t)min((int64_t)bb.nbirth[lane], cap) : 0u;
    uint32_t inc = v;
    inc = wave_incl_scan(inc);
    if (lane < kStripes) s_pre[lane] = inc - v;
    if (lane == kStripes - 1) s_pre[kStripes] = inc;
}

// Bits of the group's bitmap below `pid` (the group's words are 128-byte aligned); the
// words are read as independent 16-byte loads four at a time.
__device__ __forceinline__ uint32_t rank_in_group(const uint32_t *group, uint32_t pid)
{
    static_assert(kGroupWords % 64 == 0, "whole batches of 64 words per group");
    const int wp = (int)((pid % kGroupIds) >> 5);  // words wholly below pid
    const uint4 *v = (const uint4 *)group;
    uint32_t r = __popc(group[wp] & ((1u << (pid & 31)) - 1u));
    // batches of 64 words, each batch's sixteen 16-byte loads in flight at once; words at
    // or above wp are masked
    for (int w0 = 0; w0 < wp; w0 += 64) {
        uint4 a[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) a[u] = v[w0 / 4 + u];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int w = w0 + 4 * u;
            r += (w < wp ? __popc(a[u].x) : 0u) + (w + 1 < wp ? __popc(a[u].y) : 0u) +
                 (w + 2 < wp ? __popc(a[u].z) : 0u) + (w + 3 < wp ? __popc(a[u].w) : 0u);
        }
    }
    return r;
}

// Exclusive scan of the current half's group counts, one tile of kGroupTile groups per block:
// gpre gets each group's prefix within its tile and gtile the tile's total (the placement
// adds the tiles' bases).  Wave w owns the w-th contiguous share of the tile, whole rows of
// 64 16-byte vectors, and reads it row by row, lane l taking the row's l-th vector, so every
// load instruction reads 1 KB of consecutive bytes; the share's rows are all loaded before
// any is used (one round trip), summed, the shares' bases exchanged in LDS, and each row
// scanned across the wave and written.  (One block over every group, per-thread runs read
// four vectors at a time, had taken 60 us for the 64 batched ensembles' 1.3e5 groups.)
constexpr int kTileVec = kGroupTile / 4;  // uint4 per tile

// (a block of 256 threads: four waves of kRows rows each)
__device__ void group_tile_scan_body(const Dev &d, int t)
{
    constexpr int kRows = kTileVec / (kWave * 4);
    __shared__ uint32_t s_w[4];
    const int p = (int)(*d.step & 1);
    const int w = (int)threadIdx.x / kWave, lane = lane_id();
    const int64_t v0 = (int64_t)t * kTileVec + (int64_t)w * kRows * kWave;
    const uint4 *in = (const uint4 *)(d.gcnt + (int64_t)p * d.g_tot) + v0;
    uint4 *out = (uint4 *)d.gpre + v0;
    uint4 v[kRows];
    uint32_t sum = 0;
#pragma unroll
    for (int r = 0; r < kRows; ++r) v[r] = in[r * kWave + lane];
#pragma unroll
    for (int r = 0; r < kRows; ++r) sum += v[r].x + v[r].y + v[r].z + v[r].w;
    sum = wave_sum_u32(sum);
    if (lane == 0) s_w[w] = sum;
    __syncthreads();
    uint32_t carry = 0;  // counts of the tile before this wave's share, then before the row
    for (int i = 0; i < w; ++i) carry += s_w[i];
    if (threadIdx.x == 0) d.gtile[t] = s_w[0] + s_w[1] + s_w[2] + s_w[3];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const uint32_t ls = v[r].x + v[r].y + v[r].z + v[r].w;
        uint32_t inc = ls;
        inc = wave_incl_scan(inc);
        const uint32_t ex = carry + inc - ls;
        out[r * kWave + lane] = make_uint4(ex, ex + v[r].x, ex + v[r].x + v[r].y, ex + v[r].x + v[r].y + v[r].z);
        carry += __shfl(inc, kWave - 1);
    }
}

__global__ void __launch_bounds__(256) k_group_scan(Dev d) { group_tile_scan_body(d, (int)blockIdx.x); }

// Place the births of this step (half p = step & 1).  With `deferred`, also clear the
// bitmap bits and group counts of half 1 - p (the previous step's births) and reset its
// birth counts, so the next step starts on a clean half.  The last block updates the
// counters, makes the freshly accumulated speed maxima current and (with `advance`)
// advances the step counter.
// The constants a birth's placement needs, staged in LDS by every placing block (one round
// trip, beside the stripe counts), so that a birth's chain of dependent loads is its record
// and then its rank: per ensemble the birth-ranking bases, id capacity and segments, per
// segment the slot base and capacity and the slots and ids in use before the placement.
struct PlaceEns {
    int64_t bm_base, grp_base, idcap;
    int32_t seg[2];
    int32_t nspecies;
};
struct PlaceSeg {
    int64_t base, cap, n_slots;
    uint32_t next_id;
};

// Bases of the group-count tiles (exclusive prefix of gtile) in LDS, by the whole block of
// 256 threads (four tiles each); all zero when the global scan ran (ngt = 0).
static_assert(kSolveThreads == 256, "the solve kernels' births blocks have 256 threads, as k_birth_place");
__device__ void stage_tile_bases(const Dev &d, uint32_t *s_tb)
{
    __shared__ uint32_t s_buf[16];
    constexpr int kPer = kMaxGroupTiles / 256;
    const int i0 = (int)threadIdx.x * kPer;
    uint32_t v[kPer], sum = 0;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        v[u] = (i0 + u < d.ngt) ? d.gtile[i0 + u] : 0u;
        sum += v[u];
    }
    uint32_t tot;
    uint32_t ex = block_excl_scan_u32(sum, s_buf, tot);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        s_tb[i0 + u] = ex;
        ex += v[u];
    }
}

// The births' scanned group count at group index i (global over every ensemble's groups).
__device__ __forceinline__ uint32_t group_prefix(const Dev &d, const uint32_t *s_tb, int64_t i)
{
    return s_tb[i / kGroupTile] + d.gpre[i];
}

// After a placement, by one block: the previous step's birth counts (with `deferred`), the
// half of the speed maxima that was current (it accumulates the next step's) and the step
// tallies of that half restart.
__device__ __forceinline__ void place_reset(const Dev &d, int deferred, const BirthBuf &ob, int vc)
{
    if (deferred)
        for (int i = threadIdx.x; i < kStripes; i += blockDim.x) ob.nbirth[i] = 0u;
    for (int64_t i = threadIdx.x; i < (int64_t)kCntStripes * d.nseg; i += blockDim.x)
        d.vmax2[(int64_t)vc * kCntStripes * d.nseg + i] = 0ull;
    for (int64_t i = threadIdx.x; i < (int64_t)kCntStripes * d.nseg * T_NSTEP; i += blockDim.x)
        d.ssum[(int64_t)vc * kCntStripes * d.nseg * T_NSTEP + i] = 0.0;
}

// Exclusive scan of one tile of group counts into LDS by a block of T threads (whole 16-byte
// vectors per thread); a barrier must follow.
template <int T>
__device__ __forceinline__ void scan_group_tile(const uint32_t *gcnt, uint32_t *s_gp)
{
    __shared__ uint32_t s_buf[16];
    constexpr int kVec = kGroupTile / (4 * T);
    uint4 v[kVec];
    uint32_t sum = 0, tot;
#pragma unroll
    for (int i = 0; i < kVec; ++i) v[i] = ((const uint4 *)gcnt)[threadIdx.x * kVec + i];
#pragma unroll
    for (int i = 0; i < kVec; ++i) sum += v[i].x + v[i].y + v[i].z + v[i].w;
    uint32_t ex = block_excl_scan_u32(sum, s_buf, tot);
#pragma unroll
    for (int i = 0; i < kVec; ++i) {
        uint32_t *o = s_gp + (threadIdx.x * kVec + i) * 4;
        o[0] = ex;
        o[1] = (ex += v[i].x);
        o[2] = (ex += v[i].y);
        o[3] = (ex += v[i].z);
        ex += v[i].w;
    }
}

// The pair of one birth, r-th of its ensemble's in the step, to its slots.
template <bool F64>
__device__ __forceinline__ void put_birth(const Dev &d, const Birth &B, uint32_t r, const PlaceEns &E,
                                          const PlaceSeg *s_ps, int b)
{
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        if (s >= E.nspecies) break;
        const PlaceSeg &P = s_ps[E.seg[s]];
        const int64_t slot = P.n_slots + r;
        if (slot >= P.cap) {
            atomicOr(d.err, (int)E_CAP_PART);
            continue;
        }
        if ((int64_t)P.next_id + r >= E.idcap) {
            atomicOr(d.err, (int)E_CAP_ID);
            continue;
        }
        const int64_t i = P.base + slot;
        const double v0 = s == 0 ? B.ve[0] : B.vi[0];
        const double v1 = s == 0 ? B.ve[1] : B.vi[1];
        const double v2 = s == 0 ? B.ve[2] : B.vi[2];
        if constexpr (!F64) {
            d.cell[b][i] = B.cell;
            d.off[b][i] = B.off;
            d.fvx[b][i] = (float)v0;
            d.fvy[b][i] = (float)v1;
            d.fvz[b][i] = (float)v2;
        } else {
            d.x[b][i] = B.x;
            d.dvx[b][i] = v0;
            d.dvy[b][i] = v1;
            d.dvz[b][i] = v2;
        }
        d.id[b][i] = P.next_id + r;
    }
}

// Places the step's births (k < M) and clears the marks of the previous step's (k < Mo): block
// `bid` of `nblk`.  pre(i) is the births' scanned group count at group index i.
template <bool F64, typename Pre>
__device__ __forceinline__ void place_births(const Dev &d, const BirthBuf &bb, const BirthBuf &ob, int64_t M,
                                             int64_t Mo, const uint32_t *s_pre, const uint32_t *s_old,
                                             const PlaceEns *s_pe, const PlaceSeg *s_ps, int bid, int nblk, Pre pre)
{
    const int b = *d.cur;
    // this step's births (k < M) and, with `deferred`, the previous step's (k < Mo), whose
    // bits and group counts are cleared; both records are loaded before either is used
    for (int64_t k = (int64_t)bid * blockDim.x + threadIdx.x; k < max(M, Mo);
         k += (int64_t)nblk * blockDim.x) {
        const bool nw = k < M, od = k < Mo;
        int st = 0, sto = 0;
        uint32_t idx = 0, idxo = 0;
        if (nw) birth_locate(d, k, st, idx, s_pre);
        if (od) birth_locate(d, k, sto, idxo, s_old);
        // copies: the particle stores below cannot alias them, so nothing is read twice
        Birth B{};
        uint2 okey = make_uint2(0u, 0u);
        if (nw) B = bb.births[(int64_t)st * d.birth_stripe_cap + idx];
        if (od) okey = *(const uint2 *)&ob.births[(int64_t)sto * d.birth_stripe_cap + idxo];
        if (od) {
            const PlaceEns &E = s_pe[okey.y];
            ob.bitmap[E.bm_base + (okey.x >> 5)] = 0u;
            ob.gcnt[E.grp_base + okey.x / kGroupIds] = 0u;
        }
        if (!nw) continue;
        const PlaceEns &E = s_pe[B.ens];
        const uint32_t pid = B.pid;
        const int64_t g = pid / kGroupIds;
        const uint32_t r = pre(E.grp_base + g) - pre(E.grp_base) +
                           rank_in_group(bb.bitmap + E.bm_base + g * kGroupWords, pid);
        put_birth<F64>(d, B, r, E, s_ps, b);
    }
}

template <bool F64, bool OWN>
__device__ void birth_place_body(const Dev &d, int deferred, int advance, int bid, int nblk, uint32_t *s_gp)
{
    __shared__ uint32_t s_pre[kStripes + 1];
    __shared__ uint32_t s_old[kStripes + 1];
    __shared__ uint32_t s_tb[kMaxGroupTiles];
    __shared__ bool s_last;
    __shared__ PlaceEns s_pe[PIC_MAX_ENSEMBLES];
    __shared__ PlaceSeg s_ps[2 * PIC_MAX_ENSEMBLES];
    const int64_t step = *d.step;
    const int vc = *d.vcur;
    const int p = (int)(step & 1);
    const BirthBuf bb = birth_buf(d, p), ob = birth_buf(d, 1 - p);
    if (threadIdx.x < kWave) {
        stripe_prefix(bb, d.birth_stripe_cap, s_pre);
        if (deferred) stripe_prefix(ob, d.birth_stripe_cap, s_old);
    }
    for (int en = threadIdx.x; en < d.nens; en += blockDim.x) {
        const EnsC &e = d.ens[en];
        s_pe[en] = PlaceEns{e.bm_base, e.grp_base, e.idcap, {e.seg[0], e.seg[1]}, e.nspecies};
    }
    for (int sg = threadIdx.x; sg < d.nseg; sg += blockDim.x) {
        const SegC &S = d.seg[sg];
        s_ps[sg] = PlaceSeg{S.base, S.cap, d.n_slots[sg], d.next_id[sg]};
    }
    // (with OWN the block scans the one tile of group counts into s_gp itself)
    if constexpr (OWN)
        scan_group_tile<256>(bb.gcnt, s_gp);
    else
        stage_tile_bases(d, s_tb);
    __syncthreads();
    const int64_t M = s_pre[kStripes], Mo = deferred ? (int64_t)s_old[kStripes] : 0;
    place_births<F64>(d, bb, ob, M, Mo, s_pre, s_old, s_pe, s_ps, bid, nblk,
                      [&](int64_t i) {
                          if constexpr (OWN)
                              return s_gp[i];
                          else
                              return group_prefix(d, s_tb, i);
                      });
    // The last block only updates counters that no block of this launch reads after taking
    // its ticket (each block staged them before its first barrier), and the next kernel
    // sees every write, so no device-scope fence is needed here; on gfx950 such a fence
    // writes back the XCD's L2 and costs microseconds per block.
    __syncthreads();
    if (threadIdx.x == 0) s_last = (atomicAdd(d.ticket + 1, 1u) == (unsigned)(nblk - 1));
    __syncthreads();
    if (!s_last) return;
    for (int en = threadIdx.x; en < d.nens; en += blockDim.x) {
        const PlaceEns &E = s_pe[en];
        const int64_t ngrp = (E.idcap + kGroupIds - 1) / kGroupIds;
        uint32_t m;
        if constexpr (OWN)
            m = s_gp[E.grp_base + ngrp] - s_gp[E.grp_base];
        else
            m = group_prefix(d, s_tb, E.grp_base + ngrp) - group_prefix(d, s_tb, E.grp_base);
        for (int s = 0; s < E.nspecies; ++s) {
            const int sg = E.seg[s];
            const PlaceSeg &P = s_ps[sg];
            d.n_slots[sg] = min(P.n_slots + (int64_t)m, P.cap);
            d.next_id[sg] = P.next_id + m;
            if (m) atomicAdd(d.cnt + ((int64_t)0 * d.nseg + sg) * C_NCNT + C_CREATED, (unsigned long long)m);
        }
    }
    place_reset(d, deferred, ob, vc);
    if (threadIdx.x == 0) {
        d.ticket[1] = 0u;
        atomicExch(d.vcur, 1 - vc);  // atomic: the bound may be computed in this launch
    }
    if (threadIdx.x == 0 && advance) *d.step = step + 1;
}

// With OWN (one tile of birth groups) every block scans the group counts for itself, which saves
// k_group_scan in front of it: 4.8 + 10.9 us in two launches, 11.9 in one.
template <bool F64, bool OWN>
__global__ void __launch_bounds__(256) k_birth_place(Dev d, int deferred, int advance)
{
    __shared__ uint32_t s_gp[OWN ? kGroupTile : 1];
    birth_place_body<F64, OWN>(d, deferred, advance, (int)blockIdx.x, (int)gridDim.x, s_gp);
}

// =======================================================================================
// Small runs (Dev::small > 0): at most kSmallEns ensembles of at most G chunks each and one
// tile of birth groups.  Block `en` < nsolve solves ensemble en (solve_small); with `births`,
// kSmallPlace more blocks rank and place the step's births, each scanning the one tile of
// group counts into LDS for itself, and the last block to take its ticket updates the
// placement's counters; `params`: block en also computes its segments' collision bounds.
// Such a step is bound by its chain of dependent launches (about 5 us each, whatever they
// do), so this one launch stands for k_solve1, k_solve2 and k_phi_shift, and for the births'
// k_group_scan and k_birth_place: the 2048-cell periodic run's four launches beside its pass
// took 22.5 us a step and this one 12.2, the 256-cell collisional run's pair 15.3 us and this
// one 10.4.  Above four chunks per ensemble a block could not hold a chunk per group of
// threads (1024 at most), and the chunked solve is no slower (13 + 9 us for 20 chunks).
// =======================================================================================
constexpr int kSmallPlace = 4;
constexpr int kFewBirths = 256;  // ranked by comparison (at most one per thread of the smallest block)

template <bool F64, int G>
__global__ void __launch_bounds__(G *kSolveThreads) k_solve_small(Dev d, int nsolve, int zero_q, int births,
                                                                  int deferred, int params, int advance)
{
    __shared__ SmallSolve<G> sh;
    __shared__ bool s_last;
    const int vc = *d.vcur;
    const int64_t step = *d.step;
    const int pb = (int)(step & 1);
    const BirthBuf bb = birth_buf(d, pb), ob = birth_buf(d, 1 - pb);
    if ((int)blockIdx.x < nsolve) {
        const int ei = (int)blockIdx.x, w = (int)threadIdx.x / kWave;
        const EnsC e = d.ens[ei];
        // the speed maxima of the ensemble's segments (a wave each), in the half the births'
        // placement makes current: loaded beside the charge, reduced once they are in, and only
        // then does the block take the ticket that lets them be cleared
        unsigned long long vm[kCntStripes / kWave] = {};
        if (params && w < e.nspecies) {
            const unsigned long long *row = d.vmax2 + (int64_t)(births ? 1 - vc : vc) * kCntStripes * d.nseg + (w == 0 ? e.seg[0] : e.seg[1]);
#pragma unroll
            for (int i = 0; i < kCntStripes / kWave; ++i) vm[i] = row[(int64_t)(i * kWave + lane_id()) * d.nseg];
        }
        double m2 = 0.0;
        const double emax = solve_small<F64, G, true>(d, e, ei, zero_q, sh, d.Ecell + e.gbase, d.E + e.gbase, [&] {
#pragma unroll
            for (int i = 0; i < kCntStripes / kWave; ++i) m2 = fmax(m2, __longlong_as_double((long long)vm[i]));
            if (!births) return;
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (threadIdx.x == 0) s_last = (atomicAdd(d.ticket + 6, 1u) == gridDim.x - 1);
        });
        m2 = wave_max_f64(m2);
        if (params && w < e.nspecies && lane_id() == 0) {
            const int sg = w == 0 ? e.seg[0] : e.seg[1];
            double numax, pnull;
            seg_bound(d.seg[sg], e, m2, emax, numax, pnull);
            d.numax[sg] = numax;
            d.pnull[sg] = pnull;
        }
    } else {
        __shared__ uint32_t s_pre[kStripes + 1], s_old[kStripes + 1];
        __shared__ uint32_t s_gp[kGroupTile];
        __shared__ unsigned long long s_key[kFewBirths];
        __shared__ PlaceEns s_pe[kSmallEns];
        __shared__ PlaceSeg s_ps[2 * kSmallEns];
        const int bid = (int)blockIdx.x - nsolve;
        if (threadIdx.x < kWave) {
            stripe_prefix(bb, d.birth_stripe_cap, s_pre);
            if (deferred) stripe_prefix(ob, d.birth_stripe_cap, s_old);
        }
        if ((int)threadIdx.x < d.nens) {
            const EnsC &e = d.ens[threadIdx.x];
            s_pe[threadIdx.x] = PlaceEns{e.bm_base, e.grp_base, e.idcap, {e.seg[0], e.seg[1]}, e.nspecies};
        }
        if ((int)threadIdx.x < d.nseg) {
            const SegC &S = d.seg[threadIdx.x];
            s_ps[threadIdx.x] = PlaceSeg{S.base, S.cap, d.n_slots[threadIdx.x], d.next_id[threadIdx.x]};
        }
        __syncthreads();
        const int64_t M = s_pre[kStripes], Mo = deferred ? (int64_t)s_old[kStripes] : 0;
        if (M <= kFewBirths) {
            // a few births are ranked against one another in LDS by the first block: the scan of
            // the group counts and the bitmap words would be two more round trips, which were
            // what the launch waited for (10.2 us against 7.7 at 256 cells, a dozen births)
            if (bid == 0) {
                for (int64_t k = threadIdx.x; k < Mo; k += blockDim.x) {
                    int st;
                    uint32_t idx;
                    birth_locate(d, k, st, idx, s_old);
                    const uint2 o = *(const uint2 *)&ob.births[(int64_t)st * d.birth_stripe_cap + idx];
                    const PlaceEns &E = s_pe[o.y];
                    ob.bitmap[E.bm_base + (o.x >> 5)] = 0u;
                    ob.gcnt[E.grp_base + o.x / kGroupIds] = 0u;
                }
                const int k = (int)threadIdx.x;
                Birth B{};
                unsigned long long key = 0;
                if (k < M) {
                    int st;
                    uint32_t idx;
                    birth_locate(d, k, st, idx, s_pre);
                    B = bb.births[(int64_t)st * d.birth_stripe_cap + idx];
                    key = (unsigned long long)(uint32_t)B.ens << 32 | B.pid;
                    s_key[k] = key;
                }
                __syncthreads();
                if (k < M) {
                    uint32_t r = 0;
                    for (int i = 0; i < (int)M; ++i)
                        r += (s_key[i] < key && (s_key[i] >> 32) == (key >> 32)) ? 1u : 0u;
                    put_birth<F64>(d, B, r, s_pe[B.ens], s_ps, *d.cur);
                }
                if (k < d.nens) {
                    uint32_t m = 0;
                    for (int i = 0; i < (int)M; ++i) m += (int)(s_key[i] >> 32) == k ? 1u : 0u;
                    __hip_atomic_store(d.nbens + k, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        } else {
            scan_group_tile<G * kSolveThreads>(bb.gcnt, s_gp);
            __syncthreads();
            place_births<F64>(d, bb, ob, M, Mo, s_pre, s_old, s_pe, s_ps, bid, kSmallPlace,
                              [&](int64_t i) { return s_gp[i]; });
            // the births per ensemble, for the launch's last block (which may be another one)
            if (bid == 0 && (int)threadIdx.x < d.nens) {
                const PlaceEns &E = s_pe[threadIdx.x];
                const int64_t ngrp = (E.idcap + kGroupIds - 1) / kGroupIds;
                __hip_atomic_store(d.nbens + threadIdx.x, s_gp[E.grp_base + ngrp] - s_gp[E.grp_base], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    if (!births) {
        if (advance && blockIdx.x == 0 && threadIdx.x == 0) *d.step = step + 1;
        return;
    }
    if ((int)blockIdx.x >= nsolve) {
        // every wave's memory operations are complete before the block takes its ticket
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (threadIdx.x == 0) s_last = (atomicAdd(d.ticket + 6, 1u) == gridDim.x - 1);
    }
    __syncthreads();
    if (!s_last) return;
    // The last block updates what every block read before its ticket; the births per ensemble,
    // from another block of this launch, went out and come in by device-scope atomics.
    if (threadIdx.x == 0) d.ticket[6] = 0u;
    if ((int)threadIdx.x < d.nens) {
        const EnsC &e = d.ens[threadIdx.x];
        const uint32_t m = __hip_atomic_load(d.nbens + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int s = 0; s < e.nspecies; ++s) {
            const int sg = e.seg[s];
            d.n_slots[sg] = min(d.n_slots[sg] + (int64_t)m, d.seg[sg].cap);
            d.next_id[sg] += m;
            if (m) atomicAdd(d.cnt + ((int64_t)0 * d.nseg + sg) * C_NCNT + C_CREATED, (unsigned long long)m);
        }
    }
    place_reset(d, deferred, ob, vc);
    if (threadIdx.x == 0) {
        *d.vcur = 1 - vc;
        if (advance) *d.step = step + 1;
    }
}

// Clear one half (parity -1: the current step's): its bits and counts, then its birth counts.
__global__ void k_birth_clear(Dev d, int parity)
{
    __shared__ uint32_t s_pre[kStripes + 1];
    __shared__ bool s_last;
    const int p = parity < 0 ? (int)(*d.step & 1) : parity;
    const BirthBuf bb = birth_buf(d, p);
    if (threadIdx.x < kWave) stripe_prefix(bb, d.birth_stripe_cap, s_pre);
    __syncthreads();
    const int64_t M = s_pre[kStripes];
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < M;
         k += (int64_t)gridDim.x * blockDim.x) {
        int st;
        uint32_t idx;
        birth_locate(d, k, st, idx, s_pre);
        const Birth &B = bb.births[(int64_t)st * d.birth_stripe_cap + idx];
        birth_unmark(bb, d.ens[B.ens], B.pid);
    }
    // as in the placement: the last block only resets the counts (no fence needed)
    __syncthreads();
    if (threadIdx.x == 0) s_last = (atomicAdd(d.ticket + 2, 1u) == gridDim.x - 1);
    __syncthreads();
    if (!s_last) return;
    for (int i = threadIdx.x; i < kStripes; i += blockDim.x) bb.nbirth[i] = 0u;
    if (threadIdx.x == 0) d.ticket[2] = 0u;
}

__global__ void k_advance(Dev d)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *d.step += 1;
}

// =======================================================================================
// Counting sort by cell of the FP64 form (the FP32 form runs in k_sort32): the histogram
// is in cellcnt, scanned into cursor (global positions over the concatenated segments).
// Each tile ranks its particles per cell in LDS (wave-leader reservation), reserves one
// run per cell with one HBM atomic, and scatters into the other buffer.  Absorbed slots
// are dropped.
// =======================================================================================
template <int PPT>
__global__ void __launch_bounds__(256) k_sort_scatter(Dev d, int W)
{
    extern __shared__ unsigned long long s_dyn[];
    uint32_t *sCnt = (uint32_t *)s_dyn;   // [W] counts, then bases
    __shared__ int64_t s_tpre[kMaxSeg + 1];
    __shared__ int64_t s_lim[2 * kMaxSeg];
    __shared__ int s_min;
    __shared__ bool s_last;
    const int BLOCK = blockDim.x;
    const int64_t TILE = (int64_t)BLOCK * PPT;
    sched_prefix(d, TILE, s_tpre, s_lim);
    const int64_t T = s_tpre[d.nseg];
    int64_t t0, t1;
    block_run(T, t0, t1);
    const int b = *d.cur, nb = 1 - b;
    const int lane = lane_id();
    for (int i = threadIdx.x; i < W; i += BLOCK) sCnt[i] = 0u;
    __syncthreads();
    for (int64_t t = t0; t < t1; ++t) {
        const int sg = __builtin_amdgcn_readfirstlane(seg_of_tile(s_tpre, d.nseg, t));
        const SegC &S = d.seg[sg];
        const int64_t lt = t - s_tpre[sg];
        const int64_t first = s_lim[2 * sg] + lt * TILE;
        const int64_t last = min(first + TILE, s_lim[2 * sg + 1]);
        // the whole particle is loaded up front (every load in flight at once) and kept in
        // registers until its store to the other buffer
        double xv[PPT], vx[PPT], vy[PPT], vz[PPT];
        uint32_t idv[PPT];
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const int64_t i = first + (int64_t)k * BLOCK + threadIdx.x;
            xv[k] = -1.0;
            if (i < last) {
                xv[k] = d.x[b][i];
                vx[k] = d.dvx[b][i];
                vy[k] = d.dvy[b][i];
                vz[k] = d.dvz[b][i];
                idv[k] = d.id[b][i];
            }
        }
        const Seg64 G = seg64(S, d.ens[S.ens]);
        const int64_t sbase = S.base, scap = S.cap, scb = S.cbase, sstart = d.segstart[sg];
        int cell[PPT];
        uint32_t rank[PPT];
        int mn = INT32_MAX;
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            double f;
            cell[k] = (xv[k] >= 0.0) ? (int)cell_of_x64(G, xv[k], f) : kDead;
            if (cell[k] != kDead) mn = min(mn, cell[k]);
        }
        mn = wave_min_i32(mn);
        if (threadIdx.x == 0) s_min = INT32_MAX;
        __syncthreads();
        if (lane == 0) atomicMin(&s_min, mn);
        __syncthreads();
        const int base = s_min;
        // local ranks
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const int rel = (cell[k] != kDead) ? cell[k] - base : -1;
            const int key = (rel >= 0 && rel < W) ? rel : -1;
            rank[k] = 0xFFFFFFFFu;
            unsigned long long act = __ballot(key >= 0);
            int it = 0;
            while (act != 0ull && it < 8) {
                const int leader = __ffsll((long long)act) - 1;
                const int kk = __shfl(key, leader);
                const bool mine = (key == kk) && ((act >> lane) & 1ull);
                const unsigned long long m = __ballot(mine);
                uint32_t r0 = 0;
                if (lane == leader) r0 = atomicAdd(&sCnt[kk], (uint32_t)__popcll(m));
                r0 = __shfl(r0, leader);
                if (mine) rank[k] = r0 + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                act &= ~m;
                ++it;
            }
            if ((act >> lane) & 1ull) rank[k] = atomicAdd(&sCnt[key], 1u);
        }
        __syncthreads();
        // reserve runs: counts -> global bases
        for (int i = threadIdx.x; i < W; i += BLOCK) {
            const uint32_t c = sCnt[i];
            if (c) sCnt[i] = atomicAdd(d.cursor + scb + base + i, c);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            if (cell[k] == kDead) continue;
            uint32_t pos;
            if (rank[k] != 0xFFFFFFFFu)
                pos = sCnt[cell[k] - base] + rank[k];
            else
                pos = atomicAdd(d.cursor + scb + cell[k], 1u);
            const int64_t o = sbase + (int64_t)pos - sstart;
            if (o < sbase || o >= sbase + scap) {  // histogram and slots disagree
                atomicOr(d.err, (int)E_CAP_PART);
                continue;
            }
            d.x[nb][o] = xv[k];
            d.dvx[nb][o] = vx[k];
            d.dvy[nb][o] = vy[k];
            d.dvz[nb][o] = vz[k];
            d.id[nb][o] = idv[k];
        }
        __syncthreads();
        for (int i = threadIdx.x; i < W; i += BLOCK) sCnt[i] = 0u;
        __syncthreads();
    }
    // The last block sets the slot counts from the cursors, which the other blocks changed
    // with atomics; it reads them with device-scope atomic loads (which see every block's
    // atomics across the XCDs), so no block needs a device-scope fence: on gfx950 each such
    // fence writes back its XCD's L2, which cost this kernel more the more blocks it had.
    __syncthreads();
    if (threadIdx.x == 0) s_last = (atomicAdd(d.ticket + 3, 1u) == gridDim.x - 1);
    __syncthreads();
    if (!s_last) return;
    for (int sg = threadIdx.x; sg < d.nseg; sg += BLOCK) {
        const SegC &S = d.seg[sg];
        const uint32_t end =
            __hip_atomic_load(d.cursor + S.cbase + S.ncells - 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int64_t n = (int64_t)end - d.segstart[sg];
        d.n_slots[sg] = min(max(n, (int64_t)0), S.cap);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        *d.cur = nb;
        d.ticket[3] = 0u;
    }
}

// After the scan of cellcnt into cursor: the first global position of each segment.
__global__ void k_segstart(Dev d)
{
    for (int sg = threadIdx.x; sg < d.nseg; sg += blockDim.x) d.segstart[sg] = d.cursor[d.seg[sg].cbase];
}

// =======================================================================================
// Diagnostics: alive count and sum |v|^2 per segment (FP64, fixed order per block, then
// striped into a small array reduced on the host).
// =======================================================================================
template <bool F64>
__global__ void k_diag(Dev d, int sg, double *out /* [grid][2] */)
{
    __shared__ double s_buf[8];
    const SegC &S = d.seg[sg];
    const int b = *d.cur;
    const int64_t n = d.n_slots[sg];
    double c = 0.0, v2 = 0.0;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n;
         p += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = S.base + p;
        if constexpr (!F64) {
            if (d.cell[b][i] == kDead) continue;
            v2 += speed2_rn(d.fvx[b][i], d.fvy[b][i], d.fvz[b][i]);
        } else {
            if (!(d.x[b][i] >= 0.0)) continue;
            v2 += speed2_rn(d.dvx[b][i], d.dvy[b][i], d.dvz[b][i]);
        }
        c += 1.0;
    }
    c = block_sum(c, s_buf);
    v2 = block_sum(v2, s_buf);
    if (threadIdx.x == 0) {
        out[2 * blockIdx.x] = c;
        out[2 * blockIdx.x + 1] = v2;
    }
}

// =======================================================================================
// Read-back.  One block gathers the scalars of an ensemble from the striped tallies into one
// record in host memory (k_diag_pack), and one launch gathers its node arrays as doubles into one
// run of memory (k_grid_pack), so that reading either costs one wait for the stream: each array
// copied on its own cost a wait of its own, and the stripes of every segment went to the host
// (3.4 MB a call with 128 segments).  Twenty steps and both reads of
// the 256-cell run went from 769 to 569 us; of the 64 batched ensembles, whose 64 pairs of reads
// took 39 of 131 ms, to 106 ms.
// =======================================================================================
// Slots in use of all segments, by one wave.
__device__ __forceinline__ int64_t slots_in_use(const Dev &d)
{
    int64_t n = 0;
    for (int sg = lane_id(); sg < d.nseg; sg += kWave) n += d.n_slots[sg];
    return wave_reduce(n, [](int64_t a, int64_t b) { return a + b; });
}

// With `tallied`, counts, sums of |v|^2 and field energy come from the fused step's tallies;
// otherwise from `v2` ([species][ngrid][2], k_diag) and the field-energy kernel.  A wave takes a
// quantity of a species (or the field energy) on its own, its lanes the stripes.
constexpr int kDiagThreads = 1024;
__global__ void __launch_bounds__(kDiagThreads) k_diag_pack(Dev d, int en, int tallied, const double *v2, int ngrid,
                                                            DiagPack *out)
{
    constexpr int Q = C_NCNT + S_NSUM + 2;  // counters, wall sums, alive and |v|^2
    const EnsC &e = d.ens[en];
    const int lane = lane_id(), nsp = e.nspecies;
    const int vc = *d.vcur;
    for (int t = (int)threadIdx.x / kWave; t <= nsp * Q; t += kDiagThreads / kWave) {
        const int sp = t / Q, q = t % Q;
        if (t == nsp * Q) {
            double fe = 0.0;
            if (tallied)
                for (int64_t k = lane; k < e.nchunks; k += kWave) fe += d.part[(e.chunk0 + k) * P_NPART + P_FE];
            else if (lane == 0)
                fe = d.fe[en];
            fe = wave_sum_f64(fe);
            const int64_t n = slots_in_use(d);
            if (lane == 0) {
                out->fe = fe;
                out->slots = n;
            }
        } else if (q < C_NCNT) {
            unsigned long long c = 0;
            for (int st = lane; st < kCntStripes; st += kWave) c += d.cnt[((int64_t)st * d.nseg + e.seg[sp]) * C_NCNT + q];
            c = wave_reduce(c, [](unsigned long long a, unsigned long long b) { return a + b; });
            if (lane == 0) out->cnt[sp][q] = c;
        } else {
            const int k = q - C_NCNT;
            double f = 0.0;
            if (k < S_NSUM) {
                for (int st = lane; st < kCntStripes; st += kWave)
                    f += d.sums[((int64_t)st * d.nseg + e.seg[sp]) * S_NSUM + k];
            } else if (tallied) {
                for (int st = lane; st < kCntStripes; st += kWave)
                    f += step_sums(d, vc, st, e.seg[sp])[k == S_NSUM ? T_N : T_V2];
            } else {
                for (int i = lane; i < ngrid; i += kWave) f += v2[((int64_t)sp * ngrid + i) * 2 + (k - S_NSUM)];
            }
            f = wave_sum_f64(f);
            if (lane == 0) {
                if (k < S_NSUM)
                    out->wall_v2[sp][k] = f;
                else if (k == S_NSUM)
                    out->n[sp] = f;
                else
                    out->v2[sp] = f;
            }
        }
    }
    if (threadIdx.x < (unsigned)nsp) out->numax[threadIdx.x] = d.numax[e.seg[threadIdx.x]];
    if (threadIdx.x == kDiagThreads - 1) {
        out->emax = d.emax[en];
        out->step = *d.step;
        out->neutrals = e.recycle ? d.nneu[(int64_t)*d.ncur * d.nens + en] : 0ull;
        out->err = *d.err;
    }
}

// Node arrays of ensemble `en` as doubles: out[0..1] Q per species (particle units) and, with `fields`,
// rho, phi, E.
template <bool F64>
__global__ void __launch_bounds__(256) k_grid_pack(Dev d, int en, int fields, double *out)
{
    const EnsC &e = d.ens[en];
    const int64_t nn = e.nnodes, g = e.gbase;
    const bool two = e.nspecies > 1;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < nn; j += (int64_t)gridDim.x * blockDim.x) {
        double q0, q1 = 0.0;
        if constexpr (!F64) {
            q0 = (double)(long long)d.Qi[g + j] * (1.0 / kFix);
            if (two) q1 = (double)(long long)d.Qi[d.nodes_tot + g + j] * (1.0 / kFix);
        } else {
            q0 = d.Qd[g + j];
            if (two) q1 = d.Qd[d.nodes_tot + g + j];
        }
        out[j] = q0;
        out[nn + j] = q1;
        if (!fields) continue;
        out[2 * nn + j] = d.rho[g + j];
        out[3 * nn + j] = d.phi[g + j];
        out[4 * nn + j] = d.E[g + j];
    }
}

__global__ void __launch_bounds__(kWave) k_err_out(Dev d, int32_t *out, int64_t *slots)
{
    const int64_t n = slots_in_use(d);
    if (lane_id() == 0) {
        *out = *d.err;
        *slots = n;
    }
}

// =======================================================================================
// Host launchers.
// =======================================================================================
#define LAUNCH_CHECK()                                          \
    do {                                                        \
        hipError_t _e = hipGetLastError();                      \
        if (_e != hipSuccess) return _e;                        \
    } while (0)

hipError_t launch_particles(const Dev &d, const Launch &L, hipStream_t s, bool f64, int stages, int hist,
                            bool with_params, bool depo)
{
    // the null-collision bound of every segment from this step's speed and field maxima
    if ((stages & SB_COLLIDE) && with_params) {
        hipLaunchKernelGGL(k_params, dim3(1), dim3(256), 0, s, d);
        LAUNCH_CHECK();
    }
    if (!f64) return launch_pass32(d, L, s, stages, hist, depo);
    return launch_pass64(d, L, s, stages, hist, depo && (stages & (SB_COLLIDE | SB_DEPOSIT)) == SB_COLLIDE);
}

hipError_t launch_candidates(const Dev &d, const Launch &L, hipStream_t s, bool f64, int hist, bool depo)
{
    if (f64 || inline_candidates(d, L.ppt)) return hipSuccess;
    return launch_cand32(d, L.ppt, s, hist, d.cap_tot, depo);
}

hipError_t launch_init(const Dev &d, bool f64, int sg, int64_t n, int64_t ppc, int init_mode,
                       double vth, double amp, int mode, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int B = 256;
    const int64_t G = (n + B - 1) / B;
    if (f64)
        hipLaunchKernelGGL(k_init<true>, dim3(G), dim3(B), 0, s, d, sg, n, ppc, init_mode, vth, amp, mode);
    else
        hipLaunchKernelGGL(k_init<false>, dim3(G), dim3(B), 0, s, d, sg, n, ppc, init_mode, vth, amp, mode);
    LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_vmax(const Dev &d, bool f64, hipStream_t s)
{
    dim3 g(256, d.nseg);
    if (f64)
        hipLaunchKernelGGL(k_vmax<true>, g, dim3(256), 0, s, d);
    else
        hipLaunchKernelGGL(k_vmax<false>, g, dim3(256), 0, s, d);
    LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_zero_q(const Dev &d, bool f64, hipStream_t s)
{
    if (f64)
        hipLaunchKernelGGL(k_zero_q<true>, dim3(512), dim3(256), 0, s, d);
    else
        hipLaunchKernelGGL(k_zero_q<false>, dim3(512), dim3(256), 0, s, d);
    LAUNCH_CHECK();
    return hipSuccess;
}

bool births_fit_solve(const Dev &d) { return d.ngt > 0; }

template <bool F64>
static hipError_t launch_solve_small(const Dev &d, int nsolve, int zero_q, int births, int deferred, int params,
                                     int advance, hipStream_t s)
{
    const dim3 g((unsigned)(nsolve + (births ? kSmallPlace : 0)));
    switch (d.small) {
    case 1:
        hipLaunchKernelGGL((k_solve_small<F64, 1>), g, dim3(kSolveThreads), 0, s, d, nsolve, zero_q, births, deferred,
                           params, advance);
        break;
    case 2:
        hipLaunchKernelGGL((k_solve_small<F64, 2>), g, dim3(2 * kSolveThreads), 0, s, d, nsolve, zero_q, births,
                           deferred, params, advance);
        break;
    default:
        hipLaunchKernelGGL((k_solve_small<F64, 4>), g, dim3(4 * kSolveThreads), 0, s, d, nsolve, zero_q, births,
                           deferred, params, advance);
        break;
    }
    return hipGetLastError();
}

hipError_t launch_solve(const Dev &d, bool f64, int64_t nchunks, bool zero_q, hipStream_t s,
                        bool with_births, bool with_params, bool advance)
{
    const int nc = (int)nchunks, zq = zero_q ? 1 : 0;
    const int par = with_params ? 1 : 0, bir = with_births ? 1 : 0;
    // births advance the step in the placement; without them `advance` does it here
    const int adv = with_births || advance ? 1 : 0;
    if (d.small)
        return f64 ? launch_solve_small<true>(d, d.nens, zq, bir, 1, par, adv, s)
                   : launch_solve_small<false>(d, d.nens, zq, bir, 1, par, adv, s);
    const int nscan = with_births ? d.ngt : 0;
    const int nred = with_params ? (d.nseg + kSolveThreads / kWave - 1) / (kSolveThreads / kWave) : 0;
    const int adv2 = advance && !with_births ? 1 : 0;
    const dim3 g1(nc + nscan + nred), g2(nc + (with_births ? place_blocks(d) : 0));
    if (f64) {
        hipLaunchKernelGGL(k_solve1<true>, g1, dim3(kSolveThreads), 0, s, d, nc, nscan, nred);
        hipLaunchKernelGGL(k_solve2<true>, g2, dim3(kSolveThreads), 0, s, d, zq, nc, par, adv2);
    } else {
        hipLaunchKernelGGL(k_solve1<false>, g1, dim3(kSolveThreads), 0, s, d, nc, nscan, nred);
        hipLaunchKernelGGL(k_solve2<false>, g2, dim3(kSolveThreads), 0, s, d, zq, nc, par, adv2);
    }
    LAUNCH_CHECK();
    if (d.periodic) {
        hipLaunchKernelGGL(k_phi_shift, dim3(nchunks), dim3(kSolveThreads), 0, s, d);
        LAUNCH_CHECK();
    }
    return hipSuccess;
}

hipError_t launch_field_stats(const Dev &d, bool f64, int64_t nchunks, hipStream_t s)
{
    hipLaunchKernelGGL(k_field_stats, dim3(1), dim3(kSolveThreads), 0, s, d);
    LAUNCH_CHECK();
    if (!f64) {
        hipLaunchKernelGGL(k_ecell, dim3(nchunks), dim3(kSolveThreads), 0, s, d);
        LAUNCH_CHECK();
    }
    return hipSuccess;
}

hipError_t launch_field_energy(const Dev &d, hipStream_t s)
{
    hipLaunchKernelGGL(k_field_energy, dim3(d.nens), dim3(1024), 0, s, d);
    LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_params(const Dev &d, hipStream_t s)
{
    hipLaunchKernelGGL(k_params, dim3(1), dim3(256), 0, s, d);
    LAUNCH_CHECK();
    return hipSuccess;
}

// Tile sums, then every tile's scan: on up to kOwnTiles tiles each block adds up the sums before
// its own, beyond them one block scans the sums in between.  A sort of as many particles as cells
// takes, with the sums scanned and with each block's own: 37.0 and 34.8 us at 40000 cells, 72.7
// and 71.3 at 2e6, 221 and 215 at 8e6 (1954 tiles), 320 to 328 and 322 at 1.2e7, 418 and 414 at
// 1.6e7: the launch saved is made up for by the longer sums from about 2048 tiles on.
constexpr int64_t kOwnTiles = 2048;
static hipError_t launch_scan(uint32_t *in, uint32_t *out, int64_t n, uint32_t *part, bool zero_in,
                              const int64_t *parity_step, hipStream_t s)
{
    const int64_t nb = (n + kScanTile - 1) / kScanTile;
    if (nb <= 0) return hipSuccess;
    const int zi = zero_in ? 1 : 0;
    hipLaunchKernelGGL(k_scan_sums, dim3(nb), dim3(kScanBlock), 0, s, in, n, part, parity_step);
    if (nb <= kOwnTiles) {
        hipLaunchKernelGGL(k_scan_down<true>, dim3(nb), dim3(kScanBlock), 0, s, in, out, n, part, zi, parity_step);
    } else {
        hipLaunchKernelGGL(k_scan_part, dim3(1), dim3(1024), 0, s, part, nb);
        hipLaunchKernelGGL(k_scan_down<false>, dim3(nb), dim3(kScanBlock), 0, s, in, out, n, part, zi, parity_step);
    }
    LAUNCH_CHECK();
    return hipSuccess;
}

int64_t scan_blocks(int64_t n) { return (n + kScanTile - 1) / kScanTile; }

hipError_t launch_births(const Dev &d, bool f64, bool in_step, bool advance, hipStream_t s)
{
    hipError_t e;
    if (d.small) {
        const int df = in_step ? 1 : 0, av = advance ? 1 : 0;
        e = f64 ? launch_solve_small<true>(d, 0, 0, 1, df, 0, av, s) : launch_solve_small<false>(d, 0, 0, 1, df, 0, av, s);
        if (e != hipSuccess) return e;
        if (!in_step) hipLaunchKernelGGL(k_birth_clear, dim3(64), dim3(256), 0, s, d, -1);
        return hipGetLastError();
    }
    const int deferred = in_step ? 1 : 0, adv = advance ? 1 : 0;
    const dim3 g(place_blocks(d));
    if (d.ngt == 1) {
        if (f64)
            hipLaunchKernelGGL((k_birth_place<true, true>), g, dim3(256), 0, s, d, deferred, adv);
        else
            hipLaunchKernelGGL((k_birth_place<false, true>), g, dim3(256), 0, s, d, deferred, adv);
    } else {
        // the group-count scan: one block per tile up to kMaxGroupTiles tiles, the global
        // scan above that
        if (d.ngt > 0) {
            hipLaunchKernelGGL(k_group_scan, dim3(d.ngt), dim3(256), 0, s, d);
            LAUNCH_CHECK();
        } else if ((e = launch_scan(d.gcnt, d.gpre, d.g_tot, d.scanpart, false, d.step, s)) != hipSuccess) {
            return e;
        }
        if (f64)
            hipLaunchKernelGGL((k_birth_place<true, false>), g, dim3(256), 0, s, d, deferred, adv);
        else
            hipLaunchKernelGGL((k_birth_place<false, false>), g, dim3(256), 0, s, d, deferred, adv);
    }
    LAUNCH_CHECK();
    if (!in_step) {
        hipLaunchKernelGGL(k_birth_clear, dim3(64), dim3(256), 0, s, d, -1);
        LAUNCH_CHECK();
    }
    return hipSuccess;
}

hipError_t launch_births_clear_all(const Dev &d, hipStream_t s)
{
    hipLaunchKernelGGL(k_birth_clear, dim3(64), dim3(256), 0, s, d, 0);
    hipLaunchKernelGGL(k_birth_clear, dim3(64), dim3(256), 0, s, d, 1);
    LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_advance(const Dev &d, hipStream_t s)
{
    hipLaunchKernelGGL(k_advance, dim3(1), dim3(64), 0, s, d);
    LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_sort_prepare(const Dev &d, hipStream_t s)
{
    if (d.cells_tot <= kOneScanMax) {
        hipLaunchKernelGGL(k_sort_scan, dim3(1), dim3(kOneThreads), 0, s, d);
        return hipGetLastError();
    }
    hipError_t e = launch_scan(d.cellcnt, d.cursor, d.cells_tot, d.scanpart, true, nullptr, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_segstart, dim3(1), dim3(256), 0, s, d);
    return hipGetLastError();
}

hipError_t launch_sort(const Dev &d, bool f64, const Launch &L, hipStream_t s)
{
    hipError_t e = launch_sort_prepare(d, s);
    if (e != hipSuccess) return e;
    if (!f64) return launch_sort32_scatter(d, L.sort_ppt, L.window, s, d.cap_tot, L.sort_nt != 0);
    // the scatter's static runs of tiles are short: 8 x Launch::grid blocks (a sweep
    // from 1/2x to 8x on the 4e7-particle slab: 1.33, 1.07, 0.92, 0.85, 0.83 ms)
    const size_t lds = (size_t)L.window * 4;
    hipLaunchKernelGGL((k_sort_scatter<4>), dim3(8 * L.grid), dim3(L.block), lds, s, d, L.window);
    LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_diag_pack(const Dev &d, int en, bool tallied, const double *v2, int ngrid, DiagPack *out,
                            hipStream_t s)
{
    hipLaunchKernelGGL(k_diag_pack, dim3(1), dim3(kDiagThreads), 0, s, d, en, tallied ? 1 : 0, v2, ngrid, out);
    return hipGetLastError();
}

hipError_t launch_grid_pack(const Dev &d, bool f64, int en, int64_t nn, bool fields, double *out, hipStream_t s)
{
    const dim3 g((unsigned)std::min<int64_t>((nn + 255) / 256, 1024));
    if (f64)
        hipLaunchKernelGGL(k_grid_pack<true>, g, dim3(256), 0, s, d, en, fields ? 1 : 0, out);
    else
        hipLaunchKernelGGL(k_grid_pack<false>, g, dim3(256), 0, s, d, en, fields ? 1 : 0, out);
    return hipGetLastError();
}

hipError_t launch_err_out(const Dev &d, int32_t *out, int64_t *slots, hipStream_t s)
{
    hipLaunchKernelGGL(k_err_out, dim3(1), dim3(kWave), 0, s, d, out, slots);
    return hipGetLastError();
}

hipError_t launch_diag(const Dev &d, bool f64, int sg, double *out, int grid, hipStream_t s)
{
    if (f64)
        hipLaunchKernelGGL(k_diag<true>, dim3(grid), dim3(256), 0, s, d, sg, out);
    else
        hipLaunchKernelGGL(k_diag<false>, dim3(grid), dim3(256), 0, s, d, sg, out);
    LAUNCH_CHECK();
    return hipSuccess;
}

}  // namespace pic
