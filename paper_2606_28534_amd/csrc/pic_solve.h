// pic_solve.h -- node helpers of the field solve and the one-block solve of a small ensemble.
#pragma once
#include "pic_device.h"

namespace pic {

constexpr int kNodesPerThread = kChunk / kSolveThreads;

__device__ __forceinline__ double node_vol(const EnsC &e, int64_t j)
{
    if (!e.periodic && (j == 0 || j == e.ncells)) return 0.5 * e.dx;
    return e.dx;
}

// Reading R23: p passes of the 1-2-1 filter equal one binomial stencil of width 2p + 1
// (weights C(2p, p + i) / 4^p) applied to the periodic extension of rho, or on a bounded
// grid to its even extension across both walls (a pass maps an even extension to an even
// extension, with rho_{-1} = rho_1 at the wall, so the passes compose into the stencil).
// Each node therefore reads its 2p + 1 neighbours once instead of p sweeps over the grid.
// smooth_fold maps a node index in [-p, nn - 1 + p] onto the grid (p <= 4 and N >= 2, so a
// couple of wraps or reflections at most).
__device__ __forceinline__ int64_t smooth_fold(const EnsC &e, int64_t m)
{
    const int64_t n = e.ncells;
    if (e.periodic) {
        while (m < 0) m += n;
        while (m >= n) m -= n;
        return m;
    }
    for (int it = 0; it < 8; ++it) {
        if (m < 0)
            m = -m;
        else if (m > n)
            m = 2 * n - m;
        else
            break;
    }
    return m;
}

// One species' deposited charge at NQ nodes (offsets into the node arrays), all loads
// issued before the first is used.
template <bool F64, int NQ>
__device__ __forceinline__ void node_q_row(const Dev &d, int64_t row, const int64_t (&at)[NQ],
                                           double (&Q)[NQ])
{
    if constexpr (!F64) {
        unsigned long long raw[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) raw[q] = d.Qi[row + at[q]];
#pragma unroll
        for (int q = 0; q < NQ; ++q) Q[q] = (double)(long long)raw[q] * (1.0 / kFix);
    } else {
#pragma unroll
        for (int q = 0; q < NQ; ++q) Q[q] = d.Qd[row + at[q]];
    }
}

// Charge density sum_s q_s w_s Q_s(j) / vol(j) at NQ nodes per thread (entries with ok[q]
// false give 0).  The loads are unconditional (node 0 stands in for unused entries), so the
// thread waits for memory once instead of once per node and species.
template <bool F64, int NQ>
__device__ __forceinline__ void node_rho_raw(const Dev &d, const EnsC &e, const int64_t (&j)[NQ],
                                             const bool (&ok)[NQ], double (&r)[NQ])
{
    static_assert(sizeof(e.qw) / sizeof(e.qw[0]) == 2, "at most two charged species");
    int64_t at[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) at[q] = e.gbase + (ok[q] ? j[q] : 0);
    double Q0[NQ], Q1[NQ];
    node_q_row<F64, NQ>(d, 0, at, Q0);
    const bool two = e.nspecies > 1;
    if (two) node_q_row<F64, NQ>(d, d.nodes_tot, at, Q1);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        double c = 0.0;
        c += e.qw[0] * Q0[q];
        if (two) c += e.qw[1] * Q1[q];
        r[q] = ok[q] ? c / node_vol(e, j[q]) : 0.0;
    }
}

// =======================================================================================
// The solve of an ensemble of at most G chunks by one block of G x kSolveThreads threads, a
// chunk to each group of kSolveThreads: the two passes of the chunked solve (k_solve1,
// k_solve2) with the chunk aggregates in LDS instead of two launches with a round trip through
// memory between them.  Every sum is taken in the same order, so the fields are the same to
// the last bit.
// =======================================================================================
template <int G>
struct SmallSolve {
    double E[G][kChunk + 1];  // the raw densities while smoothing, then each chunk's node E
    double buf[G][kSolveThreads / kWave], red[G][6][kSolveThreads / kWave];
    double agg[G][A_NAGG], C0[G], F0[G], part[G][2];
    double em[G * (kSolveThreads / kWave)];
    double Eh, bg, Ctot, mean;
};

// Inclusive scan over each group of kSolveThreads threads.
__device__ __forceinline__ double group_incl_scan(double v, double *s_buf)
{
    const int w = (threadIdx.x % kSolveThreads) / kWave;
    v = wave_incl_scan(v);
    if (lane_id() == kWave - 1) s_buf[w] = v;
    __syncthreads();
    double add = 0.0;
    for (int i = 0; i < w; ++i) add += s_buf[i];
    __syncthreads();
    return v + add;
}

template <int N>
__device__ __forceinline__ void group_sums(double (&v)[N], double (*s)[kSolveThreads / kWave])
{
    const int w = (threadIdx.x % kSolveThreads) / kWave;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = wave_sum_f64(v[i]);
    if (lane_id() == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) s[i][w] = v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        double r = 0.0;
        for (int k = 0; k < kSolveThreads / kWave; ++k) r += s[i][k];
        v[i] = r;
    }
    __syncthreads();
}

// Solves ensemble `ei` from d.Qi / d.Qd.  The node field goes to Eout (unless null) and the
// gather table of the FP32 form to `table` (global memory or LDS).  FULL also writes rho and
// phi, the field-energy partials and max |E| (also returned, by every thread), and with zero_q
// clears the charge.
template <bool F64, int G, bool FULL>
__device__ __forceinline__ double solve_small(const Dev &d, const EnsC &e, int ei, int zero_q, SmallSolve<G> &sh,
                                            float2 *table, double *Eout)
{
    const int g = threadIdx.x / kSolveThreads, u = threadIdx.x % kSolveThreads;
    const int64_t N = e.ncells, nn = e.nnodes;
    const int64_t a = (int64_t)g * kChunk, j0 = a + (int64_t)u * kNodesPerThread;
    const double dx = e.dx, ce = e.dx / e.eps0;
    double rq[kNodesPerThread];
    {
        int64_t jq[kNodesPerThread];
        bool ok[kNodesPerThread];
#pragma unroll
        for (int q = 0; q < kNodesPerThread; ++q) {
            jq[q] = j0 + q;
            ok[q] = jq[q] < nn;
        }
        node_rho_raw<F64, kNodesPerThread>(d, e, jq, ok, rq);
        if (FULL && zero_q) {
#pragma unroll
            for (int q = 0; q < kNodesPerThread; ++q) {
                if (!ok[q]) continue;
                for (int s = 0; s < e.nspecies; ++s) {
                    if constexpr (!F64)
                        d.Qi[(int64_t)s * d.nodes_tot + e.gbase + jq[q]] = 0ull;
                    else
                        d.Qd[(int64_t)s * d.nodes_tot + e.gbase + jq[q]] = 0.0;
                }
            }
        }
    }
    const int p = e.smooth;
    if (p > 0) {
        double *raw = &sh.E[0][0];
#pragma unroll
        for (int q = 0; q < kNodesPerThread; ++q)
            if (j0 + q < nn) raw[j0 + q] = rq[q];
        __syncthreads();
        const double pscale = 1.0 / (double)(1 << (2 * p));
#pragma unroll
        for (int q = 0; q < kNodesPerThread; ++q) {
            double r = 0.0;
            double c = 1.0;  // C(2p, k), exact in binary64
            if (j0 + q < nn)
                for (int k = 0; k <= 2 * p; ++k) {
                    r += c * raw[smooth_fold(e, j0 + q - p + k)];
                    c = c * (double)(2 * p - k) / (double)(k + 1);
                }
            rq[q] = r * pscale;
        }
        __syncthreads();
    }
    // first pass: the chunk's aggregates
    double loc = 0.0, sumpre = 0.0, totq = 0.0, n1 = 0.0, dd = 0.0, cnt = 0.0;
    double rho_loc[kNodesPerThread];
#pragma unroll
    for (int q = 0; q < kNodesPerThread; ++q) {
        const int64_t j = j0 + q;
        double r = 0.0;
        if (j < nn) {
            r = rq[q];
            totq += r * node_vol(e, j);
        }
        rq[q] = r;
        rho_loc[q] = (j >= 1 && j <= N - 1) ? r : 0.0;
        loc += rho_loc[q];
    }
    const double excl = group_incl_scan(loc, sh.buf[g]) - loc;
    double run = excl;
    int64_t c1 = 0;
    {
        const int64_t lo = max(a, (int64_t)1), hi = min(j0, N);  // interior nodes in [a, j0)
        c1 = hi > lo ? hi - lo : 0;
    }
#pragma unroll
    for (int q = 0; q < kNodesPerThread; ++q) {
        const int64_t j = j0 + q;
        run += rho_loc[q];
        if (j >= 1 && j <= N - 1) {
            ++c1;
            n1 += 1.0;
        }
        if (j < N) {  // m in [0, N-1]
            sumpre += run;
            dd += (double)c1;
            cnt += 1.0;
        }
    }
    {
        double v[6] = {loc, sumpre, totq, n1, dd, cnt};
        group_sums<6>(v, sh.red[g]);
        if (u == 0) {
            double *x = sh.agg[g];
            x[A_SUMRHO] = v[0];
            x[A_SUMPRE] = v[1];
            x[A_TOTQ] = v[2];
            x[A_N1] = v[3];
            x[A_D] = v[4];
            x[A_CNT] = v[5];
            x[A_RHO0] = rq[0];
        }
    }
    __syncthreads();
    // the scan of the chunk aggregates, lane c taking chunk c (see solve2_body)
    if (threadIdx.x < kWave) {
        const int c = (int)threadIdx.x;
        const bool in = c < e.nchunks;
        double nabs[2] = {0.0, 0.0};
        if (e.floating)
            for (int st = c; st < kCntStripes; st += kWave) {
#pragma unroll
                for (int s = 0; s < 2; ++s)
                    if (s < e.nspecies)
                        nabs[s] += (double)d.cnt[((int64_t)st * d.nseg + e.seg[s]) * C_NCNT + C_WALL_L];
            }
        const double *x = sh.agg[in ? c : 0];
        const double tqs = wave_sum_f64(in ? x[A_TOTQ] : 0.0);
        const double bg = e.periodic ? -tqs / e.L : 0.0;
        double A = 0.0, gg = 0.0, n = 0.0;
        if (in) {
            const double Ac = x[A_SUMRHO] + bg * x[A_N1];
            const double Bc = x[A_SUMPRE] + bg * x[A_D];
            gg += x[A_CNT] * A + Bc;
            n += x[A_CNT];
            A += Ac;
        }
        const double apre = wave_incl_scan<G>(A) - A;
        const double fin = n * apre + gg;
        const double fpre = wave_incl_scan<G>(fin) - fin;
        const double Stot = wave_sum_f64(fin), Ctot = wave_sum_f64(A);
        const double nab0 = wave_sum_f64(nabs[0]), nab1 = wave_sum_f64(nabs[1]);
        if (c < G) {
            sh.C0[c] = apre;
            sh.F0[c] = fpre;
        }
        const double sigL = e.qw[0] * nab0 + (e.nspecies > 1 ? e.qw[1] * nab1 : 0.0);
        if (c == 0) {
            sh.bg = bg;
            sh.Ctot = Ctot;
            if (e.floating)
                sh.Eh = (sigL + sh.agg[0][A_RHO0] * node_vol(e, 0)) / e.eps0;
            else
                sh.Eh = -ce * Stot / (double)N;
        }
    }
    __syncthreads();
    // second pass
    const double bg = sh.bg, Eh = sh.Eh;
    double rl[kNodesPerThread];
    loc = 0.0;
#pragma unroll
    for (int q = 0; q < kNodesPerThread; ++q) {
        const int64_t j = j0 + q;
        double r = 0.0;
        if (j < nn) {
            const double rj = rq[q] + bg;
            if (FULL) d.rho[e.gbase + j] = e.periodic ? rj : rq[q];
            if (j >= 1 && j <= N - 1) r = rj;
        }
        rl[q] = r;
        loc += r;
    }
    const double cex = group_incl_scan(loc, sh.buf[g]) - loc;
    double Cj[kNodesPerThread];
    double c = sh.C0[g] + cex;
    double csum = 0.0;
#pragma unroll
    for (int q = 0; q < kNodesPerThread; ++q) {
        c += rl[q];
        Cj[q] = c;
        csum += (j0 + q < N) ? c : 0.0;
    }
    double phi[kNodesPerThread] = {};
    double F = 0.0;
    if (FULL) F = sh.F0[g] + (group_incl_scan(csum, sh.buf[g]) - csum);
    double emax = 0.0, phisum = 0.0, fe = 0.0;
    int nonfin = 0;
    double Cprev = (j0 == 0) ? 0.0 : (Cj[0] - rl[0]);
    double *s_E = sh.E[g];
#pragma unroll
    for (int q = 0; q < kNodesPerThread; ++q) {
        const int64_t j = j0 + q;
        if (j < nn) {
            if (FULL) {
                double ph = -dx * ((double)j * Eh + ce * F);
                if (!e.periodic && !e.floating && j == N) ph = 0.0;
                if (j == 0) ph = 0.0;
                phi[q] = ph;
                phisum += ph;
            }
            const double Em = Eh + ce * Cprev;  // E_{j-1/2} (j >= 1)
            const double Ep = Eh + ce * Cj[q];  // E_{j+1/2} (j <= N-1)
            double Ej;
            if (e.periodic) {
                if (j == 0) {
                    const double Elast = Eh + ce * sh.Ctot;  // E_{N-1/2}
                    Ej = 0.5 * (Elast + Ep);
                } else {
                    Ej = 0.5 * (Em + Ep);
                }
            } else if (j == 0) {
                Ej = Eh - rq[q] * node_vol(e, 0) / e.eps0;
            } else if (j == N) {
                Ej = Em + rq[q] * node_vol(e, N) / e.eps0;
            } else {
                Ej = 0.5 * (Em + Ep);
            }
            if (Eout) Eout[j] = Ej;
            if constexpr (!F64) s_E[j - a] = Ej;
            if (!isfinite(Ej)) nonfin = 1;
            emax = fmax(emax, fabs(Ej));
            if (FULL) fe += Ej * Ej * node_vol(e, j);
            if (j < N) F += Cj[q];
            Cprev = Cj[q];
        }
    }
    if constexpr (!F64) {
        // the node after the chunk's last cell: the periodic wrap, or the next chunk's first
        // node from this chunk's last C and that node's density
        const int64_t L = min((int64_t)kChunk, N - a);
        if (L > 0) {
            if (e.periodic && a + L == N) {
                if (u == 0) s_E[L] = 0.5 * ((Eh + ce * sh.Ctot) + (Eh + ce * 0.0));
            } else if (L == kChunk && u == kSolveThreads - 1) {
                const int64_t jn = a + kChunk;
                const double rn = sh.agg[g + 1 < G ? g + 1 : g][A_RHO0];  // (N < G kChunk: the next chunk exists)
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
        for (int64_t j = a + u; j < a + L; j += kSolveThreads) {
            const double E0 = s_E[j - a], E1 = s_E[j - a + 1];
            table[j] = make_float2((float)E0, (float)(E1 - E0));
        }
    }
    if (nonfin) atomicOr(d.err, (int)E_NONFINITE);
    if constexpr (FULL) {
        const double em = wave_max_f64(emax);
        if (lane_id() == 0) sh.em[threadIdx.x / kWave] = em;
        double fv[2] = {phisum, fe};
        group_sums<2>(fv, sh.red[g]);
        if (u == 0) {
            sh.part[g][0] = fv[0];
            if (g < e.nchunks) {
                d.part[(e.chunk0 + g) * P_NPART + P_PHISUM] = fv[0];
                d.part[(e.chunk0 + g) * P_NPART + P_FE] = 0.5 * e.eps0 * fv[1];  // this chunk's field energy
            }
        }
        __syncthreads();
        emax = sh.em[0];
        for (int i = 1; i < G * (kSolveThreads / kWave); ++i) emax = fmax(emax, sh.em[i]);
        if (threadIdx.x == 0) d.emax[ei] = emax;
        double mean = 0.0;
        if (e.periodic) {
            if (threadIdx.x < kWave) {
                const double ps = wave_sum_f64((int)threadIdx.x < e.nchunks ? sh.part[threadIdx.x][0] : 0.0);
                if (threadIdx.x == 0) sh.mean = ps / (double)N;
            }
            __syncthreads();
            mean = sh.mean;
        }
#pragma unroll
        for (int q = 0; q < kNodesPerThread; ++q)
            if (j0 + q < nn) d.phi[e.gbase + j0 + q] = e.periodic ? phi[q] - mean : phi[q];
    }
    return emax;
}

}  // namespace pic
