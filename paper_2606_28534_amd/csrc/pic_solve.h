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
    static constexpr int W = kSolveThreads / kWave;
    double E[G][kChunk + 1];  // the raw densities while smoothing, then each chunk's node E
    double scan[3][G][W];     // the three scans' wave totals (one each: no barrier between uses)
    double red[G][3][W], red2[G][2][W], rho0[G];
    double em[G * W], nabs[2];
};

// Inclusive scan over each group of kSolveThreads threads; s_buf is the group's, used once.
__device__ __forceinline__ double group_incl_scan(double v, double *s_buf)
{
    constexpr int W = kSolveThreads / kWave;
    const int w = (threadIdx.x % kSolveThreads) / kWave;
    v = wave_incl_scan(v);
    if (lane_id() == kWave - 1) s_buf[w] = v;
    __syncthreads();
    double t[W - 1];
#pragma unroll
    for (int i = 0; i < W - 1; ++i) t[i] = s_buf[i];  // (all in flight at once)
    double add = 0.0;
#pragma unroll
    for (int i = 0; i < W - 1; ++i) add += i < w ? t[i] : 0.0;
    return v + add;
}

// A chunk's interior nodes, nodes below N and summed prefix weights (exact small integers):
// n1 of its nodes are interior, the k-th of them the k-th term of dd, and node 0 counts in cnt
// alone.
__device__ __forceinline__ void chunk_counts(int64_t a, int64_t nn, int64_t N, double &n1, double &dd, double &cnt)
{
    const int64_t b = min(min(a + kChunk, nn), N);
    const int64_t i = max(b - max(a, (int64_t)1), (int64_t)0);
    n1 = (double)i;
    dd = (double)(i * (i + 1) / 2);
    cnt = (double)max(b - a, (int64_t)0);
}

// Solves ensemble `ei` from d.Qi / d.Qd.  The node field goes to Eout (unless null) and the
// gather table of the FP32 form to `table` (global memory or LDS).  FULL also writes rho and
// phi, the field-energy partials and max |E| (also returned, by every thread), and with zero_q
// clears the charge.  `mid` runs in every thread after the block's first barrier, when every load
// issued before the call has come in.
//
// What bounds it is the chain from the charge to the field: two round trips to memory, three
// block-wide FP64 scans (about 0.5 us each) and one of sums.  So the charge is loaded without
// waiting for the ensemble's constants where they are not needed to find it, every thread
// scans the few chunk aggregates for itself, and no LDS word is written twice between barriers:
// 2048 periodic nodes 10.7 -> 9.3 us, with the adjoint's forward step around it 11.1 -> 9.7.
template <bool F64, int G, bool FULL, typename Mid>
__device__ __forceinline__ double solve_small(const Dev &d, const EnsC &e, int ei, int zero_q, SmallSolve<G> &sh,
                                              float2 *table, double *Eout, Mid mid)
{
    constexpr int W = SmallSolve<G>::W, NPT = kNodesPerThread;
    const int g = threadIdx.x / kSolveThreads, u = threadIdx.x % kSolveThreads, w = u / kWave;
    const int64_t a = (int64_t)g * kChunk, j0 = a + (int64_t)u * NPT;
    // the charge as stored (fixed point, or doubles' bits)
    unsigned long long raw[2][NPT];
    auto load = [&](int64_t base, int64_t nodes) {
        const unsigned long long *Q = F64 ? (const unsigned long long *)d.Qd : d.Qi;
#pragma unroll
        for (int q = 0; q < NPT; ++q) raw[0][q] = Q[base + (j0 + q < nodes ? j0 + q : 0)];
        if (d.nspecies > 1) {
#pragma unroll
            for (int q = 0; q < NPT; ++q) raw[1][q] = Q[d.nodes_tot + base + (j0 + q < nodes ? j0 + q : 0)];
        }
    };
    if (d.nens == 1)
        load(0, d.nodes_tot);
    else
        load(e.gbase, e.nnodes);
    const int64_t N = e.ncells, nn = e.nnodes;
    const double dx = e.dx, ce = e.dx / e.eps0;
    if (e.floating && threadIdx.x < kWave) {
        // floating walls (R22): the particles absorbed so far at the left wall, per species
        double nabs[2] = {0.0, 0.0};
        for (int st = threadIdx.x; st < kCntStripes; st += kWave) {
#pragma unroll
            for (int s = 0; s < 2; ++s)
                if (s < e.nspecies) nabs[s] += (double)d.cnt[((int64_t)st * d.nseg + e.seg[s]) * C_NCNT + C_WALL_L];
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const double t = wave_sum_f64(nabs[s]);
            if (threadIdx.x == 0) sh.nabs[s] = t;
        }
    }
    double rq[NPT];
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
        auto val = [&](unsigned long long r) {
            if constexpr (F64)
                return __longlong_as_double((long long)r);
            else
                return (double)(long long)r * (1.0 / kFix);
        };
        double c = 0.0;
        c += e.qw[0] * val(raw[0][q]);
        if (d.nspecies > 1) c += e.qw[1] * val(raw[1][q]);
        rq[q] = j0 + q < nn ? c / node_vol(e, j0 + q) : 0.0;
    }
    if (FULL && zero_q) {
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            if (j0 + q >= nn) continue;
            for (int s = 0; s < d.nspecies; ++s) {
                if constexpr (!F64)
                    d.Qi[(int64_t)s * d.nodes_tot + e.gbase + j0 + q] = 0ull;
                else
                    d.Qd[(int64_t)s * d.nodes_tot + e.gbase + j0 + q] = 0.0;
            }
        }
    }
    const int p = e.smooth;
    if (p > 0) {
        double *den = &sh.E[0][0];
#pragma unroll
        for (int q = 0; q < NPT; ++q)
            if (j0 + q < nn) den[j0 + q] = rq[q];
        __syncthreads();
        const double pscale = 1.0 / (double)(1 << (2 * p));
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            double r = 0.0;
            double c = 1.0;  // C(2p, k), exact in binary64
            if (j0 + q < nn)
                for (int k = 0; k <= 2 * p; ++k) {
                    r += c * den[smooth_fold(e, j0 + q - p + k)];
                    c = c * (double)(2 * p - k) / (double)(k + 1);
                }
            rq[q] = r * pscale;
        }
        __syncthreads();
    }
    // first pass: the chunk's sums of rho, of its prefix and of the charge
    double loc = 0.0, totq = 0.0;
    double rho_loc[NPT];
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
        const int64_t j = j0 + q;
        if (j < nn) totq += rq[q] * node_vol(e, j);
        rho_loc[q] = (j >= 1 && j <= N - 1) ? rq[q] : 0.0;
        loc += rho_loc[q];
    }
    double run = group_incl_scan(loc, sh.scan[0][g]) - loc;
    mid();
    double sumpre = 0.0;
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
        run += rho_loc[q];
        if (j0 + q < N) sumpre += run;
    }
    {
        double v[3] = {loc, sumpre, totq};
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (i < 2 || e.periodic) v[i] = wave_sum_f64(v[i]);
        if (lane_id() == 0) {
#pragma unroll
            for (int i = 0; i < 3; ++i) sh.red[g][i][w] = v[i];
        }
        if (u == 0) sh.rho0[g] = rq[0];
    }
    __syncthreads();
    // The scan of the chunk aggregates (see solve2_body), by every thread, in the order of the
    // wave's scans and sums there: chunks beyond the ensemble's count as zero.
    double C0 = 0.0, F0 = 0.0, Stot, Ctot, bg = 0.0;
    {
        double sum[3][G];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int c = 0; c < G; ++c) {
                double r = 0.0;
#pragma unroll
                for (int k = 0; k < W; ++k) r += sh.red[c][i][k];
                sum[i][c] = c < e.nchunks ? r : 0.0;
            }
        auto total = [](const double(&v)[G]) {
            if constexpr (G == 4)
                return (v[0] + v[2]) + (v[1] + v[3]);
            else if constexpr (G == 2)
                return v[0] + v[1];
            else
                return v[0];
        };
        auto incl = [](const double(&v)[G], int c) {
            if (c == 0) return v[0];
            if (c == 1) return v[1 % G] + v[0];
            if (c == 2) return (v[2 % G] + v[1 % G]) + v[0];
            return (v[3 % G] + v[2 % G]) + (v[1 % G] + v[0]);
        };
        if (e.periodic) bg = -total(sum[2]) / e.L;
        double A[G], fin[G];
        double apre = 0.0;
#pragma unroll
        for (int c = 0; c < G; ++c) {
            double n1, dd, cnt;
            chunk_counts((int64_t)c * kChunk, nn, N, n1, dd, cnt);
            A[c] = sum[0][c] + bg * n1;
            apre = incl(A, c) - A[c];
            if (c == g) C0 = apre;
            const double B = sum[1][c] + bg * dd;
            fin[c] = c < e.nchunks ? cnt * apre + B : 0.0;
            if (c == g) F0 = incl(fin, c) - fin[c];
        }
        Stot = total(fin);
        Ctot = total(A);
    }
    // Reading R22: floating walls fix E_{1/2} by Gauss's law over the left wall; otherwise
    // phi_N = 0 (or periodicity) fixes it.
    double Eh;
    if (e.floating) {
        const double sigL = e.qw[0] * sh.nabs[0] + (e.nspecies > 1 ? e.qw[1] * sh.nabs[1] : 0.0);
        Eh = (sigL + sh.rho0[0] * node_vol(e, 0)) / e.eps0;
    } else {
        Eh = -ce * Stot / (double)N;
    }
    // second pass
    double rl[NPT];
    loc = 0.0;
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
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
    const double cex = group_incl_scan(loc, sh.scan[1][g]) - loc;
    double Cj[NPT];
    double c = C0 + cex;
    double csum = 0.0;
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
        c += rl[q];
        Cj[q] = c;
        csum += (j0 + q < N) ? c : 0.0;
    }
    double phi[NPT] = {};
    double F = 0.0;
    if (FULL) F = F0 + (group_incl_scan(csum, sh.scan[2][g]) - csum);
    double emax = 0.0, phisum = 0.0, fe = 0.0;
    int nonfin = 0;
    double Cprev = (j0 == 0) ? 0.0 : (Cj[0] - rl[0]);
    double *s_E = sh.E[g];
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
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
                    const double Elast = Eh + ce * Ctot;  // E_{N-1/2}
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
    if constexpr (FULL) {
        if (!e.periodic) {
#pragma unroll
            for (int q = 0; q < NPT; ++q)
                if (j0 + q < nn) d.phi[e.gbase + j0 + q] = phi[q];
        }
        const double em = wave_max_f64(emax), sf = wave_sum_f64(fe);
        const double sp = e.periodic ? wave_sum_f64(phisum) : 0.0;
        if (lane_id() == 0) {
            sh.em[threadIdx.x / kWave] = em;
            sh.red2[g][0][w] = sp;
            sh.red2[g][1][w] = sf;
        }
    }
    if constexpr (!F64) {
        // the node after the chunk's last cell: the periodic wrap, or the next chunk's first
        // node from this chunk's last C and that node's density
        const int64_t L = min((int64_t)kChunk, N - a);
        if (L > 0) {
            if (e.periodic && a + L == N) {
                if (u == 0) s_E[L] = 0.5 * ((Eh + ce * Ctot) + (Eh + ce * 0.0));
            } else if (L == kChunk && u == kSolveThreads - 1) {
                const int64_t jn = a + kChunk;
                const double rn = sh.rho0[g + 1 < G ? g + 1 : g];  // (N < G kChunk: the next chunk exists)
                const double Cl = Cj[NPT - 1];  // C_{jn-1}
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
    } else if (FULL) {
        __syncthreads();
    }
    if (nonfin) atomicOr(d.err, (int)E_NONFINITE);
    if constexpr (FULL) {
        auto part = [&](int ck, int k) {
            double r = 0.0;
#pragma unroll
            for (int i = 0; i < W; ++i) r += sh.red2[ck][k][i];
            return r;
        };
        emax = sh.em[0];
#pragma unroll
        for (int i = 1; i < G * W; ++i) emax = fmax(emax, sh.em[i]);
        if (threadIdx.x == 0) d.emax[ei] = emax;
        if (u == 0 && g < e.nchunks)
            d.part[(e.chunk0 + g) * P_NPART + P_FE] = 0.5 * e.eps0 * part(g, 1);  // this chunk's field energy
        if (e.periodic) {
            double v[G];
#pragma unroll
            for (int ck = 0; ck < G; ++ck) v[ck] = ck < e.nchunks ? part(ck, 0) : 0.0;
            double ps = v[0];
            if constexpr (G == 4)
                ps = (v[0] + v[2]) + (v[1] + v[3]);
            else if constexpr (G == 2)
                ps = v[0] + v[1];
            const double mean = ps / (double)N;
#pragma unroll
            for (int q = 0; q < NPT; ++q)
                if (j0 + q < nn) d.phi[e.gbase + j0 + q] = phi[q] - mean;
        }
    }
    return emax;
}

}  // namespace pic
