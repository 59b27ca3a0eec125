// pic_adjoint.hip -- discrete adjoint of the collisionless push + deposit + Poisson window
// (FP32 cell+offset forward, one periodic species on a fixed neutralising background,
// B = 0).  The floor of the cell index is treated as locally constant, so each step's
// adjoint is exact for the discrete forward:
//   x^{n+1} = x^n + dt v^{n+1/2},  v^{n+1/2} = v^{n-1/2} + dt (q/m) (E^n(x^n) + E_ext),
//   E^n = -D phi,  phi = S rho',  rho' = (q w / dx) P Q(x^n)
// with D the centred difference, S the zero-mean periodic Poisson solve (symmetric) and P
// the projection that removes the mean (the neutralising background).  Backwards:
//   lv += dt lx;  la = dt (q/m) lv;  lE_j += w_j(x) la;  lx += la (E_{j+1} - E_j) / dx;
//   lEext += la;  lQ = (q w / dx) S D lE;  lx += (lQ_{j+1} - lQ_j) / dx.
// Adjoint accumulators are FP64.
#include <algorithm>

#include "pic_device.h"
#include "pic_kernels.h"
#include "pic_particle.h"
#include "pic_solve.h"

namespace pic {

// =======================================================================================
// Windows on small grids (at most kSmallChunks solve chunks): one launch per step in either
// direction.  A window is hundreds of steps of a few hundred thousand particles that all stay in
// the caches, so it is bound by the number of dependent launches, and by the one-block solve
// between the particle kernels.  Here every block solves the field (forward) or the transposed
// field (backward) for itself in LDS, a chunk per group of kSolveThreads threads, and then
// takes its particles, so the solve costs neither a launch nor a round trip.  The charge and
// the field adjoint that one step adds up are read by the next from another buffer, while the
// third of the three is cleared.  On the 2048-cell, 409,600-particle window a forward step took
// 10.8 + 6.4 us in the run's two kernels (and three copies where it is recorded) and takes 9.6, a
// reverse step 17.8 + 13.3 + 5.7 us in the three kernels of larger grids and takes 10.5.  However
// many particles such a grid holds this is the faster way: a window of 40 steps with a
// checkpoint every 10 takes, in the general sweep and here, 3.5 and 1.0 ms for 1e5 particles in 250
// cells, 13.9 and 2.5 for 1e6, 30 and 4.3 for 2e6, 144 and 15.8 for 8e6; in 4000 cells 3.9 and 1.6 ms for
// 1e5, 6.0 and 2.6 for 1e6, 10.5 and 4.9 for 2e6, 44 and 19.5 for 8e6.
// =======================================================================================
template <int G>
struct AdjTile {
    static constexpr int kThreads = G * kSolveThreads, kPpt = 4, kSlots = kThreads * kPpt;
};

// Inclusive scan and sum of one double per thread over the whole block (16 waves at most); the
// sum in every thread.  s_w holds 16 doubles, used once.
__device__ __forceinline__ double tile_scan(double v, double *s_w, double &total)
{
    const int w = threadIdx.x / kWave, nw = blockDim.x / kWave;
    v = wave_incl_scan(v);
    if (lane_id() == kWave - 1) s_w[w] = v;
    __syncthreads();
    double add = 0.0, tot = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const double t = i < nw ? s_w[i] : 0.0;
        if (i < w) add += t;
        tot += t;
    }
    total = tot;
    return v + add;
}
__device__ __forceinline__ double tile_sum(double v, double *s_w)
{
    const int w = threadIdx.x / kWave, nw = blockDim.x / kWave;
    v = wave_sum_f64(v);
    if (lane_id() == 0) s_w[w] = v;
    __syncthreads();
    double tot = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) tot += i < nw ? s_w[i] : 0.0;
    return tot;
}

// One forward step of the window from charge d.Qi and particles `in` (n slots) to particles `out`
// and charge Qout (cleared before), clearing Qzero.  With `ck` the particles and the charge as
// they came in are also stored there (a checkpoint), with Erec the node field.  The push is
// the FP32 pass's without B, the deposit its fixed point.
template <int G>
__global__ void __launch_bounds__(AdjTile<G>::kThreads) k_adj_fwd(Dev d, AdjState in, AdjState out, AdjState ck,
                                                                  unsigned long long *ckQ, unsigned long long *Qout,
                                                                  unsigned long long *Qzero, double *Erec, int64_t n,
                                                                  int pushes)
{
    constexpr int TH = AdjTile<G>::kThreads, PPT = AdjTile<G>::kPpt;
    __shared__ SmallSolve<G> sh;
    __shared__ float2 s_tab[G * kChunk];
    __shared__ uint32_t s_np;
    // the deposit window takes the solve's node-field array once the gather table is built
    unsigned long long *s_win = (unsigned long long *)&sh.E[0][0];
    const int tid = threadIdx.x;
    const EnsC e = d.ens[0];
    const SegC &S = d.seg[0];
    const int N = (int)e.ncells;
    const int64_t i0 = ((int64_t)blockIdx.x * TH + tid) * PPT;
    int cell[PPT];
    float off[PPT], vx[PPT];
#pragma unroll
    for (int k = 0; k < PPT; ++k) cell[k] = kDead;
    if (i0 + PPT <= n) {
        *(int4 *)cell = *(const int4 *)(in.cell + i0);
        *(float4 *)off = *(const float4 *)(in.off + i0);
        *(float4 *)vx = *(const float4 *)(in.vx + i0);
    } else {
#pragma unroll
        for (int k = 0; k < PPT; ++k)
            if (i0 + k < n) {
                cell[k] = in.cell[i0 + k];
                off[k] = in.off[i0 + k];
                vx[k] = in.vx[i0 + k];
            }
    }
    const float h = (float)S.h, dtdx = (float)S.dtdx, eext = (float)e.E_ext;
    const float tv[3] = {(float)S.t[0], (float)S.t[1], (float)S.t[2]};
    const float sv[3] = {(float)S.s[0], (float)S.s[1], (float)S.s[2]};
    if (tid == 0) s_np = 0u;
    for (int j = blockIdx.x * TH + tid; j < N; j += gridDim.x * TH) {
        if (Qzero) Qzero[j] = 0ull;
        if (ckQ) ckQ[j] = d.Qi[j];
    }
    solve_small<false, G, false>(d, e, 0, 0, sh, s_tab, blockIdx.x == 0 ? Erec : nullptr, [] {});
    if (n == 0) return;  // the field alone
    if (ck.cell && i0 < n) {
#pragma unroll
        for (int k = 0; k < PPT; ++k)
            if (i0 + k < n) {
                ck.cell[i0 + k] = cell[k];
                ck.off[i0 + k] = off[k];
                ck.vx[i0 + k] = vx[k];
            }
    }
    __syncthreads();  // the table is built, the node field no longer read
    for (int j = tid; j < N; j += TH) s_win[j] = 0ull;
    uint32_t np = 0, bad = 0, chg = 0;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const bool alive = cell[k] != kDead;
        np += alive ? 1u : 0u;
        const float2 ec = s_tab[alive ? cell[k] : 0];
        const float Ep = fmaf(off[k], ec.y, ec.x) + eext;
        float vy = 0.f, vz = 0.f;
        boris<float>(h, tv, sv, Ep, vx[k], vy, vz);
        float o = off[k] + vx[k] * dtdx;
        // a non-finite motion or one of more than a period is no valid state (as in the pass)
        const bool fin = fabsf(o) < 1073741824.0f;
        o = fin ? o : 0.0f;
        bad |= (alive && !fin) ? 1u : 0u;
        const float fl = floorf(o);
        int c = ((alive && fin) ? cell[k] : 0) + (int)fl;
        o -= fl;
        const bool up = o >= 1.0f;
        off[k] = up ? o - 1.0f : o;
        c += up ? 1 : 0;
        c = (c < 0) ? c + N : ((c >= N) ? c - N : c);
        const bool inv = alive && (c < 0 || c >= N);
        bad |= inv ? 1u : 0u;
        const int cn = (alive && fin && !inv) ? c : kDead;
        chg |= cn != cell[k] ? 1u : 0u;
        cell[k] = cn;
    }
    if (bad) atomicOr(d.err, (int)E_NONFINITE);
    if (i0 + PPT <= n) {
        if (chg || out.cell != in.cell) *(int4 *)(out.cell + i0) = *(const int4 *)cell;
        *(float4 *)(out.off + i0) = *(const float4 *)off;
        *(float4 *)(out.vx + i0) = *(const float4 *)vx;
    } else {
#pragma unroll
        for (int k = 0; k < PPT; ++k)
            if (i0 + k < n) {
                out.cell[i0 + k] = cell[k];
                out.off[i0 + k] = off[k];
                out.vx[i0 + k] = vx[k];
            }
    }
    __syncthreads();  // the window is cleared
    // a word per cell: count in the high 24 bits, right-node shares in the low 40 (a tile holds
    // at most 4096 particles), runs of equal cell merged per thread
    constexpr int kShift = 40;
    int rk = kDead;
    unsigned long long run = 0;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        if (cell[k] == kDead) continue;
        if (cell[k] != rk) {
            if (rk != kDead) atomicAdd(&s_win[rk], run);
            rk = cell[k];
            run = 0;
        }
        run += (1ull << kShift) | (unsigned long long)fixed_share(off[k]);
    }
    if (rk != kDead) atomicAdd(&s_win[rk], run);
    np = wave_sum_u32(np);
    if (lane_id() == 0 && np) atomicAdd(&s_np, np);
    __syncthreads();
    for (int j = tid; j < N; j += TH) {
        const unsigned long long a = s_win[j], b = s_win[j == 0 ? N - 1 : j - 1];
        constexpr unsigned long long kMask = (1ull << kShift) - 1ull;
        const unsigned long long v = ((a >> kShift) << 24) - (a & kMask) + (b & kMask);
        if (v) atomicAdd(Qout + j, v);
    }
    if (tid == 0 && s_np && pushes)
        atomicAdd(d.cnt + (int64_t)stripe_of_block() * d.nseg * C_NCNT + C_PUSH, (unsigned long long)s_np * pushes);
}

// One step of the reverse sweep.  From the field adjoint lEin of the step above (with `seed`, of
// the objective: eps0 dx E) the block takes the slope g of lQ = (q w / dx) S D lE (see
// k_adj_grid: lQ_{j+1} - lQ_j is -q w (E_{1/2} + (dx/eps0) C_j), the mean and the second sum cancel,
// so one scan and one sum are all it needs), adds it at the positions of the step above (xc1) to lx, then the push and gather adjoint at
// this step's positions (xc, xo) and field E: lv += dt lx, la = dt (q/m) lv,
// lx += la (E_{j+1} - E_j) / dx, and the scatter of la into lEout (cleared before); lEzero is
// cleared.  Dead slots (a run the push flagged non-finite) are skipped.
template <int G>
__global__ void __launch_bounds__(AdjTile<G>::kThreads)
    k_adj_rev(const double *lEin, double *lEout, double *lEzero, int seed, double eps0, double dx, double qw,
              const int32_t *xc1, const int32_t *xc, const float *xo, const double *E, double *lx, double *lv,
              double *lEext, int64_t n, double dt, double qm, int N)
{
    constexpr int TH = AdjTile<G>::kThreads, PPT = AdjTile<G>::kPpt, NPT = kNodesPerThread;
    __shared__ double s_g[G * kChunk], s_dE[G * kChunk], s_acc[G * kChunk];
    __shared__ double s_w[3][16];
    const int tid = threadIdx.x;
    const int64_t i0 = ((int64_t)blockIdx.x * TH + tid) * PPT;
    // the particle loads are in flight during the solve
    int c1[PPT], c0[PPT];
    float o0[PPT];
    double px[PPT], pv[PPT];
    const bool full = i0 + PPT <= n;
    if (full) {
        *(int4 *)c1 = *(const int4 *)(xc1 + i0);
        *(int4 *)c0 = *(const int4 *)(xc + i0);
        *(float4 *)o0 = *(const float4 *)(xo + i0);
#pragma unroll
        for (int k = 0; k < PPT; k += 2) {
            *(double2 *)(px + k) = *(const double2 *)(lx + i0 + k);
            *(double2 *)(pv + k) = *(const double2 *)(lv + i0 + k);
        }
    } else {
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const bool ok = i0 + k < n;
            c1[k] = ok ? xc1[i0 + k] : -1;
            c0[k] = ok ? xc[i0 + k] : -1;
            o0[k] = ok ? xo[i0 + k] : 0.f;
            px[k] = ok ? lx[i0 + k] : 0.0;
            pv[k] = ok ? lv[i0 + k] : 0.0;
        }
    }
    for (int j = blockIdx.x * TH + tid; j < N; j += gridDim.x * TH) lEzero[j] = 0.0;
    const double f = seed ? eps0 * dx : 1.0;
    const int j0 = tid * NPT;
    double r[NPT], sum = 0.0;
    {
        double a[NPT + 2];
#pragma unroll
        for (int q = 0; q < NPT + 2; ++q) {
            int j = j0 + q - 1;
            j = j < 0 ? j + N : (j >= N ? j - N : j);
            a[q] = j0 < N ? f * lEin[j < N ? j : 0] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            r[q] = j0 + q < N ? (a[q + 2] - a[q]) / (2.0 * dx) : 0.0;
            sum += r[q];
        }
    }
    {
        double x[NPT + 1];
#pragma unroll
        for (int q = 0; q < NPT + 1; ++q) x[q] = E[j0 + q < N ? j0 + q : 0];  // (E_N is E_0)
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            if (j0 + q >= N) continue;
            s_dE[j0 + q] = (x[q + 1] - x[q]) / dx;
            s_acc[j0 + q] = 0.0;
        }
    }
    // C_j = sum_{i=1..j} (r_i - mean r): the scan of r gives the mean too
    if (tid == 0) sum -= r[0];
    double tot;
    double R = tile_scan(sum, s_w[0], tot) - sum;
    const double mean_r = (tot + (0.5 * f * (lEin[N > 1 ? 1 : 0] - lEin[N - 1])) / dx) / (double)N;
    double C[NPT], cs = 0.0;
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
        const int j = j0 + q;
        if (j >= 1) R += r[q];
        C[q] = R - (double)j * mean_r;
        if (j < N) cs += C[q];
    }
    const double ce = dx / eps0, Eh = -ce * tile_sum(cs, s_w[1]) / (double)N;
#pragma unroll
    for (int q = 0; q < NPT; ++q)
        if (j0 + q < N) s_g[j0 + q] = -(qw / dx) * (Eh + ce * C[q]);
    __syncthreads();
    double ext = 0.0, r0 = 0.0, r1 = 0.0;
    int rk = -1;
    auto next = [&](int j) { return j + 1 == N ? 0 : j + 1; };
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        if (c1[k] >= 0) px[k] += s_g[c1[k]];
        if (c0[k] < 0) continue;
        const int j = c0[k];
        const double fo = (double)o0[k];
        pv[k] += dt * px[k];
        const double la = dt * qm * pv[k];
        px[k] += la * s_dE[j];
        ext += la;
        if (j != rk) {
            if (rk >= 0) {
                unsafeAtomicAdd(&s_acc[rk], r0);
                unsafeAtomicAdd(&s_acc[next(rk)], r1);
            }
            rk = j;
            r0 = r1 = 0.0;
        }
        r0 += (1.0 - fo) * la;
        r1 += fo * la;
    }
    if (rk >= 0) {
        unsafeAtomicAdd(&s_acc[rk], r0);
        unsafeAtomicAdd(&s_acc[next(rk)], r1);
    }
    if (full) {
#pragma unroll
        for (int k = 0; k < PPT; k += 2) {
            *(double2 *)(lx + i0 + k) = *(const double2 *)(px + k);
            *(double2 *)(lv + i0 + k) = *(const double2 *)(pv + k);
        }
    } else {
#pragma unroll
        for (int k = 0; k < PPT; ++k)
            if (i0 + k < n) {
                lx[i0 + k] = px[k];
                lv[i0 + k] = pv[k];
            }
    }
    ext = tile_sum(ext, s_w[2]);  // (its barriers complete the scatter)
    if (tid == 0) unsafeAtomicAdd(lEext, ext);
    for (int j = tid; j < N; j += TH) {
        const double v = s_acc[j];
        if (v != 0.0) unsafeAtomicAdd(lEout + j, v);
    }
}

hipError_t launch_adj_fwd(const Dev &d, const AdjState &in, const AdjState &out, const AdjState &ck,
                          unsigned long long *ckQ, unsigned long long *Qout, unsigned long long *Qzero, double *Erec,
                          int64_t n, int pushes, hipStream_t s)
{
    auto go = [&](auto k, int slots) {
        const unsigned g = (unsigned)std::max<int64_t>((n + slots - 1) / slots, 1);
        hipLaunchKernelGGL(k, dim3(g), dim3(slots / 4), 0, s, d, in, out, ck, ckQ, Qout, Qzero, Erec, n, pushes);
    };
    if (d.small == 1)
        go(k_adj_fwd<1>, AdjTile<1>::kSlots);
    else if (d.small == 2)
        go(k_adj_fwd<2>, AdjTile<2>::kSlots);
    else
        go(k_adj_fwd<4>, AdjTile<4>::kSlots);
    return hipGetLastError();
}

hipError_t launch_adj_rev(int small, const double *lEin, double *lEout, double *lEzero, bool seed, double eps0,
                          double dx, double qw, const int32_t *xc1, const int32_t *xc, const float *xo, const double *E,
                          double *lx, double *lv, double *lEext, int64_t n, double dt, double qm, int N, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    auto go = [&](auto k, int slots) {
        hipLaunchKernelGGL(k, dim3((unsigned)((n + slots - 1) / slots)), dim3(slots / 4), 0, s, lEin, lEout, lEzero,
                           seed ? 1 : 0, eps0, dx, qw, xc1, xc, xo, E, lx, lv, lEext, n, dt, qm, N);
    };
    if (small == 1)
        go(k_adj_rev<1>, AdjTile<1>::kSlots);
    else if (small == 2)
        go(k_adj_rev<2>, AdjTile<2>::kSlots);
    else
        go(k_adj_rev<4>, AdjTile<4>::kSlots);
    return hipGetLastError();
}

// =======================================================================================
// Windows on larger grids: the forward steps of the run and three kernels per reverse step.
// =======================================================================================

// Per particle, first half of the step adjoint: pass-through of lx into lv, the gather
// adjoint (a scatter into lE) and the interpolation derivative.
template <int PPT>
__global__ void __launch_bounds__(256) k_adj_a(Dev d, const int32_t *xc, const float *xo,
                                                  const double *E, double *lx, double *lv,
                                                  double *lE, double *lEext, int64_t n, double dt,
                                                  double qm, double dx, int N)
{
    __shared__ double s_red[4];
    const int64_t i0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * PPT;
    double ext = 0.0;
    int rk = -1;
    double r0 = 0.0, r1 = 0.0;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int64_t i = i0 + k;
        if (i >= n) break;
        // a slot the push dropped as non-finite (the call reports it) holds no cell and adds nothing
        const int c = xc[i], j = max(c, 0);
        const double f = (double)xo[i];
        const int j1 = (j + 1 == N) ? 0 : j + 1;
        const double lvn = lv[i] + dt * lx[i];
        const double la = c < 0 ? 0.0 : dt * qm * lvn;
        lv[i] = lvn;
        lx[i] += la * (E[j1] - E[j]) / dx;
        ext += la;
        if (j != rk) {
            if (rk >= 0) {
                unsafeAtomicAdd(lE + rk, r0);
                unsafeAtomicAdd(lE + ((rk + 1 == N) ? 0 : rk + 1), r1);
            }
            rk = j;
            r0 = r1 = 0.0;
        }
        r0 += (1.0 - f) * la;
        r1 += f * la;
    }
    if (rk >= 0) {
        unsafeAtomicAdd(lE + rk, r0);
        unsafeAtomicAdd(lE + ((rk + 1 == N) ? 0 : rk + 1), r1);
    }
    ext = wave_sum_f64(ext);
    if (lane_id() == 0) s_red[threadIdx.x / kWave] = ext;
    __syncthreads();
    if (threadIdx.x == 0) unsafeAtomicAdd(lEext, s_red[0] + s_red[1] + s_red[2] + s_red[3]);
}

// Second half: the deposit adjoint (a gather of lQ's difference).
template <int PPT>
__global__ void __launch_bounds__(256) k_adj_b(const int32_t *xc, const double *lQ, double *lx,
                                                  int64_t n, double dx, int N)
{
    const int64_t i0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * PPT;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int64_t i = i0 + k;
        if (i >= n) break;
        const int j = max(xc[i], 0);  // (a dropped slot's lx is not used)
        const int j1 = (j + 1 == N) ? 0 : j + 1;
        lx[i] += (lQ[j1] - lQ[j]) / dx;
    }
}

// Block-wide inclusive scan of a double per thread (1024 threads).
__device__ double adj_block_scan(double v, double *s_w)
{
    const int lane = lane_id(), w = threadIdx.x / kWave, nw = blockDim.x / kWave;
    v = wave_incl_scan(v);
    if (lane == kWave - 1) s_w[w] = v;
    __syncthreads();
    double add = 0.0;
    for (int i = 0; i < w; ++i) add += s_w[i];
    double tot = 0.0;
    for (int i = 0; i < nw; ++i) tot += s_w[i];
    __syncthreads();
    s_w[16] = tot;  // read by the caller after the next barrier
    return v + add;
}

// Grid adjoint (one block): lphi = D lE; lrho = S lphi; lQ = (q w / dx) lrho; lE = 0.
// S is the zero-mean periodic solve of (phi_{j-1} - 2 phi_j + phi_{j+1}) / dx^2 = -r_j / eps0,
// computed as in the forward solve by two prefix sums with phi_0 = phi_N = 0, then the mean
// removed.  `tmp` holds N doubles of scratch.
__global__ void __launch_bounds__(1024) k_adj_grid(double *lE, double *lQ, double *tmp, int N,
                                                   double dx, double eps0, double qw)
{
    __shared__ double s_w[17];
    __shared__ double s_carry, s_tot;
    const int T = blockDim.x;
    // r = D lE (zero-sum by construction)
    for (int j = threadIdx.x; j < N; j += T) {
        const int jp = (j + 1 == N) ? 0 : j + 1, jm = (j == 0) ? N - 1 : j - 1;
        tmp[j] = (lE[jp] - lE[jm]) / (2.0 * dx);
    }
    __syncthreads();
    for (int j = threadIdx.x; j < N; j += T) lE[j] = 0.0;
    // the source used by the solve: r_j on the interior nodes 1..N-1; remove the mean of r
    // (zero up to rounding) as the forward background does
    double loc = 0.0;
    for (int j = threadIdx.x; j < N; j += T) loc += tmp[j];
    loc = wave_sum_f64(loc);
    if (lane_id() == 0) s_w[threadIdx.x / kWave] = loc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int i = 0; i < T / kWave; ++i) t += s_w[i];
        s_tot = t / N;
    }
    __syncthreads();
    const double mean_r = s_tot;
    const double ce = dx / eps0;
    // pass 1: C_m = sum_{i=1..m} r_i stored in lQ (as scratch), S = sum_{m<N} C_m
    if (threadIdx.x == 0) s_carry = 0.0;
    __syncthreads();
    double Ssum = 0.0;
    for (int base = 0; base < N; base += T) {
        const int j = base + threadIdx.x;
        const double r = (j >= 1 && j < N) ? tmp[j] - mean_r : 0.0;
        const double inc = adj_block_scan(r, s_w);
        __syncthreads();
        const double tot = s_w[16];
        const double C = s_carry + inc;
        if (j < N) lQ[j] = C;
        Ssum += (j < N) ? C : 0.0;
        __syncthreads();
        if (threadIdx.x == 0) s_carry += tot;
        __syncthreads();
    }
    Ssum = wave_sum_f64(Ssum);
    if (lane_id() == 0) s_w[threadIdx.x / kWave] = Ssum;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int i = 0; i < T / kWave; ++i) t += s_w[i];
        s_tot = t;
        s_carry = 0.0;
    }
    __syncthreads();
    const double Eh = -ce * s_tot / (double)N;
    // pass 2: phi_j = -dx (j Eh + ce F_j), F_j = sum_{m<j} C_m; accumulate the mean
    double phisum = 0.0;
    for (int base = 0; base < N; base += T) {
        const int j = base + threadIdx.x;
        const double C = (j < N) ? lQ[j] : 0.0;
        const double inc = adj_block_scan(C, s_w);
        __syncthreads();
        const double tot = s_w[16];
        const double F = s_carry + inc - C;
        if (j < N) {
            const double phi = -dx * ((double)j * Eh + ce * F);
            tmp[j] = phi;
            phisum += phi;
        }
        __syncthreads();
        if (threadIdx.x == 0) s_carry += tot;
        __syncthreads();
    }
    phisum = wave_sum_f64(phisum);
    if (lane_id() == 0) s_w[threadIdx.x / kWave] = phisum;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int i = 0; i < T / kWave; ++i) t += s_w[i];
        s_tot = t / N;
    }
    __syncthreads();
    const double mphi = s_tot;
    for (int j = threadIdx.x; j < N; j += T) lQ[j] = (qw / dx) * (tmp[j] - mphi);
}

// Seed of the reverse sweep: lE = d W / d E = eps0 dx E.
__global__ void k_adj_seed(const double *E, double *lE, int N, double eps0, double dx)
{
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < N; j += gridDim.x * blockDim.x)
        lE[j] = eps0 * dx * E[j];
}

// Gradient by particle id: out[id_i] = lv_i for the n slots (ids at or above `len` set the
// error flag instead).
__global__ void k_adj_by_id(const double *lv, const uint32_t *id, double *out, int64_t n, int64_t len,
                            int32_t *err)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t k = id[i];
        if ((int64_t)k < len)
            out[k] = lv[i];
        else
            atomicOr(err, 1);
    }
}

// The same, counting the distinct ids in *distinct through a bit per id (cleared before).
__global__ void __launch_bounds__(256) k_adj_by_id_count(const double *lv, const uint32_t *id, double *out,
                                                         uint32_t *seen, int64_t n, int64_t len, int32_t *err,
                                                         uint32_t *distinct)
{
    __shared__ uint32_t s_n;
    if (threadIdx.x == 0) s_n = 0u;
    __syncthreads();
    uint32_t mine = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t k = id[i];
        if ((int64_t)k < len) {
            out[k] = lv[i];
            const uint32_t bit = 1u << (k & 31);
            mine += (atomicOr(seen + (k >> 5), bit) & bit) ? 0u : 1u;
        } else {
            atomicOr(err, 1);
        }
    }
    mine = wave_sum_u32(mine);
    if (lane_id() == 0 && mine) atomicAdd(&s_n, mine);
    __syncthreads();
    if (threadIdx.x == 0 && s_n) atomicAdd(distinct, s_n);
}

hipError_t launch_adj_by_id_count(const double *lv, const uint32_t *id, double *out, uint32_t *seen, int64_t n,
                                  int64_t len, int32_t *err, uint32_t *distinct, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int64_t G = std::min<int64_t>((n + 255) / 256, 2048);
    hipLaunchKernelGGL(k_adj_by_id_count, dim3((unsigned)G), dim3(256), 0, s, lv, id, out, seen, n, len, err, distinct);
    return hipGetLastError();
}

hipError_t launch_adj_by_id(const double *lv, const uint32_t *id, double *out, int64_t n, int64_t len,
                            int32_t *err, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int64_t G = std::min<int64_t>((n + 255) / 256, 2048);
    hipLaunchKernelGGL(k_adj_by_id, dim3((unsigned)G), dim3(256), 0, s, lv, id, out, n, len, err);
    return hipGetLastError();
}

hipError_t launch_adj_seed(const double *E, double *lE, int N, double eps0, double dx, hipStream_t s)
{
    hipLaunchKernelGGL(k_adj_seed, dim3(8), dim3(256), 0, s, E, lE, N, eps0, dx);
    return hipGetLastError();
}

hipError_t launch_adj_a(const Dev &d, const int32_t *xc, const float *xo, const double *E, double *lx,
                        double *lv, double *lE, double *lEext, int64_t n, double dt, double qm,
                        double dx, int N, hipStream_t s)
{
    const int64_t G = (n + 256 * 8 - 1) / (256 * 8);
    if (G == 0) return hipSuccess;
    hipLaunchKernelGGL(k_adj_a<8>, dim3(G), dim3(256), 0, s, d, xc, xo, E, lx, lv, lE, lEext, n, dt, qm, dx, N);
    return hipGetLastError();
}

hipError_t launch_adj_grid(double *lE, double *lQ, double *tmp, int N, double dx, double eps0, double qw,
                           hipStream_t s)
{
    hipLaunchKernelGGL(k_adj_grid, dim3(1), dim3(1024), 0, s, lE, lQ, tmp, N, dx, eps0, qw);
    return hipGetLastError();
}

hipError_t launch_adj_b(const int32_t *xc, const double *lQ, double *lx, int64_t n, double dx, int N,
                        hipStream_t s)
{
    const int64_t G = (n + 256 * 8 - 1) / (256 * 8);
    if (G == 0) return hipSuccess;
    hipLaunchKernelGGL(k_adj_b<8>, dim3(G), dim3(256), 0, s, xc, lQ, lx, n, dx, N);
    return hipGetLastError();
}

}  // namespace pic
