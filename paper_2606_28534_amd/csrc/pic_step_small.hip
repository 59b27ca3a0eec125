// pic_step_small.hip -- one launch per step for small periodic runs without collisions.
//
// Between two steps that sort such a run (a Langmuir oscillation, a two-stream instability) is a
// chain of two dependent launches, the one-block solve and the particle pass, each of a few
// microseconds of latency and next to no work.  Nothing but the charge couples one step's particles to
// the next, so here every block solves its ensemble's field for itself in LDS, a chunk per group
// of kSolveThreads threads, and then takes its own particles: the solve costs neither a launch nor
// a round trip through the gather table.  The charge alternates between three buffers: a step
// reads one, adds up the next and clears the third.
//
// What bounds it is the solve's chain of block-wide scans, about 7 us, and beyond some 1e6
// particles that every one of the many blocks walks it.  20 steps (18 of them here) took, in two
// launches a step and in one: 2048 cells with 4e5 particles 332 and 245 us; 250, 2048 and 4000
// cells with 1e6 particles 360 and 333, 405 and 358, 517 and 406; with 2e6 485 and 519, 505 and 575,
// 621 and 694.  The line lies at 2^20 slots of capacity (kStepSlots).
#include "pic_device.h"
#include "pic_kernels.h"
#include "pic_particle.h"
#include "pic_solve.h"

namespace pic {

// One step of the particles of the block's tile from charge d.Qi, their charge added to Qout
// (cleared before); Qzero is cleared.  Push, deposit and tallies are the FP32 pass's, so
// the state is the same to the last bit; rho, phi and the field are left as they were (the
// last step of a window is always one of the two launches that write them).
template <int G>
__global__ void __launch_bounds__(G *kSolveThreads) k_step_small(Dev d, unsigned long long *Qout,
                                                                 unsigned long long *Qzero)
{
    constexpr int TH = G * kSolveThreads, PPT = 4;
    __shared__ SmallSolve<G> sh;
    __shared__ float2 s_tab[G * kChunk];
    __shared__ uint32_t s_np;
    // the deposit window takes the solve's node-field array once the gather table is built
    unsigned long long *s_win = (unsigned long long *)&sh.E[0][0];
    const int tid = threadIdx.x;
    for (int64_t j = (int64_t)blockIdx.x * TH + tid; j < d.nspecies * d.nodes_tot; j += (int64_t)gridDim.x * TH)
        Qzero[j] = 0ull;
    if (blockIdx.x == 0 && tid == 0) *d.step += 1;
    const int64_t first = (int64_t)blockIdx.x * TH * PPT;
    const int sg = seg_of_slot(d, first);
    const SegC &S = d.seg[sg];
    const int64_t last = min(first + TH * PPT, S.base + d.n_slots[sg]);
    if (first >= last) return;
    const EnsC e = d.ens[S.ens];
    const int b = *d.cur, N = S.ncells;
    const int64_t i0 = first + (int64_t)tid * PPT;
    const bool full = i0 + PPT <= last;
    int cell[PPT];
    float off[PPT], vx[PPT], vy[PPT], vz[PPT];
#pragma unroll
    for (int k = 0; k < PPT; ++k) cell[k] = kDead;
    if (full) {
        *(int4 *)cell = *(const int4 *)(d.cell[b] + i0);
        *(float4 *)off = *(const float4 *)(d.off[b] + i0);
        *(float4 *)vx = *(const float4 *)(d.fvx[b] + i0);
    } else {
#pragma unroll
        for (int k = 0; k < PPT; ++k)
            if (i0 + k < last) {
                cell[k] = d.cell[b][i0 + k];
                off[k] = d.off[b][i0 + k];
                vx[k] = d.fvx[b][i0 + k];
            }
    }
    auto load_perp = [&] {
        if (full) {
            *(float4 *)vy = *(const float4 *)(d.fvy[b] + i0);
            *(float4 *)vz = *(const float4 *)(d.fvz[b] + i0);
        } else {
#pragma unroll
            for (int k = 0; k < PPT; ++k)
                if (i0 + k < last) {
                    vy[k] = d.fvy[b][i0 + k];
                    vz[k] = d.fvz[b][i0 + k];
                }
        }
    };
    // (1024 threads have 128 registers each, too few to hold these through the solve)
    if constexpr (G < 4) load_perp();
    const float h = (float)S.h, dtdx = (float)S.dtdx, eext = (float)e.E_ext;
    const float tv[3] = {(float)S.t[0], (float)S.t[1], (float)S.t[2]};
    const float sv[3] = {(float)S.s[0], (float)S.s[1], (float)S.s[2]};
    const int64_t qbase = (int64_t)S.species * d.nodes_tot + S.gbase;
    if (tid == 0) s_np = 0u;
    solve_small<false, G, false>(d, e, S.ens, 0, sh, s_tab, nullptr, [] {});
    if constexpr (G == 4) load_perp();
    __syncthreads();  // the table is built, the node field no longer read
    for (int j = tid; j < N; j += TH) s_win[j] = 0ull;
    uint32_t np = 0, bad = 0, chg = 0;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const bool alive = cell[k] != kDead;
        np += alive ? 1u : 0u;
        const float2 ec = s_tab[alive ? cell[k] : 0];
        const float Ep = fmaf(off[k], ec.y, ec.x) + eext;
        boris<float>(h, tv, sv, Ep, vx[k], vy[k], vz[k]);
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
    if (full) {
        if (chg) *(int4 *)(d.cell[b] + i0) = *(const int4 *)cell;
        *(float4 *)(d.off[b] + i0) = *(const float4 *)off;
        *(float4 *)(d.fvx[b] + i0) = *(const float4 *)vx;
        *(float4 *)(d.fvy[b] + i0) = *(const float4 *)vy;
        *(float4 *)(d.fvz[b] + i0) = *(const float4 *)vz;
    } else {
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            if (i0 + k >= last) continue;
            d.cell[b][i0 + k] = cell[k];
            d.off[b][i0 + k] = off[k];
            if (cell[k] == kDead) continue;
            d.fvx[b][i0 + k] = vx[k];
            d.fvy[b][i0 + k] = vy[k];
            d.fvz[b][i0 + k] = vz[k];
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
        const unsigned long long a = s_win[j], am = s_win[j == 0 ? N - 1 : j - 1];
        constexpr unsigned long long kMask = (1ull << kShift) - 1ull;
        const unsigned long long v = ((a >> kShift) << 24) - (a & kMask) + (am & kMask);
        if (v) atomicAdd(Qout + qbase + j, v);
    }
    if (tid == 0 && s_np)
        atomicAdd(d.cnt + ((int64_t)stripe_of_block() * d.nseg + sg) * C_NCNT + C_PUSH, (unsigned long long)s_np);
}

// (Dev::Qx is there for the small periodic FP32 runs of at most kStepSlots slots)
bool step_in_one_launch(const Dev &d)
{
    return d.Qx && d.periodic && !d.collisions && d.ncap_tot == 0 && d.src_tot == 0;
}

hipError_t launch_step_small(const Dev &d, unsigned long long *Qout, unsigned long long *Qzero, hipStream_t s)
{
    static_assert(kSlotAlign % (4 * kSmallChunks * kSolveThreads) == 0, "whole tiles per segment");
    const int th = d.small * kSolveThreads;
    const dim3 g((unsigned)(d.cap_tot / (4 * th)));
    if (d.small == 1)
        hipLaunchKernelGGL(k_step_small<1>, g, dim3(th), 0, s, d, Qout, Qzero);
    else if (d.small == 2)
        hipLaunchKernelGGL(k_step_small<2>, g, dim3(th), 0, s, d, Qout, Qzero);
    else
        hipLaunchKernelGGL(k_step_small<4>, g, dim3(th), 0, s, d, Qout, Qzero);
    return hipGetLastError();
}

}  // namespace pic
