// pic_pass64.hip -- the FP64 (plain x, v) particle pass for gfx950.
//
// One template covers every particle stage: gather + Boris push + walls, null-collision MC,
// cloud-in-cell deposit and the sort histogram are compile-time stage bits, so the separate
// stage verbs and the fused step run the same per-particle code.
//
// One block takes one tile of consecutive slots of one segment, as in the FP32 pass: the grid covers the slot capacity, blocks beyond the slots in use return at
// once, and the dispatcher hands tiles to whichever CUs are free, so uneven segments and slow
// tiles balance themselves.  (Persistent blocks that took tiles from per-XCD queues cost 20 to
// 25 us a stage however few particles there were, and walked their tiles one latency after
// another: push, collide and deposit of 8e6 particles took 138, 134 and 167 us, now 80, 78 and
// 33 us, the push at 6.4 TB/s of the 64 B it moves; 256 cells with 5e4 particles took 20, 26
// and 26 us, now 6, 12 and 7.)
//
// A thread owns two runs of two consecutive slots, each moved as one 16-byte vector per array
// (a wave touches 1 KB of consecutive bytes per load).  What bounds each stage: the push HBM
// (64 B a particle); the collide stage its loads (36 B) and the Philox draw, since the ~1%
// that pass the null-collision test are listed in LDS and collided afterwards by the first
// lanes of the block, all at once, instead of one divergent lane at a time; the deposit its
// LDS atomics, so equal cells are merged per thread and the window holds copies of its nodes.
#include <algorithm>

#include "pic_device.h"
#include "pic_kernels.h"
#include "pic_particle.h"
#include "pic_rules.h"

namespace pic {

enum Stage : int { ST_PUSH = 1, ST_COLLIDE = 2, ST_DEPOSIT = 4, ST_HIST = 8 };

constexpr int kPpt64 = 4;     // slots per thread
constexpr int kRun64 = 2;     // of them consecutive: one 16-byte vector of doubles
constexpr int kWin64 = 1024;  // LDS window: nodes x copies

// A run of consecutive slots of one array; `in` slots of it are in range (whole runs as one
// vector: the run's first slot is even and the arrays are 256-byte aligned).
typedef double vec2d __attribute__((ext_vector_type(2)));
typedef uint32_t vec2u __attribute__((ext_vector_type(2)));
template <bool NT>
__device__ __forceinline__ void run_load(const double *p, int in, double fill, double (&v)[kRun64])
{
    if (in == kRun64) {
        const vec2d t = NT ? __builtin_nontemporal_load((const vec2d *)p) : *(const vec2d *)p;
        v[0] = t.x;
        v[1] = t.y;
    } else {
        v[0] = in > 0 ? p[0] : fill;
        v[1] = fill;
    }
}

template <bool NT>
__device__ __forceinline__ void run_store(double *p, double a, double b)
{
    const vec2d v = {a, b};
    if constexpr (NT)
        __builtin_nontemporal_store(v, (vec2d *)p);
    else
        *(vec2d *)p = v;
}

// Adds a run of equal cell (its left and right shares and its count) to the tile's LDS window
// when both nodes lie in it, else straight to HBM.
struct Window64 {
    double *w;
    uint32_t *c;
    int base, n, ls, copy;
};
template <bool DEPO>
__device__ __forceinline__ void emit64(const Dev &d, const Seg64 &G, int s, const Window64 &W, int cell, double l,
                                       double r, uint32_t cnt, bool hist)
{
    const int rel = cell - W.base;
    const bool in = rel + 1 < W.n;  // (rel >= 0: base is the tile's lowest cell)
    const int i = (rel << W.ls) + W.copy;
    if constexpr (DEPO) {
        if (in) {
            unsafeAtomicAdd(W.w + i, l);
            unsafeAtomicAdd(W.w + i + (1 << W.ls), r);
        } else {
            const int j1 = (G.periodic && cell + 1 == G.ncells) ? 0 : cell + 1;
            double *Q = d.Qd + (int64_t)s * d.nodes_tot + G.gbase;
            unsafeAtomicAdd(Q + cell, l);
            unsafeAtomicAdd(Q + j1, r);
        }
    }
    if (hist) {
        if (in)
            atomicAdd(W.c + i, cnt);
        else
            atomicAdd(d.cellcnt + G.cbase + cell, cnt);
    }
}

// Collide one candidate (its post-push state is in memory): scatter, tally, append a birth.
template <bool DEPO>
__device__ __forceinline__ double collide64(const Dev &d, const SegC &S, const EnsC &e, int b, int64_t i,
                                            double numax, double pnull, uint32_t tag, int half, int st, bool pairs,
                                            bool hist, uint32_t *s_c)
{
    PS<true> p;
    p.x = d.x[b][i];
    p.vx = d.dvx[b][i];
    p.vy = d.dvy[b][i];
    p.vz = d.dvz[b][i];
    p.id = d.id[b][i];
    double ve[3], vi[3];
    const int ch = p_collide<true>(e, S, S.species, numax, pnull, tag, p, ve, vi);
    double v2m = speed2_rn(p.vx, p.vy, p.vz);
    if (ch < 0) return v2m;
    d.dvx[b][i] = p.vx;
    d.dvy[b][i] = p.vy;
    d.dvz[b][i] = p.vz;
    atomicAdd(&s_c[ch == 0 ? C_EL : ch == 1 ? C_IZ : C_CX], 1u);
    if (ch != 1) return v2m;
    // birth record: slot in this block's stripe, or in the next ones when it is full
    const BirthBuf bb = birth_buf(d, (int)(tag & 1u));
    int bst = st & (kStripes - 1);
    uint32_t slot = atomicAdd(bb.nbirth + bst, 1u);
    for (int a = 1; a < kStripes && (int64_t)slot >= d.birth_stripe_cap; ++a) {
        bst = (bst + 1) & (kStripes - 1);
        slot = atomicAdd(bb.nbirth + bst, 1u);
    }
    if ((int64_t)slot < d.birth_stripe_cap) {
        Birth &B = bb.births[(int64_t)bst * d.birth_stripe_cap + slot];
        B.pid = p.id;
        B.ens = S.ens;
        B.cell = 0;
        B.off = 0.f;
        B.x = p.x;
        for (int q = 0; q < 3; ++q) {
            B.ve[q] = ve[q];
            B.vi[q] = vi[q];
        }
        birth_mark(bb, e, p.id);
    } else {
        atomicOr(d.err, (int)E_CAP_BIRTH);
    }
    if (S.other >= 0)
        atomicMax(d.vmax2 + ((int64_t)half * kCntStripes + st) * d.nseg + S.other, dbits(speed2_rn(vi[0], vi[1], vi[2])));
    if (DEPO || pairs) {
        // the new pair sits at the parent's position
        global_deposit64(d, S, S.species, p.x, hist);
        if (S.other >= 0) global_deposit64(d, d.seg[S.other], 1, p.x, hist);
    }
    return fmax(v2m, speed2_rn(ve[0], ve[1], ve[2]));
}

// hist_rt: count cells in the deposit's window; a collide stage without deposit adds its new
// pairs' charge all the same.
constexpr int kHist64 = 1, kPairs = 2;
template <int STAGES, bool NT>
__device__ __forceinline__ void particles_body(const Dev &d, int hist_rt, int64_t first, int64_t last, int sg, int b)
{
    constexpr bool PUSH = STAGES & ST_PUSH;
    constexpr bool COLL = STAGES & ST_COLLIDE;
    constexpr bool DEPO = STAGES & ST_DEPOSIT;
    constexpr bool HISTC = STAGES & ST_HIST;  // histogram-only pass
    constexpr bool WIN = DEPO || HISTC;
    constexpr bool NEED_V = PUSH || COLL;
    constexpr int G2 = kPpt64 / kRun64;

    __shared__ double s_win[DEPO ? kWin64 : 1];
    __shared__ uint32_t s_cell[WIN ? kWin64 : 1];  // the window's counts, for the sort
    __shared__ uint32_t s_list[COLL ? 256 * kPpt64 : 1];  // candidates: slots within the tile
    __shared__ uint32_t s_nc, s_c[C_NCNT];
    __shared__ double s_ke[2];
    __shared__ unsigned long long s_v2;
    __shared__ int s_mn[4], s_mx[4];

    const int tid = threadIdx.x, BLOCK = blockDim.x, lane = lane_id(), w = tid / kWave, nw = BLOCK / kWave;
    const SegC &S = d.seg[sg];
    const EnsC &e = d.ens[S.ens];
    const Seg64 G = seg64(S, e);  // gather, push and deposit constants in registers
    const int s = S.species;
    const bool hist = HISTC || (hist_rt & kHist64) != 0;
    const int st = stripe_of_block();

    // every load of the tile is issued before any is used
    PS<true> p[kPpt64];
#pragma unroll
    for (int g = 0; g < G2; ++g) {
        const int64_t i = first + ((int64_t)g * BLOCK + tid) * kRun64;
        const int in = (int)min((int64_t)kRun64, max((int64_t)0, last - i));
        double x[kRun64], v[3][kRun64];
        uint32_t id[kRun64] = {0u, 0u};
        run_load<NT>(d.x[b] + i, in, -1.0, x);
        if (NEED_V) {
            run_load<NT>(d.dvx[b] + i, in, 0.0, v[0]);
            run_load<NT>(d.dvy[b] + i, in, 0.0, v[1]);
            run_load<NT>(d.dvz[b] + i, in, 0.0, v[2]);
        }
        if (COLL) {
            if (in == kRun64) {
                const vec2u *ip = (const vec2u *)(d.id[b] + i);
                const vec2u u = NT ? __builtin_nontemporal_load(ip) : *ip;
                id[0] = u.x;
                id[1] = u.y;
            } else if (in > 0) {
                id[0] = d.id[b][i];
            }
        }
#pragma unroll
        for (int k = 0; k < kRun64; ++k) {
            PS<true> &q = p[g * kRun64 + k];
            q.x = x[k];
            if (NEED_V) {
                q.vx = v[0][k];
                q.vy = v[1][k];
                q.vz = v[2][k];
            }
            q.id = id[k];
        }
    }
    bool live[kPpt64];
#pragma unroll
    for (int k = 0; k < kPpt64; ++k) live[k] = p_alive<true>(p[k]);
    if (tid < C_NCNT) s_c[tid] = 0u;
    if (tid < 2) s_ke[tid] = 0.0;
    if (tid == 0) {
        s_nc = 0u;
        s_v2 = 0ull;
    }
    if constexpr (PUSH) {
        __syncthreads();  // the tallies are cleared
        double Eg[kPpt64];
        gather64<kPpt64>(d, G, p, Eg);
        uint32_t np = 0;
#pragma unroll
        for (int k = 0; k < kPpt64; ++k) np += (uint32_t)__popcll(__ballot(live[k]));
#pragma unroll
        for (int g = 0; g < G2; ++g) {
            const int64_t i = first + ((int64_t)g * BLOCK + tid) * kRun64;
            bool died = false;
#pragma unroll
            for (int k = g * kRun64; k < (g + 1) * kRun64; ++k) {
                if (!live[k]) continue;
                const int wall = p_push64(d, G, p[k], Eg[k]);
                if (wall == 0) continue;
                died = true;
                if (wall != 3) {
                    const double ke = S.halfmw * speed2_rn(p[k].vx, p[k].vy, p[k].vz);
                    atomicAdd(&s_c[wall == 1 ? C_WALL_L : C_WALL_R], 1u);
                    unsafeAtomicAdd(&s_ke[wall - 1], ke);
                }
                p_kill<true>(p[k]);
            }
            // a run that lost a particle in this push keeps that slot's velocity, as a run at
            // the end of the slots in use keeps what lies beyond them
            if (!died && i + kRun64 <= last) {
                const int k = g * kRun64;
                run_store<NT>(d.x[b] + i, p[k].x, p[k + 1].x);
                run_store<NT>(d.dvx[b] + i, p[k].vx, p[k + 1].vx);
                run_store<NT>(d.dvy[b] + i, p[k].vy, p[k + 1].vy);
                run_store<NT>(d.dvz[b] + i, p[k].vz, p[k + 1].vz);
            } else {
#pragma unroll
                for (int u = 0; u < kRun64; ++u) {
                    const int k = g * kRun64 + u;
                    if (!live[k]) continue;
                    d.x[b][i + u] = p[k].x;
                    if (!p_alive<true>(p[k])) continue;
                    d.dvx[b][i + u] = p[k].vx;
                    d.dvy[b][i + u] = p[k].vy;
                    d.dvz[b][i + u] = p[k].vz;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < kPpt64; ++k) live[k] = p_alive<true>(p[k]);
        if (lane == 0 && np) atomicAdd(&s_c[C_PUSH], np);
    }
    double v2m = 0.0;
    if constexpr (COLL) {
        if constexpr (!PUSH) __syncthreads();  // the tallies are cleared
        // Reading R12 decision R1 < P_null, taken exactly as the integer test
        // (r >> 9) < ceil(P_null 2^23 - 1/2) on the first Philox word of block 0.
        const double X = d.pnull[sg] * 8388608.0 - 0.5;
        const uint32_t thr = X <= 0.0 ? 0u : (X >= 8388608.0 ? 8388608u : (uint32_t)ceil(X));
        const uint32_t tag = (uint32_t)(*d.step);
#pragma unroll
        for (int k = 0; k < kPpt64; ++k) {
            if (!live[k]) continue;
            if ((philox(p[k].id, tag, 0u, 0u, S.seed, (uint32_t)s).x >> 9) < thr)
                s_list[atomicAdd(&s_nc, 1u)] = (uint32_t)(((k / kRun64) * BLOCK + tid) * kRun64 + k % kRun64);
            else
                v2m = fmax(v2m, speed2_rn(p[k].vx, p[k].vy, p[k].vz));
        }
    }
    Window64 W{s_win, s_cell, 0, 0, 0, 0};
    int key[kPpt64];
    double f[kPpt64];
    if constexpr (WIN) {
        int mn = INT32_MAX, mx = -1;
#pragma unroll
        for (int k = 0; k < kPpt64; ++k) {
            f[k] = 0.0;
            key[k] = live[k] ? (int)cell_of_x64(G, p[k].x, f[k]) : -1;
            if (live[k]) {
                mn = min(mn, key[k]);
                mx = max(mx, key[k]);
            }
        }
        mn = wave_min_i32(mn);
        mx = wave_max_i32(mx);
        if (lane == 0) {
            s_mn[w] = mn;
            s_mx[w] = mx;
        }
    }
    __syncthreads();  // the push's stores and the candidate list are in place
    if constexpr (WIN) {
        int mn = s_mn[0], mx = s_mx[0];
        for (int i = 1; i < nw; ++i) {
            mn = min(mn, s_mn[i]);
            mx = max(mx, s_mx[i]);
        }
        // nodes mn .. mx + 1, at most kWin64 from the lowest; as many copies of each as fit (a
        // power of two, up to one per lane)
        W.base = mn;
        W.n = mx >= 0 ? min(mx - mn + 2, kWin64) : 0;
        W.ls = W.n ? min(31 - __clz(kWin64 / W.n), 6) : 0;
        W.copy = lane & ((1 << W.ls) - 1);
        for (int i = tid; i < W.n << W.ls; i += BLOCK) {
            if constexpr (DEPO) s_win[i] = 0.0;
            if (hist) s_cell[i] = 0u;
        }
        __syncthreads();
    }
    if constexpr (COLL) {
        const uint32_t nc = s_nc, tag = (uint32_t)(*d.step);
        const int half = 1 - *d.vcur;
        if ((uint32_t)tid < nc) {
            const double numax = d.numax[sg], pnull = d.pnull[sg];
            for (uint32_t q = tid; q < nc; q += BLOCK)
                v2m = fmax(v2m, collide64<DEPO>(d, S, e, b, first + s_list[q], numax, pnull, tag, half, st,
                                                (hist_rt & kPairs) != 0, hist, s_c));
        }
        v2m = wave_max_f64(v2m);
        if (lane == 0 && v2m > 0.0) atomicMax(&s_v2, dbits(v2m));
    }
    if constexpr (WIN) {
#pragma unroll
        for (int g = 0; g < G2; ++g) {
            const int a = g * kRun64, c = a + 1;
            if (key[a] >= 0 && key[a] == key[c]) {
                emit64<DEPO>(d, G, s, W, key[a], (1.0 - f[a]) + (1.0 - f[c]), f[a] + f[c], 2u, hist);
            } else {
                if (key[a] >= 0) emit64<DEPO>(d, G, s, W, key[a], 1.0 - f[a], f[a], 1u, hist);
                if (key[c] >= 0) emit64<DEPO>(d, G, s, W, key[c], 1.0 - f[c], f[c], 1u, hist);
            }
        }
        __syncthreads();
        // each node's copies are summed from the thread's own offset, so that the lanes of a
        // wave read different banks
        const int copies = 1 << W.ls;
        double *Q = d.Qd + (int64_t)s * d.nodes_tot + G.gbase;
        for (int n = tid; n < W.n; n += BLOCK) {
            if constexpr (DEPO) {
                double a = 0.0;
                for (int r = 0; r < copies; ++r) a += s_win[(n << W.ls) + ((r + lane) & (copies - 1))];
                int node = W.base + n;
                if (G.periodic && node >= G.ncells) node -= G.ncells;
                if (a != 0.0) unsafeAtomicAdd(Q + node, a);
            }
            if (hist) {
                uint32_t c = 0;
                for (int r = 0; r < copies; ++r) c += s_cell[(n << W.ls) + ((r + lane) & (copies - 1))];
                if (c) atomicAdd(d.cellcnt + G.cbase + W.base + n, c);
            }
        }
    } else {
        __syncthreads();
    }
    if ((PUSH || COLL) && tid < C_NCNT) {
        if (s_c[tid]) atomicAdd(d.cnt + ((int64_t)st * d.nseg + sg) * C_NCNT + tid, (unsigned long long)s_c[tid]);
        if (PUSH && tid < 2 && s_ke[tid] != 0.0)
            unsafeAtomicAdd(d.sums + ((int64_t)st * d.nseg + sg) * S_NSUM + (tid == 0 ? S_KE_L : S_KE_R), s_ke[tid]);
        if (COLL && tid == 0 && s_v2) {
            const int half = 1 - *d.vcur;
            atomicMax(d.vmax2 + ((int64_t)half * kCntStripes + st) * d.nseg + sg, s_v2);
        }
    }
}

template <int STAGES, bool NT>
__global__ void __launch_bounds__(256) k_particles(Dev d, int hist_rt, int64_t T)
{
    const int64_t t = blockIdx.x;
    if (t >= T) return;
    const int64_t first = t * blockDim.x * kPpt64;
    const int sg = seg_of_slot(d, first);
    const int64_t last = min(first + (int64_t)blockDim.x * kPpt64, d.seg[sg].base + d.n_slots[sg]);
    if (first >= last) return;
    particles_body<STAGES, NT>(d, hist_rt, first, last, sg, *d.cur);
}

// One block per tile of the slot capacity (segment slot ranges are multiples of kSlotAlign,
// a multiple of every tile).
//
// The push streams its particles non-temporally once they outgrow the last-level cache (pass64_streams):
// cached and non-temporal 40.6 and 45.1 us at 4e6, 81 and 88 at 8e6, 145 and 130 at 1.2e7, 485 and
// 430 at 4e7.  The other stages read far less and write next to nothing in place.
hipError_t launch_pass64(const Dev &d, const Launch &L, hipStream_t s, int stages, int hist, bool pairs)
{
    const int block = L.block;
    const int rt = (hist ? kHist64 : 0) | (pairs ? kPairs : 0);
    static_assert(kSlotAlign % (256 * kPpt64) == 0, "whole tiles per segment");
    const int64_t T = d.cap_tot / (block * kPpt64);
    const dim3 g((unsigned)T);
#define PIC_CASE(ST)                                                                   \
    case ST:                                                                           \
        hipLaunchKernelGGL((k_particles<ST, false>), g, dim3(block), 0, s, d, rt, T);  \
        break;
    switch (stages) {
    case ST_PUSH:
        if (pass64_streams(L.lines))
            hipLaunchKernelGGL((k_particles<ST_PUSH, true>), g, dim3(block), 0, s, d, rt, T);
        else
            hipLaunchKernelGGL((k_particles<ST_PUSH, false>), g, dim3(block), 0, s, d, rt, T);
        break;
        PIC_CASE(ST_COLLIDE)
        PIC_CASE(ST_DEPOSIT)
        PIC_CASE(ST_HIST)
        PIC_CASE(ST_PUSH | ST_COLLIDE | ST_DEPOSIT)
        PIC_CASE(ST_PUSH | ST_DEPOSIT)
    default:
        return hipErrorInvalidValue;
    }
#undef PIC_CASE
    return hipGetLastError();
}

}  // namespace pic
