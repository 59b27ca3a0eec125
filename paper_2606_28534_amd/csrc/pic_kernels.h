// pic_kernels.h -- host-side launchers of the gfx950 kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>

#include "pic_device.h"

namespace pic {

// Launch shape of the particle kernels.
struct Launch {
    int block;   // threads per block of the FP64 kernels (64, 128 or 256)
    int ppt;     // particles per thread per tile of the FP32 pass (4 or 8)
    int grid;    // the FP64 sort scatter's blocks / 8 (a multiple of 8 for the XCD-aware mapping)
    int window;  // widest LDS window span, in cells, of the FP32 pass and of the sorts
    int sort_ppt;  // particles per thread of the FP32 sort scatter
    int nt;        // fused FP32 pass with collisions: particle loads and stores by size (0), always non-temporal (1)
    int lines;     // of kStreamSlots, reached by the slots in use as the host last saw them
    int sort_nt;   // FP32 sort scatter: non-temporal loads
};

enum StageBits : int { SB_PUSH = 1, SB_COLLIDE = 2, SB_DEPOSIT = 4, SB_HIST = 8 };

// With the COLLIDE stage the null-collision bound kernel runs first unless `with_params`
// is false (the caller launched it).  Small FP32 runs collide their candidates in the pass
// (inline_candidates), all others in launch_candidates or launch_after.  Without `depo` the new
// pairs of the COLLIDE stage are left to a later deposit of every particle.
hipError_t launch_particles(const Dev &d, const Launch &L, hipStream_t s, bool f64, int stages, int hist,
                            bool with_params = true, bool depo = true);
hipError_t launch_pass64(const Dev &d, const Launch &L, hipStream_t s, int stages, int hist, bool pairs);
hipError_t launch_field_energy(const Dev &d, hipStream_t s);
// After a pass with the COLLIDE stage: the FP32 form's candidate kernel (no-op for FP64,
// whose pass scatters in place).  Without `depo` the new pairs are left to a later deposit of
// every particle (so too in launch_source).
hipError_t launch_candidates(const Dev &d, const Launch &L, hipStream_t s, bool f64, int hist, bool depo = true);
hipError_t launch_init(const Dev &d, bool f64, int sg, int64_t n, int64_t ppc, int init_mode,
                       double vth, double amp, int mode, hipStream_t s);
hipError_t launch_vmax(const Dev &d, bool f64, hipStream_t s);
hipError_t launch_zero_q(const Dev &d, bool f64, hipStream_t s);
// The field solve; with `with_births` its two kernels also scan and place the previous
// step's births in extra blocks (needs births_fit_solve: the one-block group scan); with
// `with_params` extra blocks of the first kernel reduce the striped speed maxima per segment
// and the second kernel's last block computes the null-collision bound from them; `advance`
// advances the step counter (with_births always does).  Small runs (Dev::small) take one
// kernel for all of it.
hipError_t launch_solve(const Dev &d, bool f64, int64_t nchunks, bool zero_q, hipStream_t s,
                        bool with_births = false, bool with_params = false, bool advance = false);
bool births_fit_solve(const Dev &d);
// A step of a small periodic run without collisions in one launch, from charge d.Qi to Qout (zero
// before), clearing Qzero: for the runs step_in_one_launch takes, on steps that neither sort nor
// count cells, when a full step follows before anyone reads the fields.
bool step_in_one_launch(const Dev &d);
hipError_t launch_step_small(const Dev &d, unsigned long long *Qout, unsigned long long *Qzero, hipStream_t s);
hipError_t launch_field_stats(const Dev &d, bool f64, int64_t nchunks, hipStream_t s);
hipError_t launch_params(const Dev &d, hipStream_t s);
int64_t scan_blocks(int64_t n);
hipError_t launch_births(const Dev &d, bool f64, bool in_step, bool advance, hipStream_t s);
hipError_t launch_advance(const Dev &d, hipStream_t s);
hipError_t launch_births_clear_all(const Dev &d, hipStream_t s);
hipError_t launch_sort(const Dev &d, bool f64, const Launch &L, hipStream_t s);
// The first half of a sort: the histogram's scan into run cursors and the segment starts.
hipError_t launch_sort_prepare(const Dev &d, hipStream_t s);
// FP32 fused pass that also scatters into cell order (after launch_sort_prepare), then the
// slot counts and the buffer flip.
hipError_t launch_pass32_sort(const Dev &d, const Launch &L, hipStream_t s, bool coll);
hipError_t launch_pass32(const Dev &d, const Launch &L, hipStream_t s, int stages, int hist, bool depo);
bool inline_candidates(const Dev &d, int ppt);
hipError_t launch_cand32(const Dev &d, int ppt, hipStream_t s, int hist, int64_t cap_tot, bool depo);
// the fused step's candidates, neutrals and source as one launch (FP32 form)
hipError_t launch_after(const Dev &d, int ppt, hipStream_t s, int hist, int64_t cap_tot, bool coll);
hipError_t launch_stream_copy(const void *src, void *dst, int64_t nwords, bool nt, hipStream_t s);
hipError_t launch_sort32_scatter(const Dev &d, int ppt, int W, hipStream_t s, int64_t cap_tot, bool nt);
// The adjoint window on a small grid (Dev::small), one launch per step in either direction.
struct AdjState {
    int32_t *cell;
    float *off, *vx;
};
hipError_t launch_adj_fwd(const Dev &d, const AdjState &in, const AdjState &out, const AdjState &ck,
                          unsigned long long *ckQ, unsigned long long *Qout, unsigned long long *Qzero, double *Erec,
                          int64_t n, int pushes, hipStream_t s);
hipError_t launch_adj_rev(int small, const double *lEin, double *lEout, double *lEzero, bool seed, double eps0,
                          double dx, double qw, const int32_t *xc1, const int32_t *xc, const float *xo, const double *E,
                          double *lx, double *lv, double *lEext, int64_t n, double dt, double qm, int N, hipStream_t s);
hipError_t launch_adj_seed(const double *E, double *lE, int N, double eps0, double dx, hipStream_t s);
hipError_t launch_adj_a(const Dev &d, const int32_t *xc, const float *xo, const double *E, double *lx,
                        double *lv, double *lE, double *lEext, int64_t n, double dt, double qm,
                        double dx, int N, hipStream_t s);
hipError_t launch_adj_grid(double *lE, double *lQ, double *tmp, int N, double dx, double eps0, double qw,
                           hipStream_t s);
hipError_t launch_adj_b(const int32_t *xc, const double *lQ, double *lx, int64_t n, double dx, int N,
                        hipStream_t s);
// out[id_i] = lv_i for n slots; ids >= len set *err (device int).
hipError_t launch_adj_by_id(const double *lv, const uint32_t *id, double *out, int64_t n, int64_t len,
                            int32_t *err, hipStream_t s);
// The same, with the number of distinct ids in *distinct; `seen` is a cleared bit per id.
hipError_t launch_adj_by_id_count(const double *lv, const uint32_t *id, double *out, uint32_t *seen, int64_t n,
                                  int64_t len, int32_t *err, uint32_t *distinct, hipStream_t s);
hipError_t launch_diag(const Dev &d, bool f64, int sg, double *out, int grid, hipStream_t s);
// The scalars of ensemble `en` into one record and its node arrays ([Q0, Q1, rho, phi, E][nn]
// doubles) into one run of device memory; the error flags and slots in use alone.  `out` of the records is host
// memory the device can write.
hipError_t launch_diag_pack(const Dev &d, int en, bool tallied, const double *v2, int ngrid, DiagPack *out,
                            hipStream_t s);
hipError_t launch_grid_pack(const Dev &d, bool f64, int en, int64_t nn, bool fields, double *out, hipStream_t s);
hipError_t launch_err_out(const Dev &d, int32_t *out, int64_t *slots, hipStream_t s);
// Node moments of segment sg (reading R27) into out[5][nn] (n, ux, uy, uz, T); nn is the
// node count of the segment's ensemble.  `out` is device memory the launch overwrites.
hipError_t launch_moments(const Dev &d, bool f64, int sg, int64_t nn, double *out, hipStream_t s);
// Recycled neutrals of the step (stream, recycle the absorbed ions the pass listed, flip
// buffers) and the volumetric source pairs (FP32 form; no-ops when unused).
hipError_t launch_neutrals(const Dev &d, hipStream_t s);
hipError_t launch_source(const Dev &d, int hist, hipStream_t s, bool depo = true);

}  // namespace pic
