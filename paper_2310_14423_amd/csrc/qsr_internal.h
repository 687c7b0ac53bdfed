// qsr_internal.h -- declarations shared by the library's HIP sources (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qsr.h"

namespace qsr {

// Scheduler state of Alg. 2 (arXiv 2310.14423), resident in device memory.  Kernels read the
// iteration counter from here, so the host never has to wait for the device between steps.
struct DevState {
    long long t;        // global iterations done
    long long s;        // finished rounds
    long long h;        // local steps done in the current round
    long long H;        // synchronization period of the current round (0 once t == T)
    int mismatch;       // set (and kept) when the host's mirror of the schedule expected another decision
};

// Per-iteration scalars of the OPT update, prepared on the host in double precision and
// rounded once to float.  SGD: x = eta_t.  AdamW: x = eta_t*lambda, y = eta_t/(1-beta1^n),
// z = 1/sqrt(1-beta2^n), n = t+1.
struct StepScalars {
    float x, y, z, w;
};

struct SchedParams {
    long long T, T_warm;
    long long H_base;
    long long t_local_start; // post-local phase: H = 1 for rounds starting before it
    long long t_swap_start;  // SWAP phase: a round starting at or after it runs to T; 0 = off
    int power;               // exponent of the rule; 0 = constant H_base
    double alpha;
    const double *eta;      // [T] device
    long long *log_t;       // [T] device: iteration count at each averaging
    long long *log_H;       // [T] device: period of each finished round
    int expect_sync;        // per launch: what the host's mirror of the schedule expects of this iteration (1: it ends
                            // a round), compared with the device's own decision; -1 = no check (recorded launches)
};

// 128-bit streaming (non-temporal) global accesses: data touched once per kernel
typedef float vf4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 ld_nt4(const float4 *p)
{
    vf4 v = __builtin_nontemporal_load((const vf4 *)p);
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st_nt4(float4 *p, float4 v)
{
    vf4 w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, (vf4 *)p);
}

// Four consecutive floats at any 4-byte address: rows whose length is not a multiple of 4 start
// anywhere, and the hardware takes 128-bit global accesses at 4-byte alignment.  Cached, not
// streaming: a wavefront's run of 1 KiB starts and ends inside a 128-byte line, whose other part its
// neighbour writes, and L2 has to hold the line until both have.
typedef float vf4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 ld4u(const float *p)
{
    vf4u v = *(const vf4u *)p;
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st4u(float *p, float4 v)
{
    vf4u w = {v.x, v.y, v.z, v.w};
    *(vf4u *)p = w;
}
// Column group c of a row of P floats: P4 = P / 4 whole groups of four, then rem = P % 4 left over.
// rem == 0: every row is 16-byte aligned (the buffers are).
__device__ __forceinline__ float4 ld_group(const float *row, long long c, long long P4, int rem)
{
    const float *p = row + c * 4;
    if (rem == 0) return ld_nt4((const float4 *)p);
    if (c < P4) return ld4u(p);
    return make_float4(p[0], rem > 1 ? p[1] : 0.f, rem > 2 ? p[2] : 0.f, 0.f);
}
__device__ __forceinline__ void st_group(float *row, long long c, long long P4, int rem, float4 v)
{
    float *p = row + c * 4;
    if (rem == 0) { st_nt4((float4 *)p, v); return; }
    if (c < P4) { st4u(p, v); return; }
    p[0] = v.x;
    if (rem > 1) p[1] = v.y;
    if (rem > 2) p[2] = v.z;
}

// streams of the counter-based generator (second counter word)
enum : uint32_t { STREAM_GRAD = 0, STREAM_X = 1, STREAM_NOISE = 2, STREAM_LABEL = 3 };

// records the hipError_t that qsr_last_hip_error() reports for the calling thread
void set_last_hip_error(int code);

// ---- launchers (each returns the hipError_t of its launch) --------------------------------
// st[0] and st[1] <- the state at t = 0 (both copies); both clear *gave_up (linreg_gave_up) unless it is NULL
hipError_t launch_sched_init(DevState *st, SchedParams sp, int *gave_up, hipStream_t s);
hipError_t launch_sched_set(DevState *st, SchedParams sp, long long t, long long s_, long long h, long long H,
                            int *gave_up, hipStream_t s);
// *dst <- *src (the two copies of the scheduler state)
hipError_t launch_sched_copy(DevState *dst, const DevState *src, hipStream_t s);
// end of an iteration (where no update kernel has taken the step): t += 1, h += 1 and, if that was the round's
// H-th step, the round is logged and the next one opened
hipError_t launch_sched_advance(DevState *st, SchedParams sp, hipStream_t s);

// fused_sync: leave the step that completes a round to launch_update_*_sync.
// row_coef: K clipping factors the gradient rows are multiplied by as they are read, or nullptr.
// shared_g: the K gradient rows are known to be equal (Parallel OPT).
// own_gradient: a kernel of this library has just written g (else a caller's backward pass).
// st_next != nullptr (with sp): the kernel also takes the scheduler's end-of-iteration step: the advanced
// state goes to *st_next, a second copy that no kernel of this iteration reads (an averaging kernel behind
// it decides on the copy the iteration began with).
hipError_t launch_update_sgdm(float *theta, float *g, float *buf, int K, long long P,
                              const DevState *st, const StepScalars *sc, float mu, float lambda,
                              bool fused_sync, const float *row_coef, bool shared_g, bool own_gradient, hipStream_t s,
                              DevState *st_next = nullptr, const SchedParams *sp = nullptr);
hipError_t launch_update_adamw(float *theta, float *g, float *m, float *v, int K, long long P,
                               const DevState *st, const StepScalars *sc, float c1, float c2,
                               float eps, bool fused_sync, const float *row_coef, bool shared_g, bool own_gradient, hipStream_t s,
                               DevState *st_next = nullptr, const SchedParams *sp = nullptr);
// the same updates with the optimizer-only workloads' gradient g = sigma * N(0,1) drawn inside the
// kernel (and written to g if store_g); P must be a multiple of 4
hipError_t launch_update_sgdm_noise(float *theta, float *g, float *buf, int K, long long P, const DevState *st,
                                    const StepScalars *sc, float mu, float lambda, float sigma, uint64_t seed,
                                    bool store_g, hipStream_t s, DevState *st_next = nullptr,
                                    const SchedParams *sp = nullptr);
hipError_t launch_update_adamw_noise(float *theta, float *g, float *m, float *v, int K, long long P,
                                     const DevState *st, const StepScalars *sc, float c1, float c2, float eps,
                                     float sigma, uint64_t seed, bool store_g, hipStream_t s,
                                     DevState *st_next = nullptr, const SchedParams *sp = nullptr);
// update + averaging in one pass over the [K][P] buffers, only on the step that completes a round
hipError_t launch_update_sgdm_sync(float *theta, const float *g, float *buf, int K, long long P,
                                   const DevState *st, const StepScalars *sc, float mu, float lambda,
                                   const float *row_coef, hipStream_t s);
hipError_t launch_update_adamw_sync(float *theta, const float *g, float *m, float *v, int K, long long P,
                                    const DevState *st, const StepScalars *sc, float c1, float c2,
                                    float eps, const float *row_coef, hipStream_t s);

// gradient clipping: coef[k] = min(1, max_norm / (||g_k|| + 1e-6)), norm[k] = ||g_k||;
// partial: K * clip_blocks_per_row(P) doubles of scratch.  same_rows: the rows are known to be equal, only the
// first is read.
int clip_blocks_per_row(long long P);
hipError_t launch_clip_coef(const float *g, int K, long long P, float max_norm, double *partial, float *coef,
                            float *norm, hipStream_t s, bool same_rows = false);
// device address, on the current device, of the partial-sum array inside the library's image
// (qsr_clip_factors_static); looked up at the first call on a device.  Returns a QSR_* code.
int clip_static_setup(double **out);

// mean over the K rows of buf [K][P], written to all rows; with st != nullptr the launch acts only
// if the iteration in progress completes its round (st->h + 1 == st->H, read before the advance)
hipError_t launch_average_rows(float *buf, int K, long long P, const DevState *st, hipStream_t s);
hipError_t launch_broadcast_rows(float *dst, const float *src, int K, long long P, hipStream_t s);
hipError_t launch_fill_zero(float *dst, long long n, hipStream_t s);

// out[k*row_stride + i] = sigma * z for i < n, z ~ N(0,1) keyed (seed; i/4, stream, k, st->t)
hipError_t launch_fill_normal(float *out, long long row_stride, int K, long long n, float sigma,
                              uint32_t stream, uint64_t seed, const DevState *st, hipStream_t s);
hipError_t launch_noise_grad(float *g, int K, long long P, float sigma, uint64_t seed,
                             const DevState *st, hipStream_t s);

struct ModelDims {
    int K;
    long long P, B, d_in, d_hidden, d_out;
    int n_blocks;
    int n_heads;            // residual-MLP model: attention heads per block, 0 = none
    long long seq_len;      //   tokens per sequence (attention only)
    float data_sigma;
    uint64_t seed;
};

// together: launch_linreg_run will be used, which keeps the inputs of LINREG_RUN_AHEAD iterations
size_t linreg_workspace_bytes(const ModelDims &d, bool together);
hipError_t launch_linreg_grad(const ModelDims &d, const float *theta, float *g, const float *wstar,
                              void *ws, float *loss, const DevState *st, hipStream_t s);

// The same gradient in two launches of which the second also takes the OPT update (s1 != nullptr: AdamW with
// c1 = 1 - beta1, c2 = 1 - beta2; else SGD with c1 = mu, c2 = lambda), the scheduler's step (st_next as above)
// and, with average, the round's averaging where the device's scheduler says so (not for workers that linreg_can_run).
bool linreg_can_fuse(const ModelDims &d);
hipError_t launch_linreg_residual(const ModelDims &d, const float *theta, const float *wstar, void *ws,
                                  const DevState *st, hipStream_t s);
hipError_t launch_linreg_grad_update(const ModelDims &d, float *theta, float *g, float *s0, float *s1, void *ws,
                                     float *loss, const StepScalars *sc, float c1, float c2, float eps,
                                     const DevState *st, DevState *st_next, bool average, const SchedParams &sp,
                                     hipStream_t s);

// Iterations together: n_it of them, for workers that fit one workgroup each (least
// squares), and the draws of n_draw iterations from the current one plus draw_off on, which a later launch's iterations read.  The
// same bits as one by one.  A launch of draws alone (n_it = 0) has to come first in a call, and the launches of a call one behind the other.
constexpr int LINREG_RUN_AHEAD = 32, LINREG_RUN_MAX = 16;      // draws held, iterations of a launch
constexpr int LINREG_RUN_POLLS = 1 << 27;                      // looks, of about a microsecond, before a wait is given up
struct LinregSpan {
    int n_it, draw_off, n_draw;
    int in, out;                     // parameters read and written: -1 the caller's, 0 and 1 copies in `shared`
    bool wait;                       // rounds end inside the launch, where the workers wait for each other; otherwise one may end with it,
                                     // whose averaging is left to the next launch or to launch_average_rows
    bool mean;                       // if a round has just ended, the parameters read are averaged first (not with wait)
    unsigned ends;                   // bit i: iteration i ends a round, as the host's mirror expects
    int polls;                       // looks before a wait is given up
    const DevState *st;
    DevState *st_next, *st_last;     // the state after the iterations, and before the last of them
};
bool linreg_can_run(const ModelDims &d);
// `shared`, device memory (256-byte aligned, contents irrelevant before a call): what the workers exchange where a round ends, copies of the
// parameters, and a flag that a launch sets where a wait is given up (launch_sched_init and launch_sched_set clear it)
size_t linreg_run_shared_bytes(const ModelDims &d);
int *linreg_gave_up(const ModelDims &d, void *shared);
double linreg_exchange_us(const ModelDims &d);
// the averaging of a copy, if *st says that the round ends
hipError_t launch_linreg_average_copy(const ModelDims &d, void *shared, int copy, const DevState *st, hipStream_t s);
hipError_t launch_linreg_run(const ModelDims &d, float *theta, float *g, float *s0, float *s1, const float *wstar, void *ws, void *shared,
                             float *loss, const StepScalars *sc, float c1, float c2, float eps, const LinregSpan &span,
                             const SchedParams &sp, hipStream_t s);

size_t mlp2_workspace_bytes(const ModelDims &d);
hipError_t launch_mlp2_grad(const ModelDims &d, const float *theta, float *g, const float *means,
                            void *ws, float *loss, const DevState *st, hipStream_t s);

size_t resmlp_workspace_bytes(const ModelDims &d);
hipError_t launch_resmlp_grad(const ModelDims &d, const float *theta, float *g, const float *teacher,
                              void *ws, float *loss, const DevState *st, hipStream_t s);

}  // namespace qsr
