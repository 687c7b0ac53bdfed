// grad_linreg.hip -- local gradient (Eq. (1) of arXiv 2310.14423) of the linear least-squares
// workload for all K workers: loss_k = 1/(2B) sum_i (x_i.w_k - y_i)^2 with fresh Gaussian
// inputs x_i and targets y_i = x_i.w* + sigma*noise per (worker, iteration).
//   1. X[k] <- N(0,1)                              (Philox, stream X, drawn by the kernel of step 2)
//   2. r[k][i] = x_i.(w_k - w*) - sigma*eps_i      (one block per sample; the two inner
//      products are taken as one, which avoids cancellation when w_k is close to w*)
//   3. g[k][j] = (1/B) sum_i r[k][i] X[k][i][j];  loss[k] = 1/(2B) sum_i r^2
// The problem is tiny (K*B*d = 131072 inputs at the benchmark size): what counts is the number of
// launches in the dependent chain (2 to 4 us each) and of memory latencies inside them.  Every
// inner product needs all of w_k and every gradient entry all residuals, so two kernels per iteration
// are the least without a barrier across the grid; step 3's kernel therefore also takes the OPT update
// of its columns, which it holds for all workers, and in a recorded iteration the averaging and
// the scheduler's step.  256 iterations of 4 x 1024 features x 32 samples: 2879 us with four
// kernels per iteration (residuals, gradient, update, averaging).
#include "opt_elem.h"
#include "philox.h"
#include "qsr_internal.h"
#include "sched_dev.h"

namespace qsr {

__device__ __forceinline__ float block_sum_256(float v, float *red)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) red[wave] = v;
    __syncthreads();
    float s = red[0] + red[1] + red[2] + red[3];
    __syncthreads();
    return s;
}

// One workgroup per sample.  Wavefronts 0-3 draw the sample's inputs (whole groups of the generator,
// the same counters as a bulk fill of the flat [B][d] array: where d is not a multiple of 4 a row
// starts or ends inside a group, which the neighbouring row's workgroup draws too), store them for
// step 3 and take the inner product; wavefront 4 draws the observation noise meanwhile.
// WIDE (d no multiple of 4): 128-bit accesses for the groups inside the row, whose two ends take a path of their own after
// them: see launch_residual.
template <bool WIDE>
__global__ __launch_bounds__(320) void linreg_residual_kernel(
    float *__restrict__ X, const float *__restrict__ theta, const float *__restrict__ wstar,
    float *__restrict__ r, long long i0, long long B, long long d, float sigma, uint64_t seed,
    const DevState *__restrict__ st)
{
    __shared__ float red[5];
    const int k = blockIdx.y, tid = threadIdx.x, wave = tid >> 6;
    const long long i = (WIDE ? i0 : 0) + blockIdx.x;    // batches of more than one launch are WIDE
    const uint32_t t = (uint32_t)st->t;
    float acc = 0.f;
    if (wave < 4) {
        float *x = X + ((long long)k * B + i) * d;
        const float *w = theta + (long long)k * d;
        if ((d & 3) == 0) {
            for (long long q = tid; q < (d >> 2); q += 256) {
                const float4 wv = *(const float4 *)(w + q * 4), ws = *(const float4 *)(wstar + q * 4);
                const float4 z = normal4(seed, STREAM_X, (uint32_t)k, t, (uint32_t)(i * (d >> 2) + q));
                *(float4 *)(x + q * 4) = z;
                acc = fmaf(z.x, wv.x - ws.x, acc); acc = fmaf(z.y, wv.y - ws.y, acc);
                acc = fmaf(z.z, wv.z - ws.z, acc); acc = fmaf(z.w, wv.w - ws.w, acc);
            }
        } else {
            const long long f0 = i * d, q0 = f0 >> 2, nq = ((f0 + d + 3) >> 2) - q0;
            for (long long q = tid; q < nq; q += 256) {
                const long long j0 = (q0 + q) * 4 - f0;          // column of the group's first element
                if (WIDE) {
                    const float4 z = normal4(seed, STREAM_X, (uint32_t)k, t, (uint32_t)(q0 + q));
                    if (j0 >= 0 && j0 + 3 < d) {                 // all groups but the row's first and last
                        const float4 wv = ld4u(w + j0), ws = ld4u(wstar + j0);
                        st4u(x + j0, z);
                        acc = fmaf(z.x, wv.x - ws.x, acc); acc = fmaf(z.y, wv.y - ws.y, acc);
                        acc = fmaf(z.z, wv.z - ws.z, acc); acc = fmaf(z.w, wv.w - ws.w, acc);
                    } else {
                        const float zz[4] = {z.x, z.y, z.z, z.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (j0 + e >= 0 && j0 + e < d) { x[j0 + e] = zz[e]; acc = fmaf(zz[e], w[j0 + e] - wstar[j0 + e], acc); }
                    }
                    continue;
                }
                float dw[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const long long j = j0 + e;
                    dw[e] = j >= 0 && j < d ? w[j] - wstar[j] : 0.f;
                }
                const float4 z4 = normal4(seed, STREAM_X, (uint32_t)k, t, (uint32_t)(q0 + q));
                const float z[4] = {z4.x, z4.y, z4.z, z4.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const long long j = j0 + e;
                    if (j >= 0 && j < d) { x[j] = z[e]; acc = fmaf(z[e], dw[e], acc); }
                }
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
        if ((tid & 63) == 0) red[wave] = acc;
    } else if (tid == 256) {
        const float4 z = normal4(seed, STREAM_NOISE, (uint32_t)k, t, (uint32_t)(i >> 2));
        red[4] = (i & 3) == 0 ? z.x : (i & 3) == 1 ? z.y : (i & 3) == 2 ? z.z : z.w;
    }
    __syncthreads();
    if (tid == 0) r[(long long)k * B + i] = (red[0] + red[1] + red[2] + red[3]) - sigma * red[4];
}

// Step 3 with the OPT update, one workgroup per 64 columns of all K workers: K * S wavefronts, each on a
// worker's columns and every S-th run of samples (S = 16 / K: all loads of the benchmark size's 32
// samples are in flight at once); the S partial sums are added in order through LDS by the worker's first
// wavefront, which updates its columns.  average: the launch also averages, if the device's scheduler
// says that a round ends, with the averaging kernel's arithmetic.  st_next as in the update kernels.
struct LinregStep {
    float *theta, *g, *s0, *s1;          // s1: AdamW
    const StepScalars *sc;
    float c1, c2, eps;                   // SGD: c1 = mu, c2 = lambda
};
template <bool ADAMW>
__global__ __launch_bounds__(1024) void linreg_grad_update_kernel(
    const float *__restrict__ X, const float *__restrict__ r, LinregStep p, float *__restrict__ loss, int K, int S,
    long long B, long long d, const DevState *__restrict__ st, DevState *__restrict__ st_next, int average, SchedParams sp)
{
    __shared__ float part[16][64];
    __shared__ float upd[16][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int k = wave / S, s = wave - k * S;
    const long long j = (long long)blockIdx.x * 64 + lane;
    const bool in = j < d;
    // the last thread of the last workgroup, which has no column of its own where the others are busiest
    if (st_next != nullptr && blockIdx.x == gridDim.x - 1 && threadIdx.x == blockDim.x - 1) tick_into(st, st_next, sp);
    const bool sync = average != 0 && st->h + 1 == st->H;
    const StepScalars sc = p.sc[st->t];
    const long long o = (long long)k * d + j;
    float th = 0.f, m = 0.f, v = 0.f;
    if (s == 0 && in) {
        th = p.theta[o]; m = p.s0[o];
        if (ADAMW) v = p.s1[o];
    }
    const float *Xk = X + (long long)k * B * d + j;
    const float *rk = r + (long long)k * B;
    float acc = 0.f;
    if (in) {
        const long long per = (B + S - 1) / S, i0 = s * per, i1 = min(B, i0 + per);
        for (long long i = i0; i < i1; i += 8) {         // a short last run is filled up with weight 0
            float xv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) xv[u] = Xk[min(i + u, i1 - 1) * d];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc = fmaf(i + u < i1 ? rk[i + u] : 0.f, xv[u], acc);
        }
    }
    part[wave][lane] = acc;
    if (blockIdx.x == 0 && s == 0) {
        float a = 0.f;
        for (long long i = lane; i < B; i += 64) a = fmaf(rk[i], rk[i], a);
#pragma unroll
        for (int q = 32; q > 0; q >>= 1) a += __shfl_down(a, q, 64);
        if (lane == 0) loss[k] = 0.5f * a / (float)B;
    }
    __syncthreads();
    if (s == 0) {
        float gj = part[wave][lane];
        for (int q = 1; q < S; ++q) gj += part[wave + q][lane];
        gj *= 1.0f / (float)B;
        if (ADAMW) adamw_elem(th, gj, m, v, sc.x, sc.y, sc.z, p.c1, p.c2, p.eps);
        else sgdm_elem(th, gj, m, sc.x, p.c1, p.c2);
        upd[k][lane] = th;
        if (in) {
            p.g[o] = gj; p.s0[o] = m;
            if (ADAMW) p.s1[o] = v;
            if (!sync) p.theta[o] = th;
        }
    }
    if (!sync) return;                                   // the same for the whole launch
    __syncthreads();
    if (s == 0 && in) {
        float a = 0.f, c = 0.f;
        for (int q = 0; q < K; ++q) add_comp(a, c, upd[q][lane]);
        p.theta[o] = (a + c) / (float)K;
    }
}

__global__ __launch_bounds__(256) void linreg_grad_kernel(
    const float *__restrict__ X, const float *__restrict__ r, float *__restrict__ g,
    float *__restrict__ loss, long long B, long long d)
{
    __shared__ float red[4];
    const int k = blockIdx.y;
    const long long j = (long long)blockIdx.x * 256 + threadIdx.x;
    const float *Xk = X + (long long)k * B * d;
    const float *rk = r + (long long)k * B;
    const float invB = 1.0f / (float)B;
    if (j < d) {
        // eight loads in flight at a time (the launch has too few wavefronts to hide the latency of
        // one load per addition); the additions stay in sample order
        float acc = 0.f;
        long long i = 0;
        for (; i + 8 <= B; i += 8) {
            float xv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) xv[u] = Xk[(i + u) * d + j];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc = fmaf(rk[i + u], xv[u], acc);
        }
        for (; i < B; ++i) acc = fmaf(rk[i], Xk[i * d + j], acc);
        g[(long long)k * d + j] = acc * invB;
    }
    if (blockIdx.x == 0) {
        float a = 0.f;
        for (long long i = threadIdx.x; i < B; i += 256) a = fmaf(rk[i], rk[i], a);
        float s = block_sum_256(a, red);
        if (threadIdx.x == 0) loss[k] = 0.5f * s * invB;
    }
}

size_t linreg_workspace_bytes(const ModelDims &d)
{
    size_t x = (size_t)d.K * (size_t)d.B * (size_t)d.d_in * sizeof(float);
    size_t r = (size_t)d.K * (size_t)d.B * sizeof(float);
    return ((x + 255) & ~(size_t)255) + ((r + 255) & ~(size_t)255);
}

static float *linreg_r(const ModelDims &d, void *ws)
{
    size_t xb = ((size_t)d.K * d.B * d.d_in * sizeof(float) + 255) & ~(size_t)255;
    return (float *)((char *)ws + xb);
}

static hipError_t launch_residual(const ModelDims &d, const float *theta, const float *wstar, void *ws,
                                  const DevState *st, hipStream_t s)
{
    // Rows that are no multiple of 4 long: 128-bit accesses where there is enough work to be bound by them, 32-bit ones
    // where latency is all (an iteration, us, 128 / 32 bits: 8 x 184 x 2706723 10755 / 16600, 16 x 348 x 45554 601 / 874,
    // 24 x 341 x 270 42 / 45, 3 x 17 x 1003 8.25 / 8.14, 2 x 54 x 211 7.98 / 7.70).
    const bool wide = d.d_in >= 4096 || d.K * d.B >= 1024;
    auto kern = wide ? linreg_residual_kernel<true> : linreg_residual_kernel<false>;
    // a launch takes fewer than 2^32 threads in a grid dimension: runs of 2^23 samples
    for (long long i0 = 0; i0 < d.B; i0 += 1ll << 23) {
        const long long n = d.B - i0 < (1ll << 23) ? d.B - i0 : 1ll << 23;
        kern<<<dim3((unsigned)n, (unsigned)d.K), 320, 0, s>>>(
            (float *)ws, theta, wstar, linreg_r(d, ws), i0, d.B, d.d_in, d.data_sigma, d.seed, st);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_linreg_grad(const ModelDims &d, const float *theta, float *g, const float *wstar,
                              void *ws, float *loss, const DevState *st, hipStream_t s)
{
    hipError_t e = launch_residual(d, theta, wstar, ws, st, s);
    if (e != hipSuccess) return e;
    linreg_grad_kernel<<<dim3((unsigned)((d.d_in + 255) / 256), (unsigned)d.K), 256, 0, s>>>(
        (const float *)ws, linreg_r(d, ws), g, loss, d.B, d.d_in);
    return hipGetLastError();
}

// A wavefront per worker in a workgroup, and no share of samples so long that its chain of loads outlasts the wider
// gradient kernel and a separate update.  One iteration, fused against separate (us; as it was):
//   16 x 1024 features x 64 samples 16.4 / 13.3 (15.3), x 128 27.0 / 19.3 (20.7);  9 x 1024 x 32 9.8 / 9.8 (12.0),
//   x 64 13.4 / 11.9 (13.9);  8 x 1024 x 128 16.3 / 16.0 (17.7);  5 x 1024 x 128 13.0 / 14.8 (16.7)
bool linreg_can_fuse(const ModelDims &d)
{
    if (d.K > 16) return false;
    const long long S = 16 / d.K, per = (d.B + S - 1) / S;
    // 2^28 features and more: the launch would pass the limit of 2^32 threads in a grid dimension
    if ((d.d_in + 63) / 64 * (d.K * S * 64) >= 1ll << 32) return false;
    return per <= (S > 1 ? 64 : 32);
}

hipError_t launch_linreg_residual(const ModelDims &d, const float *theta, const float *wstar, void *ws,
                                  const DevState *st, hipStream_t s)
{
    return launch_residual(d, theta, wstar, ws, st, s);
}

hipError_t launch_linreg_grad_update(const ModelDims &d, float *theta, float *g, float *s0, float *s1, void *ws,
                                     float *loss, const StepScalars *sc, float c1, float c2, float eps,
                                     const DevState *st, DevState *st_next, bool average, const SchedParams &sp,
                                     hipStream_t s)
{
    if (!linreg_can_fuse(d)) return hipErrorInvalidValue;
    const int S = 16 / d.K;
    const LinregStep p{theta, g, s0, s1, sc, c1, c2, eps};
    const dim3 grid((unsigned)((d.d_in + 63) / 64));
    const int threads = d.K * S * 64;
    if (s1) linreg_grad_update_kernel<true><<<grid, threads, 0, s>>>((const float *)ws, linreg_r(d, ws), p, loss, d.K, S,
                                                                     d.B, d.d_in, st, st_next, average ? 1 : 0, sp);
    else linreg_grad_update_kernel<false><<<grid, threads, 0, s>>>((const float *)ws, linreg_r(d, ws), p, loss, d.K, S,
                                                                   d.B, d.d_in, st, st_next, average ? 1 : 0, sp);
    return hipGetLastError();
}

}  // namespace qsr
