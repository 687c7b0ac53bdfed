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
// are the least for a worker that is spread over the grid; step 3's kernel therefore also takes the OPT update
// of its columns, which it holds for all workers, and in a recorded iteration the averaging and
// the scheduler's step.  Iterations enqueued together (qsr_run) of a worker that fits one workgroup need no launch between
// them at all: linreg_run_kernel.  256 iterations of 4 x 1024 features x 32 samples: 2879 us with four
// kernels per iteration (residuals, gradient, update, averaging), 1900 with two, 560 together
// (644 where each of the 28 rounds ended a launch).
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

// Workers that fit one workgroup of 16 wavefronts (linreg_run_kernel): up to 1024 features, four consecutive ones a lane and
// so RunShape::row wavefronts a sample, `groups` samples side by side, each group of wavefronts on a run of at most
// `per` samples.  linreg_run_kernel and, where the update goes with the gradient, the kernels of single iterations
// (linreg_residual_row_kernel, linreg_grad_update_kernel) take their sums in this order, so that iterations give the same bits
// one by one and together: four columns of a lane in order, the lanes of a wavefront pairwise (lane_sum),
// the wavefronts of a sample in order; for the gradient the samples of a run in order, then the runs.
// In the workspace their rows of X are padded to a multiple of 4, the padding zero.
constexpr int RUN_MAX_D = 1024, RUN_MAX_PER = 8;
struct RunShape { int row, groups, per, d4; };
static inline RunShape run_shape(const ModelDims &d)
{
    RunShape q;
    q.row = (int)((d.d_in + 255) / 256);
    q.groups = 16 / q.row;
    q.per = (int)((d.B + q.groups - 1) / q.groups);
    q.d4 = (int)((d.d_in + 3) / 4 * 4);
    return q;
}
bool linreg_can_run(const ModelDims &d)
{
    return d.K <= 16 && d.d_in <= RUN_MAX_D && d.B <= 16 * RUN_MAX_PER && run_shape(d).per <= RUN_MAX_PER && linreg_can_fuse(d);
}
static inline long long row_stride(const ModelDims &d) { return linreg_can_run(d) ? run_shape(d).d4 : d.d_in; }
static inline size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

// Iterations together: X and the observation noise of RUN_SLOTS iterations at a time, drawn ahead
constexpr int RUN_SLOTS = LINREG_RUN_AHEAD;
static inline long long slot_worker_floats(const ModelDims &d) { return d.B * run_shape(d).d4 + (d.B + 3) / 4 * 4; }
static inline long long run_floats(const ModelDims &d) { return RUN_SLOTS * d.K * slot_worker_floats(d); }
// Library memory of a context: what the workers exchange where a round ends inside a launch, two rounds of it, a word for each
// parameter, [worker][wavefront of the row][of a lane's four][lane]; the flag of a wait given up; two copies of the parameters
static inline size_t exchange_bytes(const ModelDims &d) { return 2 * (size_t)d.K * run_shape(d).row * 256 * sizeof(unsigned long long); }
static inline float *copies(const ModelDims &d, void *shared) { return (float *)((char *)shared + exchange_bytes(d) + 256); }
size_t linreg_run_shared_bytes(const ModelDims &d) { return exchange_bytes(d) + 256 + 2 * (size_t)d.K * run_shape(d).d4 * sizeof(float); }
int *linreg_gave_up(const ModelDims &d, void *shared) { return (int *)((char *)shared + exchange_bytes(d)); }

// exchanges inside a wavefront: lane l gets the value of lane l ^ 8, l ^ 7, l ^ 2, l ^ 1
template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_xor8(float v) { return dpp<0x128>(v); }     // rotation of a row of 16 by 8
__device__ __forceinline__ float lane_xor7(float v) { return dpp<0x141>(v); }     // half rows mirrored
__device__ __forceinline__ float lane_xor2(float v) { return dpp<0x4e>(v); }
__device__ __forceinline__ float lane_xor1(float v) { return dpp<0xb1>(v); }
// a: lanes below 32 (an even row of 16) keep a, the others get b's; b: the reverse
__device__ __forceinline__ void swap32(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap16(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
}
// the sum over the wavefront, in every lane: pairs l, l ^ 32, then ^ 16, 8, 7, 2, 1
__device__ __forceinline__ float lane_sum(float v)
{
    float o = v;
    swap32(v, o); v += o;
    o = v; swap16(v, o); v += o;
    v += lane_xor8(v); v += lane_xor7(v); v += lane_xor2(v);
    return v + lane_xor1(v);
}
// The same sums of N = 2, 4 or 8 values at once: each exchange halves the values a lane still holds.  The lane ends up with
// the sum of value lane_value<N>(lane).
template <int N> __device__ __forceinline__ int lane_value(int lane)
{
    int i = (lane >> 5) * (N / 2);
    if (N >= 4) i += ((lane >> 4) & 1) * (N / 4);
    if (N >= 8) i += ((lane >> 3) & 1) * (N / 8);
    return i;
}
template <int N> __device__ __forceinline__ float lane_sums(float (&v)[N], int lane)
{
    constexpr int H = N / 2;
#pragma unroll
    for (int i = 0; i < H; ++i) { swap32(v[i], v[i + H]); v[i] += v[i + H]; }
    if constexpr (N >= 4) {
#pragma unroll
        for (int i = 0; i < H / 2; ++i) { swap16(v[i], v[i + H / 2]); v[i] += v[i + H / 2]; }
    } else {
        float o = v[0]; swap16(v[0], o); v[0] += o;
    }
    if constexpr (N >= 8) {
        const bool up = (lane & 8) != 0;
#pragma unroll
        for (int i = 0; i < H / 4; ++i) {
            const float give = up ? v[i] : v[i + H / 4], keep = up ? v[i + H / 4] : v[i];
            v[i] = keep + lane_xor8(give);
        }
    } else v[0] += lane_xor8(v[0]);
    v[0] += lane_xor7(v[0]);
    v[0] += lane_xor2(v[0]);
    return v[0] + lane_xor1(v[0]);
}

// Steps 1 and 2 for such workers, one workgroup per sample: 256 lanes draw the sample's inputs and own four columns each, a lane
// of wavefront 4 draws the noise.  Rows that are no multiple of 4 long begin inside a group of the generator: there the
// draws pass through LDS, whole groups at a time (what lies beyond the row's ends is masked where it is read), and the 257th
// group that such a row can touch is drawn by wavefront 4 too.  The parameters are loaded without a branch: behind one, each
// load was waited for before the draws.  Bound by latency; 3 x 1003 features x 17 samples 3.4 us, 4 x 1024 x 32 3.1 us
// (behind branches 3.4; four guarded stores a group 4.0 at 3 x 1003 x 17).  One structure as the argument: enqueueing an
// iteration's two kernels, 7.8 us with ten and fifteen arguments, takes 7.1, and single iterations of 3 x 1003 x 17 wait for the host.
struct LinregRows {
    float *X;
    const float *theta, *wstar;
    float *r;
    int B, d, d4;
    float sigma;
    uint64_t seed;
    const DevState *st;
};
template <bool ALIGNED>
__global__ __launch_bounds__(320) void linreg_residual_row_kernel(LinregRows a)
{
    const int B = a.B, d = a.d;
    __shared__ __attribute__((aligned(16))) float row[ALIGNED ? 4 : 4 + RUN_MAX_D + 4];   // column j at 4 + j, j from -3 on
    __shared__ float red[5];
    const int k = blockIdx.y, i = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, c = tid * 4;
    uint32_t t = (uint32_t)a.st->t;
    const float *wp = a.theta + (long long)k * d;
    float4 w, b;                                         // used behind the draws, which hide the latency
    if (ALIGNED) {
        const int j = min(c, d - 4);
        w = ld4u(wp + j); b = ld4u(a.wstar + j);
    } else {
        const int j[4] = {min(c, d - 1), min(c + 1, d - 1), min(c + 2, d - 1), min(c + 3, d - 1)};
        w = make_float4(wp[j[0]], wp[j[1]], wp[j[2]], wp[j[3]]);
        b = make_float4(a.wstar[j[0]], a.wstar[j[1]], a.wstar[j[2]], a.wstar[j[3]]);
    }
    asm volatile("" : "+s"(t));                          // requested first of all, not where the draws begin
    const long long f0 = (long long)i * d, q0 = f0 >> 2;
    const int nq = (int)(((f0 + d + 3) >> 2) - q0), q = min(tid, 256);
    const bool noise = tid == 256;
    float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
    if (noise || (tid < 258 && q < nq))
        z = normal4(a.seed, noise ? STREAM_NOISE : STREAM_X, (uint32_t)k, t, noise ? (uint32_t)(i >> 2) : (uint32_t)(q0 + q));
    if (noise) red[4] = (i & 3) == 0 ? z.x : (i & 3) == 1 ? z.y : (i & 3) == 2 ? z.z : z.w;
    if (!ALIGNED) {
        if (!noise && tid < 258 && q < nq) {
            float *to = row + 4 + (int)((q0 + q) * 4 - f0);
            to[0] = z.x; to[1] = z.y; to[2] = z.z; to[3] = z.w;
        }
        __syncthreads();
        if (wave < 4 && c < d) {
            z = *(const float4 *)(row + 4 + c);
            if (c + 1 >= d) z.y = 0.f;
            if (c + 2 >= d) z.z = 0.f;
            if (c + 3 >= d) z.w = 0.f;
        }
    }
    if (wave < 4) {
        float acc = 0.f;
        if (c < d) {
            *(float4 *)(a.X + ((long long)k * B + i) * a.d4 + c) = z;
            float dw[4] = {w.x - b.x, w.y - b.y, w.z - b.z, w.w - b.w};
#pragma unroll
            for (int e = 1; e < 4; ++e)
                if (!ALIGNED && c + e >= d) dw[e] = 0.f;
            acc = fmaf(z.x, dw[0], 0.f);
            acc = fmaf(z.y, dw[1], acc); acc = fmaf(z.z, dw[2], acc); acc = fmaf(z.w, dw[3], acc);
        }
        acc = lane_sum(acc);
        if ((tid & 63) == 0) red[wave] = acc;
    }
    __syncthreads();
    if (tid == 0) a.r[(long long)k * B + i] = fmaf(-a.sigma, red[4], ((red[0] + red[1]) + red[2]) + red[3]);
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

// Step 3 with the OPT update, one workgroup per 64 columns of KW workers.  The samples of a worker are cut into `runs` runs of
// `per`, whose sums are added in order; each of its wavefronts (threadIdx.y) takes one, eight samples' loads in
// flight, and leaves their sum in LDS, and the first one adds them up and updates the columns.  KW = 1: workers that
// linreg_run_kernel takes too, in its runs.  Else all K, 16 / K wavefronts each: the launch can average as well (average, if the
// device's scheduler says that a round ends), with the averaging kernel's arithmetic.  st_next as in the update kernels.  Bound by
// latency, of the instructions too (each launch fetches them anew: 16 samples unrolled, or the next eight requested ahead
// in code of their own, 0.5 to 1 us slower).  4 x 1024 x 32, KW = 1: 3.4 us (4.2 with KW = K).
struct LinregStep {
    float *theta, *g, *s0, *s1;          // s1: AdamW
    const StepScalars *sc;
    float c1, c2, eps;                   // SGD: c1 = mu, c2 = lambda
};
struct LinregGradStep {
    const float *X, *r;
    LinregStep p;
    float *loss;
    int K, runs, per, B, average, apart;   // apart: the scheduler's step has a workgroup of its own
    long long d, ldx;
    const DevState *st;
    DevState *st_next;
    SchedParams sp;
};
template <bool ADAMW>
__global__ __launch_bounds__(1024) void linreg_grad_update_kernel(LinregGradStep a)
{
    const LinregStep &p = a.p;
    const DevState *const st = a.st;
    const int runs = a.runs, per = a.per, B = a.B;
    const long long d = a.d, ldx = a.ldx;
    extern __shared__ float step_part[];                 // [KW][runs][64]
    float (*part)[64] = (float (*)[64])step_part;
    const int lane = threadIdx.x, s = __builtin_amdgcn_readfirstlane(threadIdx.y), kw = __builtin_amdgcn_readfirstlane(threadIdx.z);
    const int k = blockIdx.y * blockDim.z + kw;
    const long long j = (long long)blockIdx.x * 64 + lane;
    const bool in = j < d;
    if ((long long)blockIdx.x * 64 >= d) {               // a workgroup behind the columns
        if (blockIdx.y == 0 && lane == 0 && s == 0 && kw == 0) tick_into(st, a.st_next, a.sp);
        return;
    }
    // the last thread of the last workgroup, which has no column of its own where the others are busiest
    if (a.st_next != nullptr && !a.apart && blockIdx.x == gridDim.x - 1 && blockIdx.y == gridDim.y - 1 && lane == 63 && s == (int)blockDim.y - 1 &&
        kw == (int)blockDim.z - 1)
        tick_into(st, a.st_next, a.sp);
    const bool sync = a.average != 0 && st->h + 1 == st->H;
    const StepScalars sc = p.sc[st->t];
    const long long o = (long long)k * d + j;
    float th = 0.f, m = 0.f, v = 0.f;
    if (s == 0 && in) {
        th = p.theta[o]; m = p.s0[o];
        if (ADAMW) v = p.s1[o];
    }
    const int i0 = min(B, s * per), i1 = min(B, i0 + per);
    const float *rk = a.r + (long long)k * B;
    const float rv = i0 + lane < i1 ? rk[i0 + lane] : 0.f;      // the wavefront's residuals, one a lane
    const float *row = a.X + ((long long)k * B + i0) * ldx;
    const unsigned col = (unsigned)min(j, d - 1);
    float acc = 0.f;
    for (int i = i0; i < i1; i += 8) {                   // a short last group is filled up with weight 0
        float xv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            xv[u] = row[col];
            row += i + u + 1 < i1 ? ldx : 0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) acc = fmaf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(rv), i - i0 + u)), xv[u], acc);
    }
    if (i0 < i1) part[kw * runs + s][lane] = acc;
    if (blockIdx.x == 0 && s == 0) {
        float l = 0.f;
        for (int i = lane; i < B; i += 64) l = fmaf(rk[i], rk[i], l);
#pragma unroll
        for (int q = 32; q > 0; q >>= 1) l += __shfl_down(l, q, 64);
        if (lane == 0) a.loss[k] = 0.5f * l / (float)B;
    }
    __syncthreads();
    if (s == 0) {
        float gj = part[kw * runs][lane];
        for (int q = 1; q < runs; ++q) gj += part[kw * runs + q][lane];
        gj *= 1.0f / (float)B;
        if (ADAMW) adamw_elem(th, gj, m, v, sc.x, sc.y, sc.z, p.c1, p.c2, p.eps);
        else sgdm_elem(th, gj, m, sc.x, p.c1, p.c2);
        part[kw * runs][lane] = th;                      // for the average
        if (in) {
            p.g[o] = gj; p.s0[o] = m;
            if (ADAMW) p.s1[o] = v;
            if (!sync) p.theta[o] = th;
        }
    }
    if (!sync) return;                                   // the same for the whole launch
    __syncthreads();
    if (s == 0 && in) {
        float sum = 0.f, err = 0.f;
        for (int q = 0; q < a.K; ++q) add_comp(sum, err, part[q * runs][lane]);
        p.theta[o] = (sum + err) / (float)a.K;
    }
}

__global__ __launch_bounds__(256) void linreg_grad_kernel(
    const float *__restrict__ X, const float *__restrict__ r, float *__restrict__ g,
    float *__restrict__ loss, long long B, long long d, long long ldx)
{
    __shared__ float red[4];
    const int k = blockIdx.y;
    const long long j = (long long)blockIdx.x * 256 + threadIdx.x;
    const float *Xk = X + (long long)k * B * ldx;
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
            for (int u = 0; u < 8; ++u) xv[u] = Xk[(i + u) * ldx + j];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc = fmaf(rk[i + u], xv[u], acc);
        }
        for (; i < B; ++i) acc = fmaf(rk[i], Xk[i * ldx + j], acc);
        g[(long long)k * d + j] = acc * invB;
    }
    if (blockIdx.x == 0) {
        float a = 0.f;
        for (long long i = threadIdx.x; i < B; i += 256) a = fmaf(rk[i], rk[i], a);
        float s = block_sum_256(a, red);
        if (threadIdx.x == 0) loss[k] = 0.5f * s * invB;
    }
}

size_t linreg_workspace_bytes(const ModelDims &d, bool together)
{
    size_t x = (size_t)d.K * (size_t)d.B * (size_t)row_stride(d) * sizeof(float);
    size_t r = (size_t)d.K * (size_t)d.B * sizeof(float);
    size_t slots = together ? (size_t)run_floats(d) * sizeof(float) : 0;
    return up256(x) + up256(r) + up256(slots);
}

static float *linreg_r(const ModelDims &d, void *ws)
{
    return (float *)((char *)ws + up256((size_t)d.K * d.B * row_stride(d) * sizeof(float)));
}
static float *linreg_slots(const ModelDims &d, void *ws)
{
    return (float *)((char *)linreg_r(d, ws) + up256((size_t)d.K * d.B * sizeof(float)));
}

static hipError_t launch_residual(const ModelDims &d, const float *theta, const float *wstar, void *ws,
                                  const DevState *st, hipStream_t s)
{
    if (linreg_can_run(d)) {
        auto row = d.d_in % 4 == 0 ? linreg_residual_row_kernel<true> : linreg_residual_row_kernel<false>;
        row<<<dim3((unsigned)d.B, (unsigned)d.K), 320, 0, s>>>(
            LinregRows{(float *)ws, theta, wstar, linreg_r(d, ws), (int)d.B, (int)d.d_in, run_shape(d).d4, d.data_sigma, d.seed, st});
        return hipGetLastError();
    }
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
        (const float *)ws, linreg_r(d, ws), g, loss, d.B, d.d_in, row_stride(d));
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

// How linreg_grad_update_kernel shares the samples out
struct StepShape { int KW, S, runs, per; };
static StepShape step_shape(const ModelDims &d)
{
    const bool run = linreg_can_run(d);
    StepShape q;
    q.KW = run ? 1 : d.K;
    q.S = run ? run_shape(d).groups : 16 / d.K;
    q.per = run ? run_shape(d).per : (int)((d.B + q.S - 1) / q.S);
    q.runs = (int)((d.B + q.per - 1) / q.per);           // at most S, none of them empty
    return q;
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
    const StepShape q = step_shape(d);
    // a wavefront's residuals lie one a lane; the average needs all workers in a workgroup
    if (q.per > 64 || (average && q.KW < d.K)) return hipErrorInvalidValue;
    // The scheduler's step in a workgroup of its own: off the critical path, a workgroup more to start.  us an iteration at rounds
    // of one, apart / in the last wavefront: 1 x 4096 x 128 8.7 / 9.1, 12 x 2048 x 10 8.0 / 8.3, 5 x 1027 x 100 12.7 / 12.6, 3 x 1003 x 17
    // (single iterations) 7.2 / 6.9
    const bool apart = st_next != nullptr && d.d_in > 1536;
    const LinregGradStep a{(const float *)ws, linreg_r(d, ws), LinregStep{theta, g, s0, s1, sc, c1, c2, eps}, loss, d.K, q.runs,
                           q.per, (int)d.B, average ? 1 : 0, apart ? 1 : 0, d.d_in, row_stride(d), st, st_next, sp};
    const dim3 grid((unsigned)((d.d_in + 63) / 64 + (apart ? 1 : 0)), (unsigned)(d.K / q.KW)), block(64, (unsigned)q.S, (unsigned)q.KW);
    auto kern = s1 ? linreg_grad_update_kernel<true> : linreg_grad_update_kernel<false>;
    kern<<<grid, block, (size_t)q.KW * q.runs * 64 * sizeof(float), s>>>(a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// iterations together
// ---------------------------------------------------------------------------------------------
// Consecutive iterations in one launch, a workgroup of 16 wavefronts per worker: its parameters and momentum stay
// in registers, an iteration's inputs too, from the residuals to the gradient, and what has to be summed across wavefronts
// goes through LDS with two barriers per iteration.  The inputs depend on nothing that the iterations compute: the
// launch's other workgroups draw those of later iterations into the workspace (slot = iteration mod RUN_SLOTS), so that a worker
// only reads its own, one iteration ahead, into a second set of registers; these reads (128 KiB an iteration at 32 x 1024, 2000
// cycles of a compute unit's first-level cache) are spread over the iteration, where a burst of them holds up
// the arithmetic behind it (2.1 us an iteration, spread 1.5, without them 1.1).
// Between launches of a call the parameters stay in library memory, two copies that launches read and write in turn, so that the
// averaging of a round that ended with a launch is the next one's: every worker reads all rows, where the device's scheduler
// has just begun a round (a launch of its own: 4 us).  With WAIT a launch averages at its own end, and has no registers for more.
//
// WAIT: rounds end inside the launch too.  There, as every workgroup takes from its own reading of the schedule, the workers hand
// each other their parameters through memory: one 64-bit word for each, the value beside the iteration it is from, written and read past
// the caches that XCDs do not share.  A reader that finds the iteration has the value, and no flag, fence or launch is needed.  Rounds
// of a launch take two sets of words in turn: whoever writes a set again has read, in the other one, what all workers wrote behind
// their reading of this one.  The launch that draws a call's first inputs fills the words with an iteration that ends no round of the call.
// The wait is for workgroups that run or will: the K <= 16 workers are their launch's first workgroups, and the host
// keeps to devices and streams with compute units for 16 such launches at once.  Should a lane all the same have looked a.polls times
// (minutes), it waits no more, leaves NaN and sets a flag that every later reading of the state reports.
// Bound by the round trips to memory, 1.5 us for one and the words' way there.  us an iteration at rounds of 1 / 2 / 8, against launches that
// end with the round (those of one iteration: two kernels, the second averages):
//   4 x 1024 features x 32 samples 4.1 / 3.0 / 2.2, 7.2 / 5.5 / 2.5;  16 x 1024 x 32 8.0 / 5.0 / 2.75, 11.0 / 6.6 / 2.77;
//   16 x 257 x 8 5.8 / 3.6 / 1.86, 8.6 / 4.6 / 1.88;  1 x 256 x 64 2.6 / 2.1 / 1.7, 7.1 / 4.6 / 2.1
// (launches of 32 iterations, from 64 held ahead, would take another 0.2 off).  Draws that bypass the caches slow the workers' reads:
// 0.8 us an iteration.
// A lane's words next to each other instead of 64 apart take 0.7 us more a round, two workers a group of wavefronts at a time
// 0.5 more up to four workers and 0.2 less at sixteen.
// Without a round's end inside, launches without that code: it takes 6 to 18 registers more and a microsecond a launch (16 x 1000 x 20,
// rounds of 16, 128 iterations 276 us and 314 with it in all launches; 2 x 256 x 32, one long round, 185 and 199).
struct LinregRun {
    LinregStep p;                        // p.theta: where the parameters go
    const float *theta_in;               // where they come from: rows of ld_in (ld_out: p.theta's)
    long long ld_in, ld_out;
    const float *wstar;
    float *slots, *loss;
    unsigned long long *words;           // exchanged parameters: [2][K][row][4][64]
    int polls;                           // looks before a wait is given up (none, and no word counts, below 0)
    int K, B, d, d4, per, n_it, n_draw, draw_off;   // n_draw iterations from the current one plus draw_off on
    unsigned ends;                       // iterations that end a round, as the host's mirror expects
    int carried;                         // theta_in is averaged on the way in, if its round ended (not with WAIT)
    float sigma;
    uint64_t seed;
    const DevState *st;
    DevState *st_next, *st_last;         // after the launch's iterations, and before the last of them
    SchedParams sp;
};

// a workgroup's share of the draws: 1024 groups of the generator, of one iteration and worker
__device__ __forceinline__ void run_draw(const LinregRun &a, int block, int blocks, long long k_floats)
{
    const int it = block / (a.K * blocks), k = block / blocks % a.K;
    const long long t = a.st->t + a.draw_off + it;
    float *x = a.slots + ((t % RUN_SLOTS) * a.K + k) * k_floats, *eps = x + (long long)a.B * a.d4;
    const int n = a.B * a.d, groups = (n + 3) / 4;
    const int q = block % blocks * 1024 + threadIdx.x;
    if (q < groups) {
        const float4 z = normal4(a.seed, STREAM_X, (uint32_t)k, (uint32_t)t, (uint32_t)q);
        if (a.d4 == a.d) { *(float4 *)(x + q * 4) = z; return; }
        const float zz[4] = {z.x, z.y, z.z, z.w};
        int i = q * 4 / a.d, j = q * 4 - i * a.d;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (q * 4 + e < n) {
                x[i * a.d4 + j] = zz[e];
                if (++j == a.d) {
                    for (; j < a.d4; ++j) x[i * a.d4 + j] = 0.f;
                    j = 0; ++i;
                }
            }
        }
    } else if (q - groups < (a.B + 3) / 4) {
        *(float4 *)(eps + (q - groups) * 4) = normal4(a.seed, STREAM_NOISE, (uint32_t)k, (uint32_t)t, (uint32_t)(q - groups));
    }
}

template <int ROW, int PER, bool ADAMW, bool WAIT>
__global__ __launch_bounds__(1024) void linreg_run_kernel(LinregRun a)
{
    constexpr int GROUPS = 16 / ROW;
    const long long k_floats = (long long)a.B * a.d4 + (a.B + 3) / 4 * 4;
    const int workers = a.n_it > 0 ? a.K + 1 : 0;
    if ((int)blockIdx.x >= workers) {
        if (workers == 0)
            for (int i = blockIdx.x * 1024 + threadIdx.x; i < 2 * a.K * ROW * 256; i += gridDim.x * 1024)
                __hip_atomic_store(a.words + i, (unsigned long long)a.st->t << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        run_draw(a, blockIdx.x - workers, ((a.B * a.d + 3) / 4 + (a.B + 3) / 4 + 1023) / 1024, k_floats);
        return;
    }
    if ((int)blockIdx.x == a.K) {                        // the scheduler's steps
        if (threadIdx.x > 0) return;
        DevState nx = *a.st;
        SchedParams sp = a.sp;
        for (int i = 0; i < a.n_it; ++i) {
            sp.expect_sync = (int)(a.ends >> i & 1);
            if (i + 1 == a.n_it) *a.st_last = nx;
            sched_advance(&nx, sp);
        }
        *a.st_next = nx;
        return;
    }
    __shared__ __attribute__((aligned(16))) float red[16 * PER][4];     // inner products: [sample][wavefront of its row]
    __shared__ float4 part[16][64];                                     // gradient: [wavefront][lane], four columns
    __shared__ float res[16 * PER];                                     // residuals of the last iteration
    __shared__ float4 other[WAIT ? 16 : 1][64];                         // the averaging's, besides part
    const int k = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s = wave / ROW, cw = wave - s * ROW;
    const bool busy = s < GROUPS;                        // three wavefronts a row: one of the sixteen is left over
    const int c = cw * 256 + lane * 4;
    const bool in = busy && c < a.d;
    const int i0 = min(s * a.per, a.B), n_i = busy ? min(a.per, a.B - i0) : 0;
    const long long t0 = a.st->t, o = (long long)k * a.d + c;

    float th[4] = {0.f, 0.f, 0.f, 0.f}, m[4] = {0.f, 0.f, 0.f, 0.f}, v[4] = {0.f, 0.f, 0.f, 0.f}, ws[4] = {0.f, 0.f, 0.f, 0.f};
    float g[4] = {0.f, 0.f, 0.f, 0.f};
    const bool mean = !WAIT && a.carried && a.st->h == 0;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (in && c + e < a.d) {
            m[e] = a.p.s0[o + e]; ws[e] = a.wstar[c + e];
            if (ADAMW) v[e] = a.p.s1[o + e];
            if (!mean) th[e] = a.theta_in[k * a.ld_in + c + e];
        }
    if (mean && in) {                                    // rows of a copy: whole groups of four
        float4 row[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) row[q] = *(const float4 *)(a.theta_in + min(q, a.K - 1) * a.ld_in + c);
        float sum[4] = {0.f, 0.f, 0.f, 0.f}, err[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 16; ++q)
            if (q < a.K) {
                add_comp(sum[0], err[0], row[q].x); add_comp(sum[1], err[1], row[q].y);
                add_comp(sum[2], err[2], row[q].z); add_comp(sum[3], err[3], row[q].w);
            }
#pragma unroll
        for (int e = 0; e < 4; ++e) th[e] = c + e < a.d ? (sum[e] + err[e]) / (float)a.K : 0.f;
    }
    if (tid < 16 * PER) {                                // rows of fewer than four wavefronts
#pragma unroll
        for (int e = 0; e < 4; ++e) red[tid][e] = 0.f;
    }
    // an iteration's inputs: PER samples (beyond the run's, or the batch's, some that count for nothing), and the lane's noise
    struct In { float4 x[PER]; float eps; };
    const int u_own = lane & (PER - 1);
    auto slot = [&](int it) { return a.slots + (((t0 + it) % RUN_SLOTS) * a.K + k) * k_floats; };
    auto load = [&](const float *x, In &q, int u) { q.x[u] = *(const float4 *)(x + min(i0 + u, a.B - 1) * a.d4 + (in ? c : 0)); };
    auto load_noise = [&](const float *x, In &q) { q.eps = x[a.B * a.d4 + min(i0 + u_own, a.B - 1)]; };
    auto barrier = [&]() {                               // for LDS accesses only: the loads ahead stay in flight
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // the launch's per-iteration scalars, one iteration a lane, and the period of a round that starts behind it
    const StepScalars mine = a.p.sc[t0 + min(lane, a.n_it - 1)];
    int period = 0, to_go = 0;                           // to_go: iterations to the end of the round
    if constexpr (WAIT) {
        period = (int)min(get_H(a.sp, t0 + 1 + min(lane, a.n_it - 1)), 1ll << 20);
        to_go = (int)min(a.st->H - a.st->h, 1ll << 20);
    }
    int set = 0, polls = a.polls;
    // This worker's parameters to the others and everybody's mean, over the workers in order, each addition error-free: a worker a
    // group of wavefronts, GROUPS at a time through LDS, two places in turn
    auto average = [&](int it) {
        const unsigned t = (unsigned)t0 + it + 1;
        unsigned long long *const words = a.words + (set * a.K * ROW + cw) * 256 + lane;
        set ^= 1;
        if (s == 0 && in) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                __hip_atomic_store(words + k * ROW * 256 + e * 64, (unsigned long long)t << 32 | (unsigned)__float_as_int(th[e]),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        float sum[4] = {0.f, 0.f, 0.f, 0.f}, err[4] = {0.f, 0.f, 0.f, 0.f};
        for (int k0 = 0; k0 < a.K; k0 += GROUPS) {
            float4 (*const rows)[64] = k0 / GROUPS % 2 ? part : other;   // part: nobody reads it behind the first barrier here
            if (in && k0 + s < a.K) {
                unsigned long long w[4];
                bool there;
                do {
                    there = true;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        w[e] = __hip_atomic_load(words + (k0 + s) * ROW * 256 + e * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                    for (int e = 0; e < 4; ++e) there &= (unsigned)(w[e] >> 32) == t;
                } while (!there && --polls > 0);
                there &= polls >= 0;
                if (!there) *(int *)(a.words + 2 * a.K * ROW * 256) = 1;
                auto value = [&](int e) { return there ? __int_as_float((int)(unsigned)w[e]) : NAN; };
                rows[wave][lane] = make_float4(value(0), value(1), value(2), value(3));
            }
            barrier();
            if (in)
                for (int q = 0; q < min(GROUPS, a.K - k0); ++q) {
                    const float4 r = rows[cw + q * ROW][lane];
                    add_comp(sum[0], err[0], r.x); add_comp(sum[1], err[1], r.y);
                    add_comp(sum[2], err[2], r.z); add_comp(sum[3], err[3], r.w);
                }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) th[e] = in && c + e < a.d ? (sum[e] + err[e]) / (float)a.K : 0.f;
    };
    auto scalar = [&](float x, int it) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), it)); };
    barrier();
    auto iterate = [&](int it, In &q, In &ahead) {
        const bool last = it + 1 == a.n_it;
        // the loads ahead are made always: behind a branch, every wait for the loads before would be one for these too
        const float *x = slot(last ? it : it + 1);
        load_noise(x, ahead);
        const StepScalars sc = {scalar(mine.x, it), scalar(mine.y, it), scalar(mine.z, it), 0.f};
        float dw[4], dot[PER];
#pragma unroll
        for (int e = 0; e < 4; ++e) dw[e] = in ? th[e] - ws[e] : 0.f;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            float acc = fmaf(q.x[u].x, dw[0], 0.f);
            acc = fmaf(q.x[u].y, dw[1], acc); acc = fmaf(q.x[u].z, dw[2], acc);
            dot[u] = fmaf(q.x[u].w, dw[3], acc);
            if (u % 2 == 1) { load(x, ahead, u / 2); __builtin_amdgcn_sched_barrier(0); }
        }
        const float sum = lane_sums<PER>(dot, lane);
        if (busy && (lane & (64 / PER - 1)) == 0) red[s * PER + lane_value<PER>(lane)][cw] = sum;
        barrier();
        float r = 0.f;
        if (u_own < n_i) {
            const float4 d4 = *(const float4 *)red[s * PER + u_own];
            r = fmaf(-a.sigma, q.eps, ((d4.x + d4.y) + d4.z) + d4.w);
        }
        if (last && cw == 0 && lane < n_i) res[i0 + lane] = r;
#pragma unroll
        for (int e = 0; e < 4; ++e) g[e] = 0.f;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const float ru = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r), u));
            g[0] = fmaf(ru, q.x[u].x, g[0]); g[1] = fmaf(ru, q.x[u].y, g[1]);
            g[2] = fmaf(ru, q.x[u].z, g[2]); g[3] = fmaf(ru, q.x[u].w, g[3]);
            if (u % 2 == 1) { load(x, ahead, PER / 2 + u / 2); __builtin_amdgcn_sched_barrier(0); }
        }
        if (busy) part[wave][lane] = make_float4(g[0], g[1], g[2], g[3]);
        barrier();
        if (busy) {
            float4 p = part[cw][lane];
            g[0] = p.x; g[1] = p.y; g[2] = p.z; g[3] = p.w;
#pragma unroll
            for (int w = 1; w < GROUPS; ++w) {
                p = part[cw + w * ROW][lane];
                g[0] += p.x; g[1] += p.y; g[2] += p.z; g[3] += p.w;
            }
        }
        const float invB = 1.0f / (float)a.B;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            g[e] *= invB;
            if (ADAMW) adamw_elem(th[e], g[e], m[e], v[e], sc.x, sc.y, sc.z, a.p.c1, a.p.c2, a.p.eps);
            else sgdm_elem(th[e], g[e], m[e], sc.x, a.p.c1, a.p.c2);
        }
        if constexpr (WAIT) {
            if (--to_go == 0) {
                to_go = __builtin_amdgcn_readlane(period, it);
                average(it);
            }
        }
    };
    In q0, q1;
    load_noise(slot(0), q0);
#pragma unroll
    for (int u = 0; u < PER; ++u) load(slot(0), q0, u);
    for (int it = 0; it < a.n_it; it += 2) {
        iterate(it, q0, q1);
        if (it + 1 < a.n_it) iterate(it + 1, q1, q0);
    }
    if (s == 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (in && c + e < a.d) {
                a.p.theta[k * a.ld_out + c + e] = th[e]; a.p.s0[o + e] = m[e]; a.p.g[o + e] = g[e];
                if (ADAMW) a.p.s1[o + e] = v[e];
            }
    }
    if (wave == 15) {                                    // written before the last barrier
        float l = 0.f;
        for (int i = lane; i < a.B; i += 64) l = fmaf(res[i], res[i], l);
#pragma unroll
        for (int h = 32; h > 0; h >>= 1) l += __shfl_down(l, h, 64);
        if (lane == 0) a.loss[k] = 0.5f * l / (float)a.B;
    }
}

hipError_t launch_linreg_average_copy(const ModelDims &d, void *shared, int copy, const DevState *st, hipStream_t s)
{
    const long long d4 = run_shape(d).d4;
    return launch_average_rows(copies(d, shared) + copy * d.K * d4, d.K, d4, st, s);
}

// us that an exchange takes: 1.7 (2 workers x 256 features), 2.2 (4 x 1024), 2.6 (8 x 256), 4.0 (16 x 257), 6.0 (16 x 1000)
double linreg_exchange_us(const ModelDims &d)
{
    const int groups = run_shape(d).groups;
    return 1.0 + 0.8 * ((d.K + groups - 1) / groups) + 0.1 * d.K;
}

hipError_t launch_linreg_run(const ModelDims &d, float *theta, float *g, float *s0, float *s1, const float *wstar, void *ws, void *shared,
                             float *loss, const StepScalars *sc, float c1, float c2, float eps, const LinregSpan &span,
                             const SchedParams &sp, hipStream_t s)
{
    if (!linreg_can_run(d) || span.n_it < 0 || span.n_draw < 0 || span.n_it > LINREG_RUN_MAX || span.draw_off + span.n_draw > RUN_SLOTS)
        return hipErrorInvalidValue;
    // a round that ends before the last iteration needs workers that wait
    if (!span.wait && span.n_it > 0 && (span.ends & ((1u << (span.n_it - 1)) - 1)) != 0) return hipErrorInvalidValue;
    if (span.wait && span.mean) return hipErrorInvalidValue;
    const RunShape q = run_shape(d);
    LinregRun a{};
    a.slots = linreg_slots(d, ws);
    a.words = (unsigned long long *)shared;
    a.polls = span.polls - 1;
    auto copy = [&](int i) { return i < 0 ? theta : copies(d, shared) + (long long)i * d.K * q.d4; };
    a.p = LinregStep{copy(span.out), g, s0, s1, sc, c1, c2, eps};
    a.theta_in = copy(span.in);
    a.ld_in = span.in < 0 ? d.d_in : q.d4; a.ld_out = span.out < 0 ? d.d_in : q.d4;
    a.carried = span.mean;
    a.ends = span.ends;
    a.wstar = wstar; a.loss = loss;
    a.K = d.K; a.B = (int)d.B; a.d = (int)d.d_in; a.d4 = q.d4; a.per = q.per;
    a.n_it = span.n_it; a.n_draw = span.n_draw; a.draw_off = span.draw_off;
    a.sigma = d.data_sigma; a.seed = d.seed; a.st = span.st; a.st_next = span.st_next; a.st_last = span.st_last; a.sp = sp;
    const int blocks = (int)((d.B * d.d_in + 3) / 4 + (d.B + 3) / 4 + 1023) / 1024;
    const unsigned grid = (unsigned)((a.n_it > 0 ? d.K + 1 : 0) + a.n_draw * d.K * blocks);
    if (grid == 0) return hipSuccess;
#define RUN(ROW, PER, ADAMW) do { if (span.wait) linreg_run_kernel<ROW, PER, ADAMW, true><<<grid, 1024, 0, s>>>(a); \
                                  else linreg_run_kernel<ROW, PER, ADAMW, false><<<grid, 1024, 0, s>>>(a); } while (0)
#define RUN_OPT(ROW, PER) do { if (s1) RUN(ROW, PER, true); else RUN(ROW, PER, false); } while (0)
#define RUN_ROW(ROW) do { if (q.per <= 2) RUN_OPT(ROW, 2); else if (q.per <= 4) RUN_OPT(ROW, 4); else RUN_OPT(ROW, 8); } while (0)
    if (q.row == 1) RUN_ROW(1); else if (q.row == 2) RUN_ROW(2); else if (q.row == 3) RUN_ROW(3); else RUN_ROW(4);
#undef RUN_ROW
#undef RUN_OPT
#undef RUN
    return hipGetLastError();
}

}  // namespace qsr
