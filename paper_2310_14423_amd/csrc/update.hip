// update.hip -- fused multi-replica OPT update (Alg. 2's "OPT" line of arXiv 2310.14423, for
// all K workers in one launch).  The K rows share eta_t and every scalar, so the [K][P] buffers
// are treated as one vector of K*P elements.  The kernels are HBM-bound (AdamW: 16 B read +
// 12 B written per element; SGD: 12 B + 8 B): 128-bit accesses, several independent loads in
// flight per lane, streaming (non-temporal) hints because nothing is re-read within a step.
// Launch shape, from a sweep on MI355X at K*P = 0.96e9: one-wavefront workgroups that each make
// a single trip (no grid-stride loop) over 2 x 64 float4 per array reached 5.85 TB/s, against
// 5.0-5.1 TB/s for 256-thread blocks in a capped persistent grid and 5.77 TB/s for a plain
// copy kernel; non-temporal loads and stores were each worth 3-5 %.
#include "opt_elem.h"
#include "sched_dev.h"
#include "philox.h"
#include "qsr_internal.h"

namespace qsr {

constexpr int UPD_THREADS = 64;
constexpr int UPD_UNROLL = 2;      // float4 per array per thread per trip

// KEEP: plain accesses, for buffers that the caches hold from one launch to the next
template <bool KEEP>
__device__ __forceinline__ float4 ldg(const float4 *p) { return KEEP ? *p : ld_nt4(p); }
template <bool KEEP>
__device__ __forceinline__ void stg(float4 *p, float4 v)
{
    if (KEEP) *p = v;
    else st_nt4(p, v);
}

// `fused_sync`: the context folds the averaging into the last local step of a round (see the
// *_sync kernels below), so the plain update leaves that step alone.
// CLIP: the gradient is multiplied by its worker's clipping factor as it is read.  The buffers stay one
// vector of K*P elements, 16-byte aligned whatever P is; a workgroup's run of 512 elements holds at
// most one row boundary (P >= 512), found once per trip.  (With one grid row per worker, rows of
// odd length had to go one element at a time: 85 us for 8 x 3000001 SGD, 20 B per element.)
// SHARED (Parallel OPT): all workers' gradients are the same row, so only row 0 is read: one grid row per worker,
// n4 and n one worker's row; the row stays in the caches while the workers go over it (343 us for 28 B per element
// at 16 x 4000004 AdamW before).
// NOISE (optimizer-only workloads): the gradient is not read but drawn here, g = sigma * N(0,1)
// from the same Philox counters and with the same arithmetic as fill_normal_kernel.  The separate
// fill is bound by its arithmetic (about 220 vector instructions per four normals), this kernel by
// HBM, and the draw hides completely behind the loads of theta, m and v (timed on MI355X at
// 16 x 60e6: 4.02 ms against 4.63 ms for the update that reads g plus 1.01 ms for the fill).
// One grid row per worker: the draw's counters are a worker's own.  With `store` the draw is also written to the gradient
// buffer (4 B written in place of the 4 B read: 28 B per element as before, but the write-heavier
// mix runs at 5.5 TB/s instead of 5.8: 4.91 ms); without, the gradient never exists in HBM and
// the kernel moves 12 B read + 12 B written = 24 B per element.
struct NoiseDraw { float sigma; uint64_t seed; int store; };

// Worker of an element of the flat K*P vector.
struct RowAt { long long k, bound; float c0, c1; };   // row of a run's first element, where it ends, its factor and the next row's
struct RowMap {
    long long P; int K; double invP;
    __device__ __forceinline__ long long row(long long e) const
    {
        long long k = (long long)((double)e * invP);
        if (k * P > e) --k;                              // the product is off by an ulp at most
        if ((k + 1) * P <= e) ++k;
        return k;
    }
    __device__ __forceinline__ RowAt at(long long e, const float *coef) const
    {
        RowAt r;
        r.k = row(e);
        r.bound = (r.k + 1) * P;
        r.c0 = coef[min(r.k, (long long)K - 1)];
        r.c1 = coef[min(r.k + 1, (long long)K - 1)];
        return r;
    }
};
__device__ __forceinline__ void scale_by_row(float4 &b, long long e, const RowAt &ra, const RowMap &rm,
                                             const float *__restrict__ coef)
{
    if (rm.P >= UPD_THREADS * UPD_UNROLL * 4) {          // at most one boundary in the run
        b.x *= e < ra.bound ? ra.c0 : ra.c1;     b.y *= e + 1 < ra.bound ? ra.c0 : ra.c1;
        b.z *= e + 2 < ra.bound ? ra.c0 : ra.c1; b.w *= e + 3 < ra.bound ? ra.c0 : ra.c1;
    } else {
        b.x *= coef[rm.row(e)];     b.y *= coef[rm.row(e + 1)];
        b.z *= coef[rm.row(e + 2)]; b.w *= coef[rm.row(e + 3)];
    }
}

template <bool CLIP, bool NOISE, bool SHARED, bool KEEP = false>
__global__ __launch_bounds__(UPD_THREADS) void update_adamw_kernel(
    float4 *__restrict__ theta, float4 *__restrict__ g, float4 *__restrict__ m,
    float4 *__restrict__ v, long long n4, long long n, const DevState *__restrict__ st,
    const StepScalars *__restrict__ sc, float c1, float c2, float eps, int fused_sync,
    const float *__restrict__ row_coef, RowMap rm, NoiseDraw nd, DevState *__restrict__ st_next, SchedParams sp)
{
    if (st_next != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) tick_into(st, st_next, sp);
    if (fused_sync && st->h + 1 == st->H) return;
    if (NOISE || SHARED) {
        const long long off = (long long)blockIdx.y * n4;      // rows are 16-byte aligned here
        theta += off; m += off; v += off;
        if (!SHARED) g += off;
    }
    const float gs = SHARED && row_coef != nullptr ? row_coef[0] : 1.0f;
    const long long t = st->t;
    const StepScalars s = sc[t];
    const long long stride = (long long)gridDim.x * UPD_THREADS * UPD_UNROLL;
    long long base = (long long)blockIdx.x * UPD_THREADS * UPD_UNROLL + threadIdx.x;
    for (; base < n4; base += stride) {
        float4 a[UPD_UNROLL], b[UPD_UNROLL], c[UPD_UNROLL], d[UPD_UNROLL];
#pragma unroll
        for (int u = 0; u < UPD_UNROLL; ++u) {
            long long i = base + (long long)u * UPD_THREADS;
            if (i < n4) {
                a[u] = ldg<KEEP>(theta + i); c[u] = ldg<KEEP>(m + i); d[u] = ldg<KEEP>(v + i);
                if (!NOISE) b[u] = SHARED ? g[i] : ldg<KEEP>(g + i);
            }
            if (SHARED) { b[u].x *= gs; b[u].y *= gs; b[u].z *= gs; b[u].w *= gs; }
        }
        if (CLIP) {
            const RowAt ra = rm.at((base - threadIdx.x) * 4, row_coef);
#pragma unroll
            for (int u = 0; u < UPD_UNROLL; ++u) {
                const long long i = base + (long long)u * UPD_THREADS;
                if (i < n4) scale_by_row(b[u], i * 4, ra, rm, row_coef);
            }
        }
        if (NOISE) {
#pragma unroll
            for (int u = 0; u < UPD_UNROLL; ++u) {
                long long i = base + (long long)u * UPD_THREADS;
                if (i < n4) {
                    b[u] = normal4(nd.seed, STREAM_GRAD, blockIdx.y, (uint32_t)t, (uint32_t)i);
                    b[u].x *= nd.sigma; b[u].y *= nd.sigma; b[u].z *= nd.sigma; b[u].w *= nd.sigma;
                }
            }
            if (nd.store) {
#pragma unroll
                for (int u = 0; u < UPD_UNROLL; ++u) {
                    long long i = base + (long long)u * UPD_THREADS;
                    if (i < n4) stg<KEEP>(g + i, b[u]);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < UPD_UNROLL; ++u) {
            long long i = base + (long long)u * UPD_THREADS;
            if (i < n4) {
                adamw_elem(a[u].x, b[u].x, c[u].x, d[u].x, s.x, s.y, s.z, c1, c2, eps);
                adamw_elem(a[u].y, b[u].y, c[u].y, d[u].y, s.x, s.y, s.z, c1, c2, eps);
                adamw_elem(a[u].z, b[u].z, c[u].z, d[u].z, s.x, s.y, s.z, c1, c2, eps);
                adamw_elem(a[u].w, b[u].w, c[u].w, d[u].w, s.x, s.y, s.z, c1, c2, eps);
                stg<KEEP>(theta + i, a[u]); stg<KEEP>(m + i, c[u]); stg<KEEP>(v + i, d[u]);
            }
        }
    }
    // ragged tail (n not a multiple of 4): at most 3 elements, done by the first threads
    if (!NOISE && !SHARED && blockIdx.x == 0 && threadIdx.x < (int)(n - n4 * 4)) {
        long long i = n4 * 4 + threadIdx.x;
        float *th = (float *)theta, *mm = (float *)m, *vv = (float *)v;
        float gi = ((const float *)g)[i];
        if (CLIP) gi *= row_coef[rm.row(i)];
        float a = th[i], c = mm[i], d = vv[i];
        adamw_elem(a, gi, c, d, s.x, s.y, s.z, c1, c2, eps);
        th[i] = a; mm[i] = c; vv[i] = d;
    }
}

template <bool CLIP, bool NOISE, bool SHARED, bool KEEP = false>
__global__ __launch_bounds__(UPD_THREADS) void update_sgdm_kernel(
    float4 *__restrict__ theta, float4 *__restrict__ g, float4 *__restrict__ buf,
    long long n4, long long n, const DevState *__restrict__ st,
    const StepScalars *__restrict__ sc, float mu, float lambda, int fused_sync,
    const float *__restrict__ row_coef, RowMap rm, NoiseDraw nd, DevState *__restrict__ st_next, SchedParams sp)
{
    if (st_next != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) tick_into(st, st_next, sp);
    if (fused_sync && st->h + 1 == st->H) return;
    if (NOISE || SHARED) {
        const long long off = (long long)blockIdx.y * n4;
        theta += off; buf += off;
        if (!SHARED) g += off;
    }
    const float gs = SHARED && row_coef != nullptr ? row_coef[0] : 1.0f;
    const long long t = st->t;
    const float eta = sc[t].x;
    const long long stride = (long long)gridDim.x * UPD_THREADS * UPD_UNROLL;
    long long base = (long long)blockIdx.x * UPD_THREADS * UPD_UNROLL + threadIdx.x;
    for (; base < n4; base += stride) {
        float4 a[UPD_UNROLL], b[UPD_UNROLL], c[UPD_UNROLL];
#pragma unroll
        for (int u = 0; u < UPD_UNROLL; ++u) {
            long long i = base + (long long)u * UPD_THREADS;
            if (i < n4) {
                a[u] = ldg<KEEP>(theta + i); c[u] = ldg<KEEP>(buf + i);
                if (!NOISE) b[u] = SHARED ? g[i] : ldg<KEEP>(g + i);
            }
            if (SHARED) { b[u].x *= gs; b[u].y *= gs; b[u].z *= gs; b[u].w *= gs; }
        }
        if (CLIP) {
            const RowAt ra = rm.at((base - threadIdx.x) * 4, row_coef);
#pragma unroll
            for (int u = 0; u < UPD_UNROLL; ++u) {
                const long long i = base + (long long)u * UPD_THREADS;
                if (i < n4) scale_by_row(b[u], i * 4, ra, rm, row_coef);
            }
        }
        if (NOISE) {
#pragma unroll
            for (int u = 0; u < UPD_UNROLL; ++u) {
                long long i = base + (long long)u * UPD_THREADS;
                if (i < n4) {
                    b[u] = normal4(nd.seed, STREAM_GRAD, blockIdx.y, (uint32_t)t, (uint32_t)i);
                    b[u].x *= nd.sigma; b[u].y *= nd.sigma; b[u].z *= nd.sigma; b[u].w *= nd.sigma;
                }
            }
            if (nd.store) {
#pragma unroll
                for (int u = 0; u < UPD_UNROLL; ++u) {
                    long long i = base + (long long)u * UPD_THREADS;
                    if (i < n4) stg<KEEP>(g + i, b[u]);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < UPD_UNROLL; ++u) {
            long long i = base + (long long)u * UPD_THREADS;
            if (i < n4) {
                sgdm_elem(a[u].x, b[u].x, c[u].x, eta, mu, lambda);
                sgdm_elem(a[u].y, b[u].y, c[u].y, eta, mu, lambda);
                sgdm_elem(a[u].z, b[u].z, c[u].z, eta, mu, lambda);
                sgdm_elem(a[u].w, b[u].w, c[u].w, eta, mu, lambda);
                stg<KEEP>(theta + i, a[u]); stg<KEEP>(buf + i, c[u]);
            }
        }
    }
    if (!NOISE && !SHARED && blockIdx.x == 0 && threadIdx.x < (int)(n - n4 * 4)) {
        long long i = n4 * 4 + threadIdx.x;
        float *th = (float *)theta, *bb = (float *)buf;
        float gi = ((const float *)g)[i];
        if (CLIP) gi *= row_coef[rm.row(i)];
        float a = th[i], c = bb[i];
        sgdm_elem(a, gi, c, eta, mu, lambda);
        th[i] = a; bb[i] = c;
    }
}

// One trip per workgroup; the kernels keep their stride loop so that any grid is correct, and
// the grid is only capped where it would overflow the launch limit.
static int update_grid(long long n4)
{
    long long per_block = (long long)UPD_THREADS * UPD_UNROLL;
    long long blocks = (n4 + per_block - 1) / per_block;
    const long long cap = 0x7FFFFFFFll;
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    return (int)blocks;
}

// ---------------------------------------------------------------------------------------------
// The last local step of a round and the averaging that follows it, in one pass (Alg. 2's OPT
// line for h = H-1 and its All-Reduce line): a lane owns four consecutive parameters, walks the
// K rows (ROWS of them in flight), updates each worker's state in place, adds the updated
// parameters up with the same error-free summation and in the same order as the averaging
// kernel, and writes the mean to all K rows.  AdamW then moves 16 B read + 8 B (m, v) + 4 B
// (mean) written = 28 B per replica-parameter on such a step instead of 28 + 8; SGD 12 + 8 = 20
// instead of 20 + 8.  Acts only when this step completes the round (decided on the device, like
// the averaging); results are bit-identical to update followed by average.
// ---------------------------------------------------------------------------------------------
constexpr int SYNC_ROWS = 4;
// 256 threads: these launches are skipped on the device in all but a handful of iterations, and a
// skipped launch then has four times fewer workgroups to retire than with one-wavefront blocks
constexpr int SYNC_THREADS = 256;

template <bool ALIGNED>
__global__ __launch_bounds__(SYNC_THREADS) void update_adamw_sync_kernel(
    float *__restrict__ theta, const float *__restrict__ g, float *__restrict__ m,
    float *__restrict__ v, int K, long long P, const DevState *__restrict__ st,
    const StepScalars *__restrict__ sc, float c1, float c2, float eps, const float *__restrict__ row_coef)
{
    if (st->h + 1 != st->H) return;
    const StepScalars s = sc[st->t];
    const float fK = (float)K;
    const long long P4 = P >> 2, C4 = (P + 3) >> 2;
    const int rem = ALIGNED ? 0 : (int)(P & 3);
    const long long stride = (long long)gridDim.x * SYNC_THREADS;
    for (long long i = (long long)blockIdx.x * SYNC_THREADS + threadIdx.x; i < C4; i += stride) {
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f), cmp = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int k0 = 0; k0 < K; k0 += SYNC_ROWS) {
            float4 a[SYNC_ROWS], b[SYNC_ROWS], c[SYNC_ROWS], d[SYNC_ROWS];
#pragma unroll
            for (int u = 0; u < SYNC_ROWS; ++u)
                if (k0 + u < K) {
                    const long long o = (long long)(k0 + u) * P;
                    a[u] = ld_group(theta + o, i, P4, rem); b[u] = ld_group(g + o, i, P4, rem); c[u] = ld_group(m + o, i, P4, rem); d[u] = ld_group(v + o, i, P4, rem);
                    if (row_coef != nullptr) { const float gs = row_coef[k0 + u]; b[u].x *= gs; b[u].y *= gs; b[u].z *= gs; b[u].w *= gs; }
                }
#pragma unroll
            for (int u = 0; u < SYNC_ROWS; ++u)
                if (k0 + u < K) {
                    const long long o = (long long)(k0 + u) * P;
                    adamw_elem(a[u].x, b[u].x, c[u].x, d[u].x, s.x, s.y, s.z, c1, c2, eps);
                    adamw_elem(a[u].y, b[u].y, c[u].y, d[u].y, s.x, s.y, s.z, c1, c2, eps);
                    adamw_elem(a[u].z, b[u].z, c[u].z, d[u].z, s.x, s.y, s.z, c1, c2, eps);
                    adamw_elem(a[u].w, b[u].w, c[u].w, d[u].w, s.x, s.y, s.z, c1, c2, eps);
                    st_group(m + o, i, P4, rem, c[u]); st_group(v + o, i, P4, rem, d[u]);
                    add_comp(acc.x, cmp.x, a[u].x); add_comp(acc.y, cmp.y, a[u].y);
                    add_comp(acc.z, cmp.z, a[u].z); add_comp(acc.w, cmp.w, a[u].w);
                }
        }
        const float4 mean = make_float4((acc.x + cmp.x) / fK, (acc.y + cmp.y) / fK,
                                        (acc.z + cmp.z) / fK, (acc.w + cmp.w) / fK);
        for (int k = 0; k < K; ++k) st_group(theta + (long long)k * P, i, P4, rem, mean);
    }
}

template <bool ALIGNED>
__global__ __launch_bounds__(SYNC_THREADS) void update_sgdm_sync_kernel(
    float *__restrict__ theta, const float *__restrict__ g, float *__restrict__ buf, int K,
    long long P, const DevState *__restrict__ st, const StepScalars *__restrict__ sc, float mu,
    float lambda, const float *__restrict__ row_coef)
{
    if (st->h + 1 != st->H) return;
    const float eta = sc[st->t].x;
    const float fK = (float)K;
    const long long P4 = P >> 2, C4 = (P + 3) >> 2;
    const int rem = ALIGNED ? 0 : (int)(P & 3);
    const long long stride = (long long)gridDim.x * SYNC_THREADS;
    for (long long i = (long long)blockIdx.x * SYNC_THREADS + threadIdx.x; i < C4; i += stride) {
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f), cmp = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int k0 = 0; k0 < K; k0 += SYNC_ROWS) {
            float4 a[SYNC_ROWS], b[SYNC_ROWS], c[SYNC_ROWS];
#pragma unroll
            for (int u = 0; u < SYNC_ROWS; ++u)
                if (k0 + u < K) {
                    const long long o = (long long)(k0 + u) * P;
                    a[u] = ld_group(theta + o, i, P4, rem); b[u] = ld_group(g + o, i, P4, rem); c[u] = ld_group(buf + o, i, P4, rem);
                    if (row_coef != nullptr) { const float gs = row_coef[k0 + u]; b[u].x *= gs; b[u].y *= gs; b[u].z *= gs; b[u].w *= gs; }
                }
#pragma unroll
            for (int u = 0; u < SYNC_ROWS; ++u)
                if (k0 + u < K) {
                    const long long o = (long long)(k0 + u) * P;
                    sgdm_elem(a[u].x, b[u].x, c[u].x, eta, mu, lambda);
                    sgdm_elem(a[u].y, b[u].y, c[u].y, eta, mu, lambda);
                    sgdm_elem(a[u].z, b[u].z, c[u].z, eta, mu, lambda);
                    sgdm_elem(a[u].w, b[u].w, c[u].w, eta, mu, lambda);
                    st_group(buf + o, i, P4, rem, c[u]);
                    add_comp(acc.x, cmp.x, a[u].x); add_comp(acc.y, cmp.y, a[u].y);
                    add_comp(acc.z, cmp.z, a[u].z); add_comp(acc.w, cmp.w, a[u].w);
                }
        }
        const float4 mean = make_float4((acc.x + cmp.x) / fK, (acc.y + cmp.y) / fK,
                                        (acc.z + cmp.z) / fK, (acc.w + cmp.w) / fK);
        for (int k = 0; k < K; ++k) st_group(theta + (long long)k * P, i, P4, rem, mean);
    }
}

// Short rows that are no multiple of 4: one element per lane (v == nullptr: SGD with momentum, m is its buffer, c1 = mu, c2 = lambda)
__global__ __launch_bounds__(SYNC_THREADS) void update_sync_scalar_kernel(
    float *__restrict__ theta, const float *__restrict__ g, float *__restrict__ m,
    float *__restrict__ v, int K, long long P, const DevState *__restrict__ st,
    const StepScalars *__restrict__ sc, float c1, float c2, float eps, const float *__restrict__ row_coef)
{
    if (st->h + 1 != st->H) return;
    const StepScalars s = sc[st->t];
    const float fK = (float)K;
    const long long stride = (long long)gridDim.x * SYNC_THREADS;
    for (long long i = (long long)blockIdx.x * SYNC_THREADS + threadIdx.x; i < P; i += stride) {
        float acc = 0.f, cmp = 0.f;
        for (int k = 0; k < K; ++k) {
            const long long o = (long long)k * P + i;
            float a = theta[o], c = m[o];
            const float gk = row_coef != nullptr ? g[o] * row_coef[k] : g[o];
            if (v != nullptr) {
                float d = v[o];
                adamw_elem(a, gk, c, d, s.x, s.y, s.z, c1, c2, eps);
                v[o] = d;
            } else {
                sgdm_elem(a, gk, c, s.x, c1, c2);
            }
            m[o] = c;
            add_comp(acc, cmp, a);
        }
        const float mean = (acc + cmp) / fK;
        for (int k = 0; k < K; ++k) theta[(long long)k * P + i] = mean;
    }
}

static int sync_grid(long long items)
{
    long long blocks = (items + SYNC_THREADS - 1) / SYNC_THREADS;
    const long long cap = 0x7FFFFFFFll;
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    return (int)blocks;
}

// Rows that are no multiple of 4: one element per lane while the columns are too few to fill the chip otherwise
// (a lane's walk over the K rows is then the time, and four elements with the tests of the row's end make it longer).
// One iteration that ends a round, one element / four, us: SGD 16 x 20001 9.9 / 12.1, 64 x 100003 32 / 39, 16 x 300001
// 18.3 / 18.2, 16 x 500001 26.8 / 24.7, 32 x 700002 90 / 77; AdamW 16 x 100003 13.7 / 19.3, 32 x 300001 41 / 46,
// 64 x 500001 205 / 194, 32 x 700002 128 / 116.
static bool sync_one_per_lane(long long P) { return P <= 400000; }

hipError_t launch_update_adamw_sync(float *theta, const float *g, float *m, float *v, int K, long long P,
                                    const DevState *st, const StepScalars *sc, float c1, float c2,
                                    float eps, const float *row_coef, hipStream_t s)
{
    const int blocks = sync_grid((P + 3) / 4);
    if ((P & 3) == 0) update_adamw_sync_kernel<true><<<blocks, SYNC_THREADS, 0, s>>>(theta, g, m, v, K, P, st, sc, c1, c2, eps, row_coef);
    else if (sync_one_per_lane(P)) update_sync_scalar_kernel<<<sync_grid(P), SYNC_THREADS, 0, s>>>(theta, g, m, v, K, P, st, sc, c1, c2, eps, row_coef);
    else update_adamw_sync_kernel<false><<<blocks, SYNC_THREADS, 0, s>>>(theta, g, m, v, K, P, st, sc, c1, c2, eps, row_coef);
    return hipGetLastError();
}

hipError_t launch_update_sgdm_sync(float *theta, const float *g, float *buf, int K, long long P,
                                   const DevState *st, const StepScalars *sc, float mu, float lambda,
                                   const float *row_coef, hipStream_t s)
{
    const int blocks = sync_grid((P + 3) / 4);
    if ((P & 3) == 0) update_sgdm_sync_kernel<true><<<blocks, SYNC_THREADS, 0, s>>>(theta, g, buf, K, P, st, sc, mu, lambda, row_coef);
    else if (sync_one_per_lane(P)) update_sync_scalar_kernel<<<sync_grid(P), SYNC_THREADS, 0, s>>>(theta, g, buf, nullptr, K, P, st, sc, mu, lambda, 0.f, row_coef);
    else update_sgdm_sync_kernel<false><<<blocks, SYNC_THREADS, 0, s>>>(theta, g, buf, K, P, st, sc, mu, lambda, row_coef);
    return hipGetLastError();
}

// The clipped update of buffers that the caches hold: its norm pass and the averaging or fused synchronization behind it
// read what it read and wrote.  One iteration with rounds of four, plain / streaming accesses, us: SGD fused
// 200 x 3457 30.4 / 37.3, 64 x 20001 19.7 / 21.7, 16 x 1000000 60 / 67; AdamW fused 64 x 4311 21 / 25; separate
// 16 x 1000000 80 / 93, 8 x 300000 22.3 / 21.6.
static bool clip_keeps(int K, long long P) { return (long long)K * P <= 16000000; }

// The plain update of buffers that the caches hold together with what produces its gradient and reads its parameters.
// Behind this library's own gradient kernels (own): up to 7e6 elements; over 140 random perceptrons an iteration takes 0.98 of the
// time (0.95 to 1.00), over 33 block models 0.99.  Behind a caller's backward pass, of which nothing is known: arrays of 24 to
// 96 MB, smaller than the last-level cache with some more and larger than half of what the second-level caches hold together;
// below and above, plain accesses are up to 14 % slower as soon as several problems take turns.  us an iteration, plain /
// streaming, a gradient written before each: one problem, three in turn:
//   AdamW  1.0e6 elements 10.5 / 10.2   11.4 / 10.5        SGD  1.4e6  11.0 / 10.6   11.5 / 10.5
//          1.6e6          12.4 / 12.9   14.4 / 15.1             2.1e6  13.2 / 12.9   14.2 / 14.7
//          3.2e6          22.8 / 21.5   22.3 / 24.4             4.0e6  22.2 / 20.4   21.1 / 22.9
//          5.0e6          31.1 / 32.3   30.8 / 34.3             6.0e6  29.3 / 29.1   28.9 / 32.0
//          6.9e6          40.8 / 41.5   46.4 / 45.4 (four in turn 46.7 / 43.7)
static bool update_keeps(long long n, int arrays, bool own)
{
    return n <= 7000000 && (own || (n * arrays * 4 >= 24000000 && n * arrays * 4 <= 96000000));
}

// row_coef != nullptr: clipped update.  shared_g: all rows of g are the same (rows of whole float4 only:
// anything else reads its own row, with the same result).
hipError_t launch_update_adamw(float *theta, float *g, float *m, float *v, int K, long long P,
                               const DevState *st, const StepScalars *sc, float c1, float c2,
                               float eps, bool fused_sync, const float *row_coef, bool shared_g, bool own_gradient, hipStream_t s,
                               DevState *st_next, const SchedParams *sp)
{
    const SchedParams spv = sp ? *sp : SchedParams{};
    const int fs = fused_sync ? 1 : 0;
    const NoiseDraw none{0.f, 0, 0};
    const RowMap rm{P, K, 1.0 / (double)P};
    const long long n = (long long)K * P, n4 = n / 4;
    float4 *th4 = (float4 *)theta, *g4 = (float4 *)g, *m4 = (float4 *)m, *v4 = (float4 *)v;
    if (shared_g && (P & 3) == 0)
        update_adamw_kernel<false, false, true><<<dim3((unsigned)update_grid(P / 4), (unsigned)K), UPD_THREADS, 0, s>>>(
            th4, g4, m4, v4, P / 4, P, st, sc, c1, c2, eps, fs, row_coef, rm, none, st_next, spv);
    else if (row_coef != nullptr && clip_keeps(K, P))
        update_adamw_kernel<true, false, false, true><<<update_grid(n4), UPD_THREADS, 0, s>>>(
            th4, g4, m4, v4, n4, n, st, sc, c1, c2, eps, fs, row_coef, rm, none, st_next, spv);
    else if (row_coef != nullptr)
        update_adamw_kernel<true, false, false><<<update_grid(n4), UPD_THREADS, 0, s>>>(
            th4, g4, m4, v4, n4, n, st, sc, c1, c2, eps, fs, row_coef, rm, none, st_next, spv);
    else if (update_keeps(n, 4, own_gradient))
        update_adamw_kernel<false, false, false, true><<<update_grid(n4), UPD_THREADS, 0, s>>>(
            th4, g4, m4, v4, n4, n, st, sc, c1, c2, eps, fs, nullptr, rm, none, st_next, spv);
    else
        update_adamw_kernel<false, false, false><<<update_grid(n4), UPD_THREADS, 0, s>>>(
            th4, g4, m4, v4, n4, n, st, sc, c1, c2, eps, fs, nullptr, rm, none, st_next, spv);
    return hipGetLastError();
}

hipError_t launch_update_sgdm(float *theta, float *g, float *buf, int K, long long P,
                              const DevState *st, const StepScalars *sc, float mu, float lambda,
                              bool fused_sync, const float *row_coef, bool shared_g, bool own_gradient, hipStream_t s,
                              DevState *st_next, const SchedParams *sp)
{
    const SchedParams spv = sp ? *sp : SchedParams{};
    const int fs = fused_sync ? 1 : 0;
    const NoiseDraw none{0.f, 0, 0};
    const RowMap rm{P, K, 1.0 / (double)P};
    const long long n = (long long)K * P, n4 = n / 4;
    float4 *th4 = (float4 *)theta, *g4 = (float4 *)g, *b4 = (float4 *)buf;
    if (shared_g && (P & 3) == 0)
        update_sgdm_kernel<false, false, true><<<dim3((unsigned)update_grid(P / 4), (unsigned)K), UPD_THREADS, 0, s>>>(
            th4, g4, b4, P / 4, P, st, sc, mu, lambda, fs, row_coef, rm, none, st_next, spv);
    else if (row_coef != nullptr && clip_keeps(K, P))
        update_sgdm_kernel<true, false, false, true><<<update_grid(n4), UPD_THREADS, 0, s>>>(
            th4, g4, b4, n4, n, st, sc, mu, lambda, fs, row_coef, rm, none, st_next, spv);
    else if (row_coef != nullptr)
        update_sgdm_kernel<true, false, false><<<update_grid(n4), UPD_THREADS, 0, s>>>(
            th4, g4, b4, n4, n, st, sc, mu, lambda, fs, row_coef, rm, none, st_next, spv);
    else if (update_keeps(n, 3, own_gradient))
        update_sgdm_kernel<false, false, false, true><<<update_grid(n4), UPD_THREADS, 0, s>>>(
            th4, g4, b4, n4, n, st, sc, mu, lambda, fs, nullptr, rm, none, st_next, spv);
    else
        update_sgdm_kernel<false, false, false><<<update_grid(n4), UPD_THREADS, 0, s>>>(
            th4, g4, b4, n4, n, st, sc, mu, lambda, fs, nullptr, rm, none, st_next, spv);
    return hipGetLastError();
}

// The optimizer-only workloads' gradient g = sigma * N(0,1) drawn inside the update (P a multiple of 4)
hipError_t launch_update_adamw_noise(float *theta, float *g, float *m, float *v, int K, long long P,
                                     const DevState *st, const StepScalars *sc, float c1, float c2, float eps,
                                     float sigma, uint64_t seed, bool store_g, hipStream_t s, DevState *st_next,
                                     const SchedParams *sp)
{
    if ((P & 3) != 0) return hipErrorInvalidValue;
    const SchedParams spv = sp ? *sp : SchedParams{};
    update_adamw_kernel<false, true, false><<<dim3((unsigned)update_grid(P / 4), (unsigned)K), UPD_THREADS, 0, s>>>(
        (float4 *)theta, (float4 *)g, (float4 *)m, (float4 *)v, P / 4, P, st, sc, c1, c2, eps, 0, nullptr, RowMap{P, K, 0.0},
        NoiseDraw{sigma, seed, store_g ? 1 : 0}, st_next, spv);
    return hipGetLastError();
}

hipError_t launch_update_sgdm_noise(float *theta, float *g, float *buf, int K, long long P, const DevState *st,
                                    const StepScalars *sc, float mu, float lambda, float sigma, uint64_t seed,
                                    bool store_g, hipStream_t s, DevState *st_next, const SchedParams *sp)
{
    if ((P & 3) != 0) return hipErrorInvalidValue;
    const SchedParams spv = sp ? *sp : SchedParams{};
    update_sgdm_kernel<false, true, false><<<dim3((unsigned)update_grid(P / 4), (unsigned)K), UPD_THREADS, 0, s>>>(
        (float4 *)theta, (float4 *)g, (float4 *)buf, P / 4, P, st, sc, mu, lambda, 0, nullptr, RowMap{P, K, 0.0},
        NoiseDraw{sigma, seed, store_g ? 1 : 0}, st_next, spv);
    return hipGetLastError();
}

}  // namespace qsr
