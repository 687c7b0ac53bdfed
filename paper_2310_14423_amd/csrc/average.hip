// average.hip -- replica averaging: theta_k <- (1/K) sum_k theta_k for every worker k (the
// All-Reduce line of Alg. 2, arXiv 2310.14423), as a reduction over the K axis of the [K][P]
// buffer on one GPU.  HBM-bound: 4 B read + 4 B written per replica-parameter.
//
// Buffers that the caches hold: one or two columns per lane (avg_narrow_most).  Larger ones with K <= 64: a
// workgroup owns a tile of columns and stages it in LDS as [K][columns]: its wavefronts
// split the K rows between them (wavefront w copies rows w, w + W, ... with 128-bit loads, 1 or
// 2 KiB contiguous from each), and after a barrier every lane adds up its columns from LDS and
// the wavefront writes the mean back to the rows it loaded.  Any K: each lane owns four
// consecutive parameters and walks the K rows in registers, 16 in flight at a time.  Rows whose
// length is not a multiple of 4 take the same kernels with unaligned 128-bit accesses
// (ld_group / st_group); one or two elements per lane, as they were read before, ran 3.4-4.4 TB/s.
// What decides is the number of loads a lane has in flight: 8 wavefronts for up to 16 rows left one
// load per lane at K = 8.  Timed on MI355X, launches in a row on one buffer (us):
//                        8 x 3000001  8 x 814090  16 x 60e6  24 x 6000002  32 x 20e6  32 x 20000003  64 x 6e6
//   2 wavefronts x 1 KiB     33.9        9.1        1343          -           -           -           914 (4 x)
//   8 wavefronts x 1 KiB     41.6       14.7        1545         300 (4 x)   959        1158          586
//   2 wavefronts x 2 KiB      -           -          -           247         894        1077           -
//   rows in registers        33.1        9.7        1382         255         990        1240          578
//   as it was                41.2       10.8        1539         263         890        1262          592
// Chosen: 2 x 1 KiB up to K = 16, 2 x 2 KiB up to K = 32, 8 x 1 KiB up to K = 64 (a plain copy kernel
// reaches 5.8 TB/s on this chip; 16 x 60e6 in 1343 us is 5.7).
//
// In every variant the sum runs over k in ascending order in fp32 with an error-free
// transformation of every addition (the rounding error of each partial sum is carried in a
// second accumulator), so the mean is accurate to about one rounding whatever K is, does not
// depend on the launch shape, all K rows receive the same bits, and averaging K identical rows
// returns that row when K is a power of two.
#include "opt_elem.h"
#include "qsr_internal.h"

namespace qsr {

constexpr int AVG_THREADS = 64;
constexpr int AVG_KU = 16;

// LDS-staged tile: W wavefronts, RUN x 64 float4 columns (RUN KiB contiguous per row and wavefront)
template <int KMAX, int W, int RUN>
__device__ __forceinline__ void average_tile_body(float *__restrict__ buf, int K, long long P, float4 *avg_tile)
{
    const long long P4 = P >> 2;
    const int rem = (int)(P & 3);
    const long long C4 = P4 + (rem != 0);            // column groups, the last one possibly partial
    constexpr int TC = RUN * 64;
    constexpr int RPW = (KMAX + W - 1) / W;          // rows per wavefront
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const long long c0 = (long long)blockIdx.x * TC;
    float4 r[RPW][RUN];
#pragma unroll
    for (int j = 0; j < RPW; ++j) {
        const int k = w + j * W;
        if (k < K) {
#pragma unroll
            for (int u = 0; u < RUN; ++u) {
                const long long c = c0 + u * 64 + lane;
                if (c < C4) r[j][u] = ld_group(buf + (long long)k * P, c, P4, rem);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < RPW; ++j) {
        const int k = w + j * W;
        if (k < K) {
#pragma unroll
            for (int u = 0; u < RUN; ++u) avg_tile[k * TC + u * 64 + lane] = r[j][u];
        }
    }
    __syncthreads();
    float4 mean[RUN];
#pragma unroll
    for (int u = 0; u < RUN; ++u) {
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        float4 cmp = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int k = 0; k < K; ++k) {
            const float4 v = avg_tile[k * TC + u * 64 + lane];
            add_comp(acc.x, cmp.x, v.x); add_comp(acc.y, cmp.y, v.y);
            add_comp(acc.z, cmp.z, v.z); add_comp(acc.w, cmp.w, v.w);
        }
        const float fK = (float)K;
        mean[u] = make_float4((acc.x + cmp.x) / fK, (acc.y + cmp.y) / fK,
                              (acc.z + cmp.z) / fK, (acc.w + cmp.w) / fK);
    }
#pragma unroll
    for (int j = 0; j < RPW; ++j) {
        const int k = w + j * W;
        if (k < K) {
#pragma unroll
            for (int u = 0; u < RUN; ++u) {
                const long long c = c0 + u * 64 + lane;
                if (c < C4) st_group(buf + (long long)k * P, c, P4, rem, mean[u]);
            }
        }
    }
}

template <int KMAX, int W, int RUN>
__global__ __launch_bounds__(64 * W) void average_rows_tile_kernel(float *__restrict__ buf, int K, long long P,
                                                                   const DevState *__restrict__ st)
{
    extern __shared__ float4 avg_tile[];            // [K][RUN * 64]
    if (st != nullptr && st->h + 1 != st->H) return;        // not the step that completes a round
    average_tile_body<KMAX, W, RUN>(buf, K, P, avg_tile);
}

// any K: a lane owns four consecutive columns, AVG_KU rows in flight at a time
__global__ __launch_bounds__(AVG_THREADS) void average_rows_vec4_kernel(
    float *__restrict__ buf, int K, long long P, const DevState *__restrict__ st)
{
    if (st != nullptr && st->h + 1 != st->H) return;
    const float fK = (float)K;
    const long long P4 = P >> 2, C4 = (P + 3) >> 2;
    const int rem = (int)(P & 3);
    const long long stride = (long long)gridDim.x * AVG_THREADS;
    for (long long i = (long long)blockIdx.x * AVG_THREADS + threadIdx.x; i < C4; i += stride) {
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        float4 cmp = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int k0 = 0; k0 < K; k0 += AVG_KU) {
            float4 r[AVG_KU];
#pragma unroll
            for (int u = 0; u < AVG_KU; ++u)
                if (k0 + u < K) r[u] = ld_group(buf + (long long)(k0 + u) * P, i, P4, rem);
#pragma unroll
            for (int u = 0; u < AVG_KU; ++u)
                if (k0 + u < K) {
                    add_comp(acc.x, cmp.x, r[u].x); add_comp(acc.y, cmp.y, r[u].y);
                    add_comp(acc.z, cmp.z, r[u].z); add_comp(acc.w, cmp.w, r[u].w);
                }
        }
        float4 mean = make_float4((acc.x + cmp.x) / fK, (acc.y + cmp.y) / fK,
                                  (acc.z + cmp.z) / fK, (acc.w + cmp.w) / fK);
        for (int k = 0; k < K; ++k) st_group(buf + (long long)k * P, i, P4, rem, mean);
    }
}

// any K, buffers that the caches hold: a lane owns one column (V = 2: two, rows then being 8-byte aligned), so that
// short rows still fill the chip and no lane has a serial chain of 4 * K additions; plain loads and stores
template <int V>
__global__ __launch_bounds__(AVG_THREADS) void average_rows_kernel(float *__restrict__ buf, int K, long long P,
                                                                   const DevState *__restrict__ st)
{
    typedef float vec __attribute__((ext_vector_type(V)));
    if (st != nullptr && st->h + 1 != st->H) return;
    const long long i = ((long long)blockIdx.x * AVG_THREADS + threadIdx.x) * V;
    if (i >= P) return;
    float acc[V] = {}, cmp[V] = {};
    for (int k0 = 0; k0 < K; k0 += AVG_KU) {
        vec r[AVG_KU];
#pragma unroll
        for (int u = 0; u < AVG_KU; ++u)
            if (k0 + u < K) r[u] = *(const vec *)(buf + (long long)(k0 + u) * P + i);
#pragma unroll
        for (int u = 0; u < AVG_KU; ++u)
            if (k0 + u < K) {
#pragma unroll
                for (int e = 0; e < V; ++e) add_comp(acc[e], cmp[e], r[u][e]);
            }
    }
    vec mean;
#pragma unroll
    for (int e = 0; e < V; ++e) mean[e] = (acc[e] + cmp[e]) / (float)K;
    for (int k = 0; k < K; ++k) *(vec *)(buf + (long long)k * P + i) = mean;
}

static int avg_grid(long long items, int threads)
{
    long long blocks = (items + threads - 1) / threads;
    const long long cap = 0x7FFFFFFFll;
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    return (int)blocks;
}

template <int KMAX, int W, int RUN>
static hipError_t launch_tile(float *buf, int K, long long P, const DevState *st, hipStream_t s)
{
    const size_t lds = (size_t)K * RUN * 64 * sizeof(float4);
    static bool raised = false;                       // above the default only for more than 48 rows of 1 KiB
    if (lds > 48 * 1024 && !raised) {
        hipError_t e = hipFuncSetAttribute((const void *)average_rows_tile_kernel<KMAX, W, RUN>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, KMAX * RUN * 64 * (int)sizeof(float4));
        if (e != hipSuccess) return e;
        raised = true;
    }
    average_rows_tile_kernel<KMAX, W, RUN><<<avg_grid((P + 3) / 4, RUN * 64), 64 * W, lds, s>>>(buf, K, P, st);
    return hipGetLastError();
}

// Largest K * P that takes one or two columns per lane.  Launches in a row on one buffer, narrow against tiles (us):
//   P % 4 == 0   32 x 131072   7.0 / 12.0   24 x 1e6     29 / 40    32 x 1.5e6     57 / 86    100 x 1e6    166 / 151
//     the same on buffers taken in turn, more than the caches hold: 24 x 1e6 40 / 44, 24 x 2e6 79 / 77,
//     32 x 1.5e6 80 / 87, 8 x 3e6 39 / 36, 16 x 3e6 77 / 72, 40 x 600000 45 / 45
//   P odd        25 x 5173      6.5 / 10.0  16 x 500001 15.1 / 10.9 32 x 1500001  80 / 90     24 x 3000001 126 / 112
//                64 x 300001   32.4 / 35.3  64 x 600003  64 / 66    40 x 1500001  98 / 85
//   P % 4 == 2   25 x 3000002  112 / 118    29 x 2000002 82 / 109   64 x 1000002  91 / 100
// With fewer than 8 rows a lane has too few loads in flight, and where the launch is part of every iteration and
// mostly returns at once (in_step) many small workgroups cost more than they save: short rows only.
static long long avg_narrow_most(int K, long long P, bool in_step)
{
    if (P <= 131072) return 24000000;
    if (in_step || K < 8) return 0;
    switch (P & 3) {
    case 0: return K <= 16 || K > 32 ? 0 : K <= 24 ? 24000000 : 50000000;
    case 2: return K <= 16 ? 6000000 : K <= 24 ? 48000000 : K <= 32 ? 100000000 : K <= 64 ? 66000000 : 32000000;
    default: return K <= 16 ? 0 : K <= 32 ? 50000000 : K <= 64 ? 40000000 : 20000000;
    }
}

// st != nullptr: the launch acts only on the step that completes a round (h + 1 == H in the copy of the scheduler
// state that the iteration's kernels read)
hipError_t launch_average_rows(float *buf, int K, long long P, const DevState *st, hipStream_t s)
{
    const long long C4 = (P + 3) / 4;
    if (C4 > 0x7FFFFFFFll * 64) return hipErrorInvalidValue;
    if ((long long)K * P <= avg_narrow_most(K, P, st != nullptr)) {
        if ((P & 3) == 2)                            // rows are 8-byte aligned: two columns at a time
            average_rows_kernel<2><<<avg_grid(P / 2, AVG_THREADS), AVG_THREADS, 0, s>>>(buf, K, P, st);
        else
            average_rows_kernel<1><<<avg_grid(P, AVG_THREADS), AVG_THREADS, 0, s>>>(buf, K, P, st);
        return hipGetLastError();
    }
    if (K <= 16) return launch_tile<16, 2, 1>(buf, K, P, st, s);
    if (K <= 32) return launch_tile<32, 2, 2>(buf, K, P, st, s);
    // rows in registers against tiles, buffers in turn (us): 40 x 600000 38 / 45, 64 x 750000 76 / 82, 40 x 1.8e6 112 / 111
    const bool small = (P & 3) == 0 && (long long)K * P <= 66000000;
    if (K <= 64 && !small) return launch_tile<64, 8, 1>(buf, K, P, st, s);
    average_rows_vec4_kernel<<<avg_grid(C4, AVG_THREADS), AVG_THREADS, 0, s>>>(buf, K, P, st);
    return hipGetLastError();
}

// Alg. 2's initialisation theta_k <- theta_bar^(0): copy src [P] into each of the K rows
__global__ __launch_bounds__(256) void broadcast_rows_kernel(float *__restrict__ dst,
                                                             const float *__restrict__ src, int K,
                                                             long long P)
{
    const long long stride = (long long)gridDim.x * 256;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < P; i += stride) {
        float x = src[i];
        for (int k = 0; k < K; ++k) dst[(long long)k * P + i] = x;
    }
}

__global__ __launch_bounds__(256) void fill_zero_kernel(float *__restrict__ dst, long long n)
{
    const long long stride = (long long)gridDim.x * 256;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) dst[i] = 0.f;
}

hipError_t launch_broadcast_rows(float *dst, const float *src, int K, long long P, hipStream_t s)
{
    broadcast_rows_kernel<<<avg_grid(P, 256), 256, 0, s>>>(dst, src, K, P);
    return hipGetLastError();
}

hipError_t launch_fill_zero(float *dst, long long n, hipStream_t s)
{
    fill_zero_kernel<<<avg_grid(n, 256), 256, 0, s>>>(dst, n);
    return hipGetLastError();
}

}  // namespace qsr
