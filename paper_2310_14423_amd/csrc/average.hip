// average.hip -- replica averaging: theta_k <- (1/K) sum_k theta_k for every worker k (the
// All-Reduce line of Alg. 2, arXiv 2310.14423), as a reduction over the K axis of the [K][P]
// buffer on one GPU.  HBM-bound: 4 B read + 4 B written per replica-parameter.
//
// Three kernels, chosen by size and alignment (launch_average_rows, where the timings stand):
//  - a tile of columns staged in LDS as [K][columns], K <= 64: the workgroup's wavefronts split the K rows between
//    them (wavefront w copies rows w, w + W, ... with 128-bit loads, 1 or 2 KiB contiguous from each), and after a
//    barrier every lane adds up its columns from LDS and the wavefront writes the mean back to the rows it loaded;
//  - rows in registers, any K: each lane owns four consecutive parameters and walks the K rows, 16 in flight;
//  - one or two columns per lane, any K.
// Rows whose length is not a multiple of 4 take the first two with unaligned 128-bit accesses (ld_group / st_group).
// A plain copy kernel reaches 5.8 TB/s on this chip; 16 x 60e6 in 1325 us is 5.8.
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

// Which part of the columns a workgroup takes.  Rows of other lengths than multiples of 4 start anywhere in a 128-byte line, so
// that neighbouring parts share a line of every row; workgroups go to the 8 XCDs round-robin by their id, and in order each of
// those lines would be written half by one XCD's L2 and half by another's.  Where rows are not aligned each XCD takes 64
// parts in a row instead (the rest of the grid goes in order).  us, in order / 16 / 64 / 256 parts: 8 x 3000001 33.3 / 30.4 / 31.0 /
// 30.5 (buffers in turn 36.1 / 32.4 / 32.4 / 32.7), 8 x 814090 10.8 / 9.9 / 9.6 / 10.5, 17 x 20000001 583 / 532 / 530 / 530,
// 12 x 16666665 327 / 310 / 307 / 309, 24 x 6000002 240.6 / 235.0 / 235.6 / 237, 48 x 4166663 370 / 347 / 344 / 338, 64 x 2000001 228 /
// 217 / 213 / 219, 100 x 2000002 395 / 380 / 375 / 378.  Aligned rows share nothing and stay in order: 16 x 60000000 1352 / 1462 /
// 1422 / 1459, 32 x 9000004 469 / 482 / 490 / 495.
__device__ __forceinline__ long long column_part(long long P)
{
    constexpr unsigned EACH = 64, TURN = 8 * EACH;
    const unsigned b = blockIdx.x, r = b % TURN, first = b - r;
    return (P & 3) != 0 && first + TURN <= gridDim.x ? first + r % 8 * EACH + r / 8 : b;
}

// LDS-staged tile: W wavefronts, RUN x 64 float4 columns (RUN KiB contiguous per row and wavefront).
// ALIGNED (here and below): P is known to be a multiple of 4.  With the test of P's remainder around every access
// 32 x 2250000 took 127 us for 120, 32 x 3125000 176 for 169.
template <int KMAX, int W, int RUN, bool ALIGNED>
__device__ __forceinline__ void average_tile_body(float *__restrict__ buf, int K, long long P, float4 *avg_tile)
{
    const long long P4 = P >> 2;
    const int rem = ALIGNED ? 0 : (int)(P & 3);
    const long long C4 = P4 + (rem != 0);            // column groups, the last one possibly partial
    constexpr int TC = RUN * 64;
    constexpr int RPW = (KMAX + W - 1) / W;          // rows per wavefront
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const long long c0 = (ALIGNED ? (long long)blockIdx.x : column_part(P)) * TC;
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

template <int KMAX, int W, int RUN, bool ALIGNED>
__global__ __launch_bounds__(64 * W) void average_rows_tile_kernel(float *__restrict__ buf, int K, long long P,
                                                                   const DevState *__restrict__ st)
{
    extern __shared__ float4 avg_tile[];            // [K][RUN * 64]
    if (st != nullptr && st->h + 1 != st->H) return;        // not the step that completes a round
    average_tile_body<KMAX, W, RUN, ALIGNED>(buf, K, P, avg_tile);
}

// any K: a lane owns four consecutive columns, AVG_KU rows in flight at a time
template <bool ALIGNED>
__global__ __launch_bounds__(AVG_THREADS) void average_rows_vec4_kernel(
    float *__restrict__ buf, int K, long long P, const DevState *__restrict__ st)
{
    if (st != nullptr && st->h + 1 != st->H) return;
    const float fK = (float)K;
    const long long P4 = P >> 2, C4 = (P + 3) >> 2;
    const int rem = ALIGNED ? 0 : (int)(P & 3);
    const long long stride = (long long)gridDim.x * AVG_THREADS;
    for (long long i = (ALIGNED ? (long long)blockIdx.x : column_part(P)) * AVG_THREADS + threadIdx.x; i < C4; i += stride) {
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

// any K: a lane owns one column (V = 2: two, rows then being 8-byte aligned), so that short rows still fill the chip
// and no lane has a serial chain of 4 * K additions; plain loads and stores, which find what the caches hold and leave
// the result there for the update behind
template <int V>
__global__ __launch_bounds__(AVG_THREADS) void average_rows_kernel(float *__restrict__ buf, int K, long long P,
                                                                   const DevState *__restrict__ st)
{
    typedef float vec __attribute__((ext_vector_type(V)));
    if (st != nullptr && st->h + 1 != st->H) return;
    const long long i = (column_part(P) * AVG_THREADS + threadIdx.x) * V;
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

template <int KMAX, int W, int RUN, bool ALIGNED>
static hipError_t launch_tile(float *buf, int K, long long P, const DevState *st, hipStream_t s)
{
    const size_t lds = (size_t)K * RUN * 64 * sizeof(float4);
    static bool raised = false;                       // above the default only for more than 48 rows of 1 KiB
    if (lds > 48 * 1024 && !raised) {
        hipError_t e = hipFuncSetAttribute((const void *)average_rows_tile_kernel<KMAX, W, RUN, ALIGNED>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, KMAX * RUN * 64 * (int)sizeof(float4));
        if (e != hipSuccess) return e;
        raised = true;
    }
    average_rows_tile_kernel<KMAX, W, RUN, ALIGNED><<<avg_grid((P + 3) / 4, RUN * 64), 64 * W, lds, s>>>(buf, K, P, st);
    return hipGetLastError();
}

// V columns per lane
template <int V>
static hipError_t launch_narrow(float *buf, int K, long long P, const DevState *st, hipStream_t s)
{
    average_rows_kernel<V><<<avg_grid(P / V, AVG_THREADS), AVG_THREADS, 0, s>>>(buf, K, P, st);
    return hipGetLastError();
}
template <bool ALIGNED>
static hipError_t launch_vec4(float *buf, int K, long long P, const DevState *st, hipStream_t s)
{
    average_rows_vec4_kernel<ALIGNED><<<avg_grid((P + 3) / 4, AVG_THREADS), AVG_THREADS, 0, s>>>(buf, K, P, st);
    return hipGetLastError();
}

// Which kernel, by alignment, K and K * P, from 4000 timed sizes (K to 120, K * P from 1e5 to 6e8, every P mod 4) on one
// buffer again and again ("hot") and on buffers in turn that together exceed the caches ("cold"), and from whole
// iterations.  One size on either side of each line, hot / cold in us; two, one: columns per lane; tile: wavefronts x KiB.
//   short rows: one column keeps the chip busy          32 x 131072   one 6.5 / 9.4    four in registers 7.3 / 8.9    tile 12 / 11
//   P a multiple of 4, the buffer in the caches (K * P <= 56e6): two columns
//                                                        24 x 1e6     two 29.5 / 42     tile 2 x 2 40 / 43
//                                                        16 x 3e6     two 56 / 77       tile 2 x 1 73 / 72
//                                                        24 x 2e6     two 56 / 79       tile 2 x 2 74 / 76
//                             beyond                     24 x 3e6     two 88 / 116      tile 2 x 2 109 / 109
//                             K <= 16, below 24e6        12 x 1e6     two 15.6 / 21.4   tile 2 x 1 17.2 / 19.6
//                             K <= 8                      8 x 3e6     two 29 / 38       tile 2 x 1 34 / 35
//     K * P > 56e6, K of 9 to 32                         12 x 16666668 tile 2 x 2 344 / 335  tile 2 x 1 377 / 373  tile 8 x 1 349 / 346
//     K of 9 to 16 beyond 5e8                            16 x 60e6    alone: tile 2 x 1 1325 / 1343, 2 x 2 1349 / 1365;
//                                                                     a whole AdamW iteration: 5990 with 2 x 2, 5880 with 8 x 1
//     K > 32                                             64 x 750000  in registers 74 / 76  tile 8 x 1 80 / 82   two 61 / 92
//                                                        48 x 4166664 in registers 377 / 382  tile 8 x 1 408 / 402
//   other P (in the order of column_part), K <= 16       16 x 1500001 tile 2 x 1 31 / 42   one 30 / 41   in registers 30 / 41;  16 x 6000002
//                                                        tile 2 x 1 140 / 150  one 151 / 159  in registers 144 / 152
//                                                        12 x 250002  two 6.6 / 7.7        tile 2 x 1 6.7 / 8.3 (fewer than 8 rows: too few
//                                                                     loads in flight a lane, 10 % behind in hot buffers)
//     K > 16, few columns                                24 x 200002  two 7.5 / 10.2       in registers 9.2 / 12.2
//                                                        40 x 250002  two 13.4 / 20.0      in registers 16.1 / 20.1
//     K > 16                                             24 x 500001  in registers 15 / 22  one 16 / 23  tile 2 x 2 26 / 31
//     K of 17 to 32 beyond 100e6                         24 x 6000002 tile 2 x 2 235 / 234  in registers 240 / 237  tile 8 x 1 229 / 228
//                                   below                24 x 3500002 tile 2 x 2 129 / 142  in registers 116 / 138
//     K of 33 to 64 beyond 72e6                          64 x 2000001 tile 8 x 1 214 / 215  in registers 237 / 242
//                                   below                48 x 1200001 tile 8 x 1 82 / 106   in registers 68 / 103
//     K > 64                                             100 x 2000002 in registers 379 / 381  two 402 / 405
//                                   odd beyond 150e6     72 x 2100001 one 267 / 267  in registers 277 / 278
// Of 27 unaligned sizes with every kernel the rule's is within 5 % of the fastest, but 28 x 4000002: tile 2 x 2 201 / 201, tile 8 x 1
// 183 / 183, in registers 184 / 185.
// st != nullptr: the launch acts only on the step that completes a round (h + 1 == H in the copy of the scheduler
// state that the iteration's kernels read)
hipError_t launch_average_rows(float *buf, int K, long long P, const DevState *st, hipStream_t s)
{
    if ((P + 3) / 4 > 0x7FFFFFFFll * 64) return hipErrorInvalidValue;
    const long long n = (long long)K * P;
    const bool even = (P & 3) == 2;                  // rows are 8-byte aligned: two columns at a time
    if (P <= 131072 && n <= 24000000)
        return even ? launch_narrow<2>(buf, K, P, st, s) : launch_narrow<1>(buf, K, P, st, s);
    if ((P & 3) == 0) {
        if (K > 32) return n <= 24000000 ? launch_vec4<true>(buf, K, P, st, s) : launch_vec4<false>(buf, K, P, st, s);
        if (K > 8 && (K > 16 || n >= 24000000)) {
            if (n <= 56000000) return launch_narrow<2>(buf, K, P, st, s);
            if (K > 16 || n <= 500000000) return launch_tile<32, 2, 2, true>(buf, K, P, st, s);
            if (st != nullptr) return launch_tile<16, 8, 1, true>(buf, K, P, st, s);
        }
        return launch_tile<16, 2, 1, false>(buf, K, P, st, s);   // (the test of the remainder costs nothing here: 1331 / 1366)
    }
    if (K <= 16) {
        if (even && K >= 8 && n <= 6000000) return launch_narrow<2>(buf, K, P, st, s);
        return launch_tile<16, 2, 1, false>(buf, K, P, st, s);
    }
    if (n <= 6000000 || (n <= 24000000 && (P <= 200000 || (even && K > 32))))
        return even ? launch_narrow<2>(buf, K, P, st, s) : launch_narrow<1>(buf, K, P, st, s);
    if (K <= 32 && n > 100000000) return launch_tile<32, 2, 2, false>(buf, K, P, st, s);
    if (K > 32 && K <= 64 && n > 72000000) return launch_tile<64, 8, 1, false>(buf, K, P, st, s);
    if (K > 64 && !even && n > 150000000) return launch_narrow<1>(buf, K, P, st, s);
    return launch_vec4<false>(buf, K, P, st, s);
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
