// sgemm.h -- batched single-precision GEMM, LDS-tiled, for the small fp32 model workload
// (two-layer perceptron).  C[b] = op(A[b]) * op(B[b]) with optional epilogue; one launch covers
// all K workers (blockIdx.z).  64x64 output tile, 16-deep k-slabs, four wavefronts, each a 32x32
// block on the fp32 matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands, fp32 accumulation, two
// k per instruction), global loads three slabs ahead in registers.  A long contraction is cut in
// two halves that two such groups of four wavefronts in one workgroup run side by side (KSPLIT =
// 2; the halves are added through LDS at the end).  Any M, N, Kd is accepted.  Fixed order: deterministic.
// dgemm_nn_kernel: fp32 operands (row-major, not transposed) multiplied and accumulated in double
// precision on the fp64 matrix cores (v_mfma_f64_16x16x4_f64): products of fp32 values are exact in
// double, so the result is the exact sum rounded once.  Used for the hidden layer's
// pre-activations, whose rounding errors the output layer and the softmax amplify by two to three
// orders of magnitude once the logits have grown into the hundreds.
#pragma once
#include <hip/hip_runtime.h>

#include "qsr_internal.h"
#include "tile_grid.h"

namespace qsr {

enum { EPI_NONE = 0, EPI_BIAS_RELU = 1, EPI_BIAS = 2, EPI_MASK_POS = 3 };

struct GemmArgs {
    const float *A, *B;
    float *C;
    int M, N, Kd;
    long long lda, ldb, ldc;
    long long sA, sB, sC;      // per-batch strides (elements)
    const float *bias;         // [N], per-batch stride sBias
    long long sBias;
    const float *aux;          // EPI_MASK_POS: same layout as C; C = aux > 0 ? acc : 0
    // weight gradients (A transposed, B as it is): column sums of B as a by-product, the bias gradient
    float *colsum;             // [N], per-batch stride sCol, or nullptr
    long long sCol;
    const float *part;         // with colsum, or nullptr: out[b] = scale * sum of part[b*n_part ..], fixed order
    int n_part; float *part_out; float part_scale;
};

typedef double f64x4_t __attribute__((ext_vector_type(4)));

// Every row of an operand that is read along its rows (A transposed, B as it is) starts at 16 bytes and may be read to the next
// multiple of 4 elements: one 128-bit load of each per thread and slab.  The other form (A as it is, B transposed: both read
// along k, four elements a thread) takes B's rows at any address, and reads up to three elements beyond their end.  No
// load is behind a test of its own (rows beyond the matrix are read as the last one, k beyond Kd cleared in registers): as a
// branch around each load and a wait behind it, 5 x 50 x 500 x 100 took 14.4 us.
// Workgroup (bx, by, bz) of 256 KSPLIT threads.  The LDS is the kernel's, one for whichever tiles it has, and the other
// groups' partial sums come after the slabs: a workgroup of two groups holds 24 KiB, and six would fit the 160 KiB of a
// compute unit (with a static array for the sums in each kind of tile it was 56, and two did).
struct SgemmSlabs { float A[16][96], B[16][96]; };
template <int KSPLIT> union SgemmLds {
    static_assert(KSPLIT == 2, "one group or two");
    SgemmSlabs slab[KSPLIT];
    float part[4][16][64];                               // the second group's sums
};
template <> union SgemmLds<1> { SgemmSlabs slab[1]; };
static_assert(sizeof(SgemmLds<2>) == 24 * 1024, "partial sums inside the slabs");
template <bool TA, bool TB, int EPI, int KSPLIT>
__device__ __forceinline__ void sgemm_tile(const GemmArgs &a, int bx, int by, int bz_, SgemmLds<KSPLIT> &lds)
{
    static_assert(TA != TB, "weight gradients (A transposed) and data gradients (B transposed)");
    constexpr int TM = 64, TN = 64, TK = 16;             // LDS rows of 96: rows k and k+1 of a slab 32 banks apart
    // The workgroup is KSPLIT groups of 256 threads; group grp contracts over its own run of
    // slabs with its own LDS slabs.  With one workgroup of four wavefronts per compute unit (the
    // batch is 128 rows) every slab's load -> LDS -> barrier -> MFMA chain ran unhidden; a second
    // group per SIMD fills part of those gaps (hidden layer forward, 8 x 128 x 784 x 1024: 46 -> 37 us).
    const int grp = threadIdx.x >> 8, tid = threadIdx.x & 255;
    float (*As)[96] = lds.slab[grp].A;
    float (*Bs)[96] = lds.slab[grp].B;
    const int lane = tid & 63, wm = tid >> 7, wn = (tid >> 6) & 1;   // wavefront (wm, wn) owns a 32x32 block
    const int m0 = by * TM, n0 = bx * TN;
    const long long bz = bz_;
    const float *A = a.A + bz * a.sA;
    const float *B = a.B + bz * a.sB;
    typedef float f32x16_t __attribute__((ext_vector_type(16)));
    f32x16_t acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;

    // Global loads run PF slabs ahead of the multiplication, in registers: these problems have few
    // workgroups per compute unit (the batch is 128 rows), so a slab's load latency is not hidden
    // by other wavefronts and, unprefetched, every one of the Kd/16 steps paid it in full
    // (timed on MI355X, 128 x 784 x 1024, 8 workers, with the products still on the vector ALUs:
    // 178 us per launch without, 98 us with; 46 us with the products on the matrix cores.  Six
    // slabs ahead or 32-deep slabs timed the same to slower; 64-deep slabs one ahead, for the weight
    // gradient whose contraction is 128 long: 29.5 against 27.4 us; 64 x 256 tiles with four wavefronts
    // of 64 x 64 side by side, one fragment read per instruction: 30.4 us).
    constexpr int PF = 3;
    constexpr int R = TK / 4;                       // elements of each operand per thread and slab
    float ra[PF][R], rb[PF][R];
    // A transposed, B as it is: row k of a slab and four columns.  Else: row of the tile and four k.
    const int vk = TA ? tid >> 4 : (tid & 3) * 4, vc = TA ? (tid & 15) * 4 : tid >> 2;
    const float *pa = TA ? A + min(m0 + vc, (a.M - 1) / 4 * 4) : A + (long long)min(m0 + vc, a.M - 1) * a.lda;
    const float *pb = TA ? B + min(n0 + vc, (a.N - 1) / 4 * 4) : B + (long long)min(n0 + vc, a.N - 1) * a.ldb;
    auto gload = [&](int k0, float (&xa)[R], float (&xb)[R]) {
        const int gk = k0 + vk;
        float4 va, vb;
        if (TA) {
            const int k = min(gk, a.Kd - 1);
            va = *(const float4 *)(pa + (long long)k * a.lda);
            vb = *(const float4 *)(pb + (long long)k * a.ldb);
            if (gk >= a.Kd) va = vb = make_float4(0.f, 0.f, 0.f, 0.f);
        } else {
            const int k = min(gk, (a.Kd - 1) / 4 * 4);
            va = *(const float4 *)(pa + k);
            vb = ld4u(pb + k);
            if (gk >= a.Kd) { va.x = 0.f; vb.x = 0.f; }
            if (gk + 1 >= a.Kd) { va.y = 0.f; vb.y = 0.f; }
            if (gk + 2 >= a.Kd) { va.z = 0.f; vb.z = 0.f; }
            if (gk + 3 >= a.Kd) { va.w = 0.f; vb.w = 0.f; }
        }
        xa[0] = va.x; xa[1] = va.y; xa[2] = va.z; xa[3] = va.w;
        xb[0] = vb.x; xb[1] = vb.y; xb[2] = vb.z; xb[3] = vb.w;
    };
    auto sstore = [&](const float (&xa)[R], const float (&xb)[R]) {
        if (TA) {
            *(float4 *)&As[vk][vc] = make_float4(xa[0], xa[1], xa[2], xa[3]);
            *(float4 *)&Bs[vk][vc] = make_float4(xb[0], xb[1], xb[2], xb[3]);
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) { As[vk + r][vc] = xa[r]; Bs[vk + r][vc] = xb[r]; }
        }
    };
    // every group runs the same number of slabs (the barriers are the workgroup's); slabs past
    // Kd load zeros
    const int nslab = ((a.Kd + TK - 1) / TK + KSPLIT - 1) / KSPLIT;
    const int kbase = grp * nslab * TK;
    const bool col_wg = TA && !TB && a.colsum != nullptr && by == 0;   // the workgroups of the first rows
    float cs = 0.f;
#pragma unroll
    for (int u = 0; u < PF; ++u)
        if (u < nslab) gload(kbase + u * TK, ra[u], rb[u]);
    for (int s0 = 0; s0 < nslab; s0 += PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int sl = s0 + u;                  // uniform over the workgroup
            if (sl < nslab) {
                sstore(ra[u], rb[u]);
                if (sl + PF < nslab) gload(kbase + (sl + PF) * TK, ra[u], rb[u]);
                __syncthreads();
                if (TA && !TB && col_wg && tid < 64) {
#pragma unroll
                    for (int kk = 0; kk < TK; ++kk) cs += Bs[kk][tid];
                }
                    // lane l supplies A[row l%32][k l/32] and B[k l/32][column l%32] of the instruction
#pragma unroll
                for (int kk = 0; kk < TK; kk += 2) {
                    const float av = As[kk + (lane >> 5)][wm * 32 + (lane & 31)];
                    const float bv = Bs[kk + (lane >> 5)][wn * 32 + (lane & 31)];
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv, acc, 0, 0, 0);
                }
                __syncthreads();
            }
        }
    }

    if (TA && !TB && col_wg) {
        if (tid < 64) As[0][tid] = cs;                // the slabs are done with
        __syncthreads();
        if (grp == 0 && tid < 64 && n0 + tid < a.N) {
            float v = lds.slab[0].A[0][tid];
#pragma unroll
            for (int g = 1; g < KSPLIT; ++g) v += lds.slab[g].A[0][tid];
            a.colsum[bz * a.sCol + n0 + tid] = v;
        }
        if (a.part != nullptr && bx == 0 && threadIdx.x < 64) {
            float v = 0.f;
            for (int i = lane; i < a.n_part; i += 64) v += a.part[bz * a.n_part + i];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
            if (lane == 0) a.part_out[bz] = v * a.part_scale;
        }
    }
    float *C = a.C + bz * a.sC;
    // The second group's sums go to the first, which writes the tile alone: the second's wavefronts make room for the next
    // workgroup's.  (Half of the tile written by each: 8 x 400 x 784 x 1024 74.7 against 66.9 us, 1 x 70 x 300 x 500 7.0 against 5.6.)
    if constexpr (KSPLIT == 2) {
        if (TA && !TB && col_wg) __syncthreads();     // the column sums are read
        if (grp > 0) {
#pragma unroll
            for (int i = 0; i < 16; ++i) lds.part[tid >> 6][i][lane] = acc[i];
        }
        __syncthreads();
        if (grp > 0) return;
    }
    // Accumulator element i of lane l is C[(i/4)*8 + (l/32)*4 + i%4][l%32] of the wavefront's block.  What the epilogue reads comes before
    // the first use, clamped into the matrix: behind a test and a wait of its own, each of the sixteen loads took its latency
    // (4 x 70 x 500 x 100, both products in a launch: 12.3 -> 9.6 us).
    const int gn = n0 + wn * 32 + (lane & 31);
    auto row = [&](int i) { return m0 + wm * 32 + (i >> 2) * 8 + (lane >> 5) * 4 + (i & 3); };
    float aux[16];
    if (EPI == EPI_MASK_POS) {
        const float *x = a.aux + bz * a.sC + min(gn, a.N - 1);
#pragma unroll
        for (int i = 0; i < 16; ++i) aux[i] = x[(long long)min(row(i), a.M - 1) * a.ldc];
    }
    if constexpr (KSPLIT == 2) {
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] += lds.part[tid >> 6][i][lane];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        if (row(i) >= a.M || gn >= a.N) continue;
        float v = acc[i];
        if (EPI == EPI_MASK_POS) v = aux[i] > 0.f ? v : 0.f;
        C[(long long)row(i) * a.ldc + gn] = v;
    }
}

template <bool TA, bool TB, int EPI, int KSPLIT>
__global__ __launch_bounds__(256 * KSPLIT) void sgemm_kernel(GemmArgs a)
{
    __shared__ __attribute__((aligned(16))) SgemmLds<KSPLIT> lds;
    sgemm_tile<TA, TB, EPI, KSPLIT>(a, blockIdx.x, blockIdx.y, blockIdx.z, lds);
}
// A weight gradient and a data gradient that do not depend on each other, in one launch: workgroups below `first` of `all`
// take the weight gradient's tiles, the others the data gradient's.
template <int EPI, int KSPLIT>
__global__ __launch_bounds__(256 * KSPLIT) void sgemm_pair_kernel(GemmArgs w, GemmArgs d, unsigned first, unsigned all, unsigned row,
                                                                  unsigned nxw, unsigned nxd)
{
    __shared__ __attribute__((aligned(16))) SgemmLds<KSPLIT> lds;
    unsigned b = blockIdx.y * row + blockIdx.x;        // row: the grid's x extent
    if (b >= all) return;
    if (b < first) { sgemm_tile<true, false, EPI_NONE, KSPLIT>(w, b % nxw, b / nxw, blockIdx.z, lds); return; }
    b -= first;
    sgemm_tile<false, true, EPI, KSPLIT>(d, b % nxd, b / nxd, blockIdx.z, lds);
}

// two groups per workgroup for a long contraction, and for a shorter one that would leave compute units idle
static inline bool sgemm_two(int Kd, long long workgroups) { return Kd >= 256 || (Kd >= 64 && workgroups < 256); }
static inline bool sgemm_rows_ok(const float *p, long long ld, long long s, int cols)
{
    return ((ld | s) & 3) == 0 && ld >= (cols + 3) / 4 * 4 && ((unsigned long long)p & 15) == 0;
}

// C = A^T B
inline hipError_t launch_sgemm_tn(const GemmArgs &a, int batch, hipStream_t s)
{
    if (!sgemm_rows_ok(a.A, a.lda, a.sA, a.M) || !sgemm_rows_ok(a.B, a.ldb, a.sB, a.N)) return hipErrorInvalidValue;
    dim3 grid((unsigned)((a.N + 63) / 64), (unsigned)((a.M + 63) / 64), (unsigned)batch);
    if (sgemm_two(a.Kd, (long long)grid.x * grid.y * grid.z)) sgemm_kernel<true, false, EPI_NONE, 2><<<grid, 512, 0, s>>>(a);
    else sgemm_kernel<true, false, EPI_NONE, 1><<<grid, 256, 0, s>>>(a);
    return hipGetLastError();
}

// w: C = A^T B; d: C = epilogue(A B^T), the rows of its B followed by at least three more floats
template <int EPI>
inline hipError_t launch_sgemm_pair(const GemmArgs &w, const GemmArgs &d, int batch, hipStream_t s)
{
    if (!sgemm_rows_ok(w.A, w.lda, w.sA, w.M) || !sgemm_rows_ok(w.B, w.ldb, w.sB, w.N) || !sgemm_rows_ok(d.A, d.lda, d.sA, d.Kd))
        return hipErrorInvalidValue;
    const long long nxw = (w.N + 63) / 64, nxd = (d.N + 63) / 64, first = nxw * ((w.M + 63) / 64), all = first + nxd * ((d.M + 63) / 64);
    const bool two = sgemm_two(w.Kd > d.Kd ? w.Kd : d.Kd, all * batch);
    const TileGrid t = tile_grid(all, two ? 512 : 256);
    if (t.x == 0 || all > 0x7FFFFFFFll) return hipErrorInvalidValue;
    const dim3 grid(t.x, t.y, (unsigned)batch);
    if (two) sgemm_pair_kernel<EPI, 2><<<grid, 512, 0, s>>>(w, d, (unsigned)first, (unsigned)all, t.x, (unsigned)nxw, (unsigned)nxd);
    else sgemm_pair_kernel<EPI, 1><<<grid, 256, 0, s>>>(w, d, (unsigned)first, (unsigned)all, t.x, (unsigned)nxw, (unsigned)nxd);
    return hipGetLastError();
}

// C = epilogue(A B) in double precision, A [M][Kd] and B [Kd][N] fp32 and row-major, C fp32, for contractions shorter than
// 64 (dgemm_nn_lds_kernel below takes the others): at most four groups of 16, too few for its rings.  A wavefront has a
// block of 32 x 32 (2 x 2 instructions of 16x16x4): WT = 4, a workgroup takes 64 x 64; WT = 1, 32 x 32, for problems of
// few tiles.  No LDS and no barrier: a lane's share of an instruction's operands, A[row l%16][k l/16] and
// B[k l/16][column l%16], comes straight from global memory (a float4 of A along k feeds four instructions in a
// row, the matching four rows of B one element each; the order of k inside a group of 16 is a permutation, the same
// for both operands).  Rows of A start at 16 bytes.
template <int EPI, int WT>
__global__ __launch_bounds__(64 * WT) void dgemm_nn_kernel(GemmArgs a)
{
    constexpr int PF = 3, TILE = WT == 4 ? 64 : 32;
    const int tid = threadIdx.x, lane = tid & 63, wm = tid >> 7, wn = (tid >> 6) & 1;
    const int r = lane & 15, q = lane >> 4;
    const int m0 = blockIdx.y * TILE + wm * 32, n0 = blockIdx.x * TILE + wn * 32;
    const long long bz = blockIdx.z;
    const float *A = a.A + bz * a.sA;
    const float *B = a.B + bz * a.sB;
    const int ng = (a.Kd + 15) / 16;

    // Guarded loads: the compiler turns each into a short branch with a wait behind it, so the
    // PF groups "ahead" are in fact waited for where they are loaded, and the wavefronts beside
    // hide the latency.  Timed at 8 x 128 x 784 x 1024, four groups of wavefronts sharing the contraction:
    // 46.7 us this way; 56.6 us with clamped addresses and selects, 73.3 us with unconditional clamped loads
    // and the masks applied at the point of use (62.0 us two groups ahead, without register spills).
    struct Frag { float a[2][4]; float b[2][4]; };
    auto gload = [&](int g, Frag &f) {
        const int k = g * 16 + 4 * q;
#pragma unroll
        for (int bi = 0; bi < 2; ++bi) {
            const int gm = m0 + bi * 16 + r;
            const float *ar = A + (long long)gm * a.lda + k;
            if (gm < a.M && k + 3 < a.Kd) {
                const float4 v = *(const float4 *)ar;
                f.a[bi][0] = v.x; f.a[bi][1] = v.y; f.a[bi][2] = v.z; f.a[bi][3] = v.w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) f.a[bi][j] = (gm < a.M && k + j < a.Kd) ? ar[j] : 0.f;
            }
        }
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) {
            const int gn = n0 + bj * 16 + r;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                f.b[bj][j] = (gn < a.N && k + j < a.Kd) ? B[(long long)(k + j) * a.ldb + gn] : 0.f;
        }
    };
    f64x4_t dacc[2][2];                              // 16x16 block (bi, bj) of the wavefront's 32x32
#pragma unroll
    for (int e = 0; e < 4; ++e) { dacc[0][0][e] = 0.0; dacc[0][1][e] = 0.0; dacc[1][0][e] = 0.0; dacc[1][1][e] = 0.0; }
    auto multiply = [&](const Frag &f) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double a0 = (double)f.a[0][j], a1 = (double)f.a[1][j];
            const double b0 = (double)f.b[0][j], b1 = (double)f.b[1][j];
            dacc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, dacc[0][0], 0, 0, 0);
            dacc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, dacc[0][1], 0, 0, 0);
            dacc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, dacc[1][0], 0, 0, 0);
            dacc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, dacc[1][1], 0, 0, 0);
        }
    };
    Frag fr[PF];
#pragma unroll
    for (int u = 0; u < PF; ++u)
        if (u < ng) gload(u, fr[u]);
    for (int gb = 0; gb < ng; gb += PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int g = gb + u;                   // uniform over the wavefront
            if (g < ng) {
                const Frag f = fr[u];
                if (g + PF < ng) gload(g + PF, fr[u]);
                multiply(f);
            }
        }
    }

    float *C = a.C + bz * a.sC;
    // accumulator element e of lane l is C[4*e + l/16][l%16] of its 16x16 block
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int gm = m0 + bi * 16 + 4 * e + q;
                const int gn = n0 + bj * 16 + r;
                if (gm >= a.M || gn >= a.N) continue;
                double v = dacc[bi][bj][e];
                if (EPI == EPI_BIAS_RELU || EPI == EPI_BIAS) v += (double)a.bias[bz * a.sBias + gn];
                if (EPI == EPI_BIAS_RELU) v = v > 0.0 ? v : 0.0;
                C[(long long)gm * a.ldc + gn] = (float)v;
            }
}

// The same product for longer contractions, A in 128-bit copies, B in 32- or 128-bit ones (BX4): every
// wavefront keeps a ring of NS stages of 16 k (32 rows of A, 32 columns of B, 4 KiB) in LDS of its own, copied
// there directly (global_load_lds), so there is no barrier in the main loop and no load whose arrival stalls the
// wavefront: a stage's fragments are read while the stage before is multiplied.  In LDS the 16-byte pieces of
// an A row (64 B) are permuted by (row / 4) % 4 and the 64-byte groups of two B rows by (k / 4) % 4, which makes the
// 128-bit reads of A and the 32-bit reads of B free of bank conflicts.  k beyond Kd is cleared in the
// registers, rows and columns beyond the matrix are clamped and not stored.
// The fp64 matrix instruction issues at 75-78 TFLOP/s from one wavefront per SIMD on (70-72 with the conversions);
// 8 x 128 x 784 x 1024: 46.3 us with guarded loads straight to registers, 35.9 us this way (four groups, two stages);
// 5 x 50 x 333 x 500 and 5 x 50 x 500 x 100, few tiles: 28-32 us with 64x64 tiles and two groups from registers, 13.7 us with
// 32x32 tiles and sixteen.  In an iteration these took 11.8 us where the groups' sums went through LDS in four steps to the
// first, which wrote the tile alone, and take 8.4 and 9.0 with one step and a share of the tile for each group (8 x 128 x 784 x
// 1024: 37.2 -> 35.4).
template <int EPI, int KSPLIT, int WT, int NS, bool BX4>
__global__ __launch_bounds__(64 * WT * KSPLIT) void dgemm_nn_lds_kernel(GemmArgs a)
{
    constexpr int TILE = WT == 4 ? 64 : 32, STAGE = 1024;    // floats per stage: 512 of A, 512 of B
    constexpr int CP = 2 + (BX4 ? 2 : 8);                    // copies per stage
    extern __shared__ __attribute__((aligned(1024))) float dg_ring[];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = wv / WT, w4 = wv % WT, wm = WT == 4 ? w4 >> 1 : 0, wn = WT == 4 ? w4 & 1 : 0;
    const int r = lane & 15, q = lane >> 4;
    const int m0 = blockIdx.y * TILE + wm * 32, n0 = blockIdx.x * TILE + wn * 32;
    const long long bz = blockIdx.z;
    const float *A = a.A + bz * a.sA;
    const float *B = a.B + bz * a.sB;
    float *ring = dg_ring + wv * NS * STAGE;
    const int ng = (a.Kd + 15) / 16, per = (ng + KSPLIT - 1) / KSPLIT;
    const int g0 = grp * per, nk = max(0, min(ng, g0 + per) - g0);

    // the lane's place in each 1 KiB (256 B) copy: row of A and its piece, k and column of B
    const unsigned lds_ring = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)ring;
    constexpr int CB = BX4 ? 2 : 8;
    const float *srcA[2], *srcB[CB];
    int kA[2], kB[CB];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int row = c * 16 + (lane >> 2);
        kA[c] = ((lane & 3) ^ ((row >> 2) & 3)) * 4;
        srcA[c] = A + (long long)min(m0 + row, a.M - 1) * a.lda + g0 * 16 + kA[c];
    }
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        // pair of rows pp, 64-byte group gl (in memory order: column half + 2 * row parity), column inside it
        const int pp = BX4 ? c * 4 + (lane >> 4) : c;
        const int gl = (BX4 ? (lane >> 2) & 3 : lane >> 4) ^ ((pp >> 1) & 3);
        const int col = (gl & 1) * 16 + (BX4 ? (lane & 3) * 4 : lane & 15);
        kB[c] = pp * 2 + (gl >> 1);
        srcB[c] = B + min(n0 + col, BX4 ? a.N - 4 : a.N - 1) + (long long)(g0 * 16 + kB[c]) * a.ldb;
    }
    const long long stepB = 16 * a.ldb;
    int d_slot = 0, d_k = g0 * 16;                           // slot and first k of the next stage to copy
    auto issue = [&]() {
        const unsigned dst = __builtin_amdgcn_readfirstlane(lds_ring + d_slot * (STAGE * 4));
        if (d_k + 16 > a.Kd) {                               // k is clamped, and cleared once it is in registers
#pragma unroll
            for (int c = 0; c < 2; ++c) srcA[c] -= max(d_k + kA[c] - (a.Kd - 1) / 4 * 4, 0);
#pragma unroll
            for (int c = 0; c < CB; ++c) srcB[c] -= (long long)max(d_k + kB[c] - (a.Kd - 1), 0) * a.ldb;
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            // as asm: behind the builtin, the compiler takes every LDS read for a possible reader of the copies in flight;
            // the s_nop is the wait state that a copy needs behind the compiler's write of m0
            asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "{m0}"(dst + c * 1024), "v"(srcA[c]) : "memory");
            srcA[c] += 16;
        }
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            if (BX4) asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "{m0}"(dst + 2048 + c * 1024), "v"(srcB[c]) : "memory");
            else asm volatile("s_nop 0\n\tglobal_load_lds_dword %1, off" :: "{m0}"(dst + 2048 + c * 256), "v"(srcB[c]) : "memory");
            srcB[c] += stepB;
        }
        d_slot = d_slot + 1 == NS ? 0 : d_slot + 1;
        d_k += 16;
    };
    struct Frag { float4 a[2]; float b[2][4]; } fr[2];
    auto read = [&](int slot, Frag &f) {
        const float *sa = ring + slot * STAGE, *sb = sa + 512;
#pragma unroll
        for (int bi = 0; bi < 2; ++bi) {
            const int row = bi * 16 + r;
            f.a[bi] = *(const float4 *)(sa + row * 16 + ((q ^ ((row >> 2) & 3)) * 4));
        }
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int j = 0; j < 4; ++j) {                    // k = 4 q + j of the stage
                const int k = 4 * q + j;
                f.b[bj][j] = sb[(k >> 1) * 64 + (((bj + 2 * (k & 1)) ^ q) * 16) + r];
            }
    };
    f64x4_t dacc[2][2];
#pragma unroll
    for (int e = 0; e < 4; ++e) { dacc[0][0][e] = 0.0; dacc[0][1][e] = 0.0; dacc[1][0][e] = 0.0; dacc[1][1][e] = 0.0; }
    auto multiply = [&](const Frag &f) {
        const float av[2][4] = {{f.a[0].x, f.a[0].y, f.a[0].z, f.a[0].w}, {f.a[1].x, f.a[1].y, f.a[1].z, f.a[1].w}};
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                for (int bj = 0; bj < 2; ++bj)
                    dacc[bi][bj] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)av[bi][j], (double)f.b[bj][j], dacc[bi][bj], 0, 0, 0);
    };
    auto clear_tail = [&](Frag &f, int k0) {                 // k >= Kd
        float *x[2] = {&f.a[0].x, &f.a[1].x};
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (k0 + 4 * q + j >= a.Kd) { x[0][j] = 0.f; x[1][j] = 0.f; f.b[0][j] = 0.f; f.b[1][j] = 0.f; }
    };
    // vmcnt(n): at most n of this wavefront's copies outstanding
#define DG_WAIT_VM(n) do { asm volatile("" ::: "memory"); __builtin_amdgcn_s_waitcnt(0x0f70 | ((n) & 15) | (((n) >> 4) << 14)); asm volatile("" ::: "memory"); } while (0)
#define DG_WAIT_LDS() do { asm volatile("" ::: "memory"); __builtin_amdgcn_s_waitcnt(0xc07f); asm volatile("" ::: "memory"); } while (0)
#pragma unroll
    for (int s = 0; s < NS; ++s)
        if (s < nk) issue();
    if (nk > 0) {
        if (nk >= NS) DG_WAIT_VM(CP * (NS - 1)); else DG_WAIT_VM(0);
        read(0, fr[0]);
        if (nk == 1) clear_tail(fr[0], g0 * 16);
        int slot = 0;
        for (int kt = 0; kt < nk; kt += 2) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int k = kt + u;
                if (k >= nk) break;
                DG_WAIT_LDS();                               // the fragments of stage k are in: its slot is free
                if (k + NS < nk) issue();
                slot = slot + 1 == NS ? 0 : slot + 1;
                if (k + 1 < nk) {
                    if (k + NS < nk) DG_WAIT_VM(CP * (NS - 1));      // stage k + 1 has landed
                    else DG_WAIT_VM(0);
                    read(slot, fr[u ^ 1]);
                    if (k + 2 == nk) clear_tail(fr[u ^ 1], (g0 + k + 1) * 16);
                }
                multiply(fr[u]);
            }
        }
    }
    float *C = a.C + bz * a.sC;
    // The groups' partial sums, each wavefront's in the ring it is done with; each adds up, pairwise in a fixed order, and
    // writes its share of the tile
    double *const dpart = (double *)dg_ring;
    constexpr int RING = NS * STAGE / 2, EACH = 16 / KSPLIT; // doubles of a ring, accumulator elements of a wavefront
    static_assert(RING >= 16 * 64 && 16 % KSPLIT == 0, "a wavefront's accumulators in its ring");
    if constexpr (KSPLIT > 1) {
#pragma unroll
        for (int i = 0; i < 16; ++i) dpart[wv * RING + i * 64 + lane] = dacc[i >> 3][(i >> 2) & 1][i & 3];
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < EACH; ++u) {
        const int i = grp * EACH + u;
        // accumulator element e of lane l is C[4*e + l/16][l%16] of its 16x16 block
        const int gm = m0 + (i >> 3) * 16 + 4 * (i & 3) + q;
        const int gn = n0 + ((i >> 2) & 1) * 16 + r;
        double v;
        if constexpr (KSPLIT > 1) {
            double part[KSPLIT];
#pragma unroll
            for (int g = 0; g < KSPLIT; ++g) part[g] = dpart[(g * WT + w4) * RING + i * 64 + lane];
#pragma unroll
            for (int stride = KSPLIT / 2; stride >= 1; stride >>= 1)
#pragma unroll
                for (int g = 0; g < stride; ++g) part[g] += part[g + stride];
            v = part[0];
        } else v = dacc[u >> 3][(u >> 2) & 1][u & 3];
        if (gm >= a.M || gn >= a.N) continue;
        if (EPI == EPI_BIAS_RELU || EPI == EPI_BIAS) v += (double)a.bias[bz * a.sBias + gn];
        if (EPI == EPI_BIAS_RELU) v = v > 0.0 ? v : 0.0;
        C[(long long)gm * a.ldc + gn] = (float)v;
    }
#undef DG_WAIT_VM
#undef DG_WAIT_LDS
}

template <int EPI, int KSPLIT, int WT, int NS>
inline hipError_t launch_dgemm_lds(const GemmArgs &a, int batch, bool bx4, hipStream_t s)
{
    constexpr int TILE = WT == 4 ? 64 : 32;
    constexpr size_t smem = (size_t)WT * KSPLIT * NS * 4096;
    static_assert(smem <= 160 * 1024, "rings");
    static bool raised = false;               // per instantiation; contexts are not thread-safe
    if (smem > 64 * 1024 && !raised) {
        hipError_t e = hipFuncSetAttribute((const void *)dgemm_nn_lds_kernel<EPI, KSPLIT, WT, NS, false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e == hipSuccess) e = hipFuncSetAttribute((const void *)dgemm_nn_lds_kernel<EPI, KSPLIT, WT, NS, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        raised = true;
    }
    dim3 grid((unsigned)((a.N + TILE - 1) / TILE), (unsigned)((a.M + TILE - 1) / TILE), (unsigned)batch);
    if (bx4) dgemm_nn_lds_kernel<EPI, KSPLIT, WT, NS, true><<<grid, 64 * WT * KSPLIT, smem, s>>>(a);
    else dgemm_nn_lds_kernel<EPI, KSPLIT, WT, NS, false><<<grid, 64 * WT * KSPLIT, smem, s>>>(a);
    return hipGetLastError();
}

template <int EPI>
inline hipError_t launch_dgemm_nn(const GemmArgs &a, int batch, hipStream_t s)
{
    dim3 grid((unsigned)((a.N + 63) / 64), (unsigned)((a.M + 63) / 64), (unsigned)batch);
    const bool few = (long long)grid.x * grid.y * grid.z < 200;
    // 128-bit copies of A: 16-byte rows in every batch entry, readable to a multiple of 4; of B as well, or 32-bit ones
    if (!sgemm_rows_ok(a.A, a.lda, a.sA, a.Kd)) return hipErrorInvalidValue;
    const bool bx4 = ((a.ldb | a.sB | a.N) & 3) == 0 && (((unsigned long long)a.B) & 15) == 0;
    if (a.Kd < 64) {
        const dim3 small((unsigned)((a.N + 31) / 32), (unsigned)((a.M + 31) / 32), (unsigned)batch);
        if (few) dgemm_nn_kernel<EPI, 1><<<small, 64, 0, s>>>(a);       // 64x64 tiles would leave the chip idle
        else dgemm_nn_kernel<EPI, 4><<<grid, 256, 0, s>>>(a);
        return hipGetLastError();
    }
    // Groups per workgroup: several only where the tiles leave compute units idle (us, one / two / four groups):
    // 256 tiles, contraction 784 38 / 34.6 / 33.8, 256 15.9 / 15.3 / 15.7;  752 tiles 784 89 / 88 / 98, 128 21 / 23 / 30;
    // 5292 tiles 784 559 / 569 / 666, 112 95 / 114 / 181 (guarded loads 125)
    if (few) return a.Kd >= 256 ? launch_dgemm_lds<EPI, 16, 1, 2>(a, batch, bx4, s) : launch_dgemm_lds<EPI, 4, 1, 4>(a, batch, bx4, s);
    if ((long long)grid.x * grid.y * grid.z >= 512) return launch_dgemm_lds<EPI, 1, 4, 2>(a, batch, bx4, s);
    return a.Kd < 512 ? launch_dgemm_lds<EPI, 2, 4, 2>(a, batch, bx4, s) : launch_dgemm_lds<EPI, 4, 4, 2>(a, batch, bx4, s);
}

}  // namespace qsr
