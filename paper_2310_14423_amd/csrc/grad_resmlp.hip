// grad_resmlp.hip -- local gradient (Eq. (1) of arXiv 2310.14423) of the residual-MLP workload
// for all K workers, batched over the workers in every launch.  The workload has the MLP
// sub-block shapes of the paper's ViT-B (Sec. 4; width d, hidden width dh, L blocks):
//
//   x_0 = tokens [M][d] ~ N(0,1);  y = x_0 W_T / sqrt(d)
//   u_l = LayerNorm(x_l; gamma_l, beta_l);  h_l = u_l W1_l + b1_l;  a_l = gelu_erf(h_l)
//   x_l+1 = x_l + a_l W2_l + b2_l;  loss = 1/(2 M d) sum (x_L - y)^2
//
// The six GEMMs per block (2 forward, 2 data-gradient, 2 weight-gradient) run on the bf16
// matrix cores with fp32 accumulation (gemm_bf16.h); the residual stream, LayerNorm statistics,
// loss and all gradients stay fp32.  The forward and data-gradient GEMMs are brought to the
// K-contiguous "NT" form by keeping bf16 copies of the weights in both orientations; the
// weight-gradient GEMMs reduce over the token axis and read the same bf16 activations as they are
// ("TN" form, LDS transpose reads), so no transposed activation copies exist.  The bf16 weights
// and the bf16 activations that GEMM epilogues and the LayerNorm forward pass produce (LayerNorm
// output, GELU output and derivative, the gradient of the hidden layer) are stored in 32-row x
// 32-column blocks (gemm_bf16.h), written that way by their producers, so that the slab copies of
// the GEMMs read consecutive memory.  The bf16 copy of the residual gradient stays row-major (the
// LayerNorm backward pass that writes it lost more on 64-byte store pieces than its two GEMMs
// gained), and so does what the attention core reads and writes.
// Per-block parameter packing: gamma[d], beta[d], W1[d][dh], b1[dh], W2[dh][d], b2[d].
//
// With n_heads > 0 each block first runs the attention half of a ViT encoder block,
//   u = LayerNorm(x_l; gamma_a, beta_a);  q|k|v = u Wqkv + bqkv;
//   o = softmax(q k^T / sqrt(64)) v per head and sequence;  x_l' = x_l + o Wo + bo,
// its parameters gamma_a[d], beta_a[d], Wqkv[d][3d], bqkv[3d], Wo[d][d], bo[d] packed in front of
// the block's six arrays above: four more GEMMs forward/data-gradient and two weight-gradient
// GEMMs of the same kinds, and the attention core of attention.h.
#include "attention.h"
#include "gemm_bf16.h"
#include "gemm_tn.h"
#include "ln_rows.h"
#include "philox.h"
#include "qsr_internal.h"
#include "wgrad_plan.h"

namespace qsr {

static inline size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

constexpr float LN_EPS = 1e-5f;

struct ResWs {
    // per-replica strides are the element counts of one replica's array
    // "sub" counts residual sub-blocks: L without attention, 2L with (attention, MLP, attention, ...)
    float *X;      long long sX;       // [sub+1][M][d]
    float *MU, *RSTD; long long sStat; // [sub][M]
    bf16_t *H;     long long sH;       // [L][M][dh]  gelu'(pre-activation)
    bf16_t *U;     long long sU;       // [sub][M][d] LayerNorm output
    bf16_t *A;     long long sA;       // [L][M][dh]  GELU output
    float *DX;     long long sDX;      // [M][d]
    bf16_t *DXb;   long long sDXb;     // [M][d]
    bf16_t *DH;    long long sDH;      // [M][dh]
    float *DU;     long long sDU;      // [M][d]; holds the tokens in bf16 (blocked) until the loss is known
    bf16_t *W1b, *W1Tb, *W2b, *W2Tb; long long sW; // [L][blocked d x dh or dh x d] each
    long long mdB, mdhB;               // elements of one blocked [M][d] / [M][dh] activation
    long long wB[2];                   // elements of one blocked [d][dh] / [dh][d] weight
    bf16_t *WTt;                       // [d][d], shared: teacher map transposed
    float *PART;   long long sPART;    // [2][rows of partial sums][d] partial dgamma, dbeta
    float *LPART;  long long sLPART;   // loss partials
    bf16_t *ZERO;                      // 256 bytes of zeros (stand-in rows of ragged GEMM slabs)
    float *SPLITK; long long split_floats;   // partial weight gradients of a launch, [K][ranges][its part of a worker's gradient]
    // All weight gradients in one launch: a copy of DXb for each sub-block (sDXb covers them), of DH and of DQKV for each block
    bool defer;
    // attention sub-blocks only
    bf16_t *QKV;   long long sQKV;     // [L][M][3d]
    bf16_t *O;     long long sO;       // [L][M][d]   attention output before the projection
    float *LSE;    long long sLSE;     // [L][heads][M]
    bf16_t *DO;    long long sDO;      // [M][d]
    bf16_t *DQKV;  long long sDQKV;    // [M][3d]
    bf16_t *Wqb, *WqTb; long long sWq; // [L][d*3d] each
    bf16_t *Wob, *WoTb; long long sWo; // [L][d*d] each
};

static ResWs carve(const ModelDims &dm, void *ws, size_t *total)
{
    const long long K = dm.K, M = dm.B, d = dm.d_in, dh = dm.d_hidden, L = dm.n_blocks;
    const long long heads = dm.n_heads, sub = heads > 0 ? 2 * L : L;
    char *p = (char *)ws;
    size_t off = 0;
    ResWs w;
    // Per-worker arrays are laid out [K][stride].  The natural strides of the benchmark size are
    // exact multiples of 512 KiB, which puts the 8 workers' arrays in phase with every power-of-two
    // interleaving of the memory channels: XCDs that sweep one worker each, at the same relative
    // offsets and the same time, would all sit on the same channels.  8448 extra bytes per worker
    // take them out of phase.
    auto padded = [&](long long n, size_t elt) { return (long long)(up256((size_t)n * elt) + 8448) / (long long)elt; };
    auto take = [&](long long per_replica, size_t elt, long long copies) {
        void *r = p + off;
        off += up256((size_t)per_replica * elt * (size_t)copies);
        return r;
    };
    // blocked arrays: token rows padded to a multiple of 256, weight rows likewise
    w.mdB = blk_elems(M, d); w.mdhB = blk_elems(M, dh);
    w.wB[0] = blk_elems(d, dh); w.wB[1] = blk_elems(dh, d);
    const long long wmax = w.wB[0] > w.wB[1] ? w.wB[0] : w.wB[1];
    w.sX = padded((sub + 1) * M * d, 4); w.X = (float *)take(w.sX, 4, K);
    w.sStat = padded(sub * M, 4);        w.MU = (float *)take(w.sStat, 4, K); w.RSTD = (float *)take(w.sStat, 4, K);
    w.sH = padded(L * w.mdhB, 2);        w.H = (bf16_t *)take(w.sH, 2, K);
    w.sU = padded(sub * w.mdB, 2);       w.U = (bf16_t *)take(w.sU, 2, K);
    w.sA = padded(L * w.mdhB, 2);        w.A = (bf16_t *)take(w.sA, 2, K);
    w.sDX = padded(M * d, 4);            w.DX = (float *)take(w.sDX, 4, K);
    w.defer = wgrad_defer(K, M, d, dh, heads > 0, L);
    w.sDXb = padded((w.defer ? sub : 1) * M * d, 2); w.DXb = (bf16_t *)take(w.sDXb, 2, K);
    w.sDH = padded((w.defer ? L : 1) * w.mdhB, 2); w.DH = (bf16_t *)take(w.sDH, 2, K);
    w.sDU = padded(w.mdB > M * d ? w.mdB : M * d, 4); w.DU = (float *)take(w.sDU, 4, K);
    w.sW = padded(L * wmax, 2);
    w.W1b = (bf16_t *)take(w.sW, 2, K);  w.W1Tb = (bf16_t *)take(w.sW, 2, K);
    w.W2b = (bf16_t *)take(w.sW, 2, K);  w.W2Tb = (bf16_t *)take(w.sW, 2, K);
    w.WTt = (bf16_t *)take(blk_elems(d, d), 2, 1);
    const long long part_rows = ln_bwd_plan(K, M, d).waves;
    w.sPART = padded((w.defer ? sub : 1) * 2 * part_rows * d, 4); w.PART = (float *)take(w.sPART, 4, K);
    w.sLPART = padded(4 * ((M + 63) / 64) * (d / 64) + 8, 4);   // a wavefront of a tile each: most for 64 x 64
     w.LPART = (float *)take(w.sLPART, 4, K);
    w.ZERO = (bf16_t *)take(128, 2, 1);
    w.split_floats = wgrad_split_floats(K, M, d, dh, heads > 0, L, w.defer);
    w.SPLITK = (float *)take(w.split_floats, 4, 1);
    w.QKV = w.O = w.DO = w.DQKV = w.Wqb = w.WqTb = w.Wob = w.WoTb = nullptr; w.LSE = nullptr;
    w.sQKV = w.sO = w.sLSE = w.sDO = w.sDQKV = w.sWq = w.sWo = 0;
    if (heads > 0) {
        w.sQKV = padded(L * M * 3 * d, 2);   w.QKV = (bf16_t *)take(w.sQKV, 2, K);
        w.sO = padded(L * M * d, 2);         w.O = (bf16_t *)take(w.sO, 2, K);
        w.sLSE = padded(L * heads * M, 4);   w.LSE = (float *)take(w.sLSE, 4, K);
        w.sDO = padded(M * d, 2);            w.DO = (bf16_t *)take(w.sDO, 2, K);
        w.sDQKV = padded((w.defer ? L : 1) * M * 3 * d, 2); w.DQKV = (bf16_t *)take(w.sDQKV, 2, K);
        const long long wq = blk_elems(3 * d, d) > blk_elems(d, 3 * d) ? blk_elems(3 * d, d) : blk_elems(d, 3 * d);
        w.sWq = padded(L * wq, 2);                           // blocked [d][3d] and [3d][d]
        w.Wqb = (bf16_t *)take(w.sWq, 2, K); w.WqTb = (bf16_t *)take(w.sWq, 2, K);
        w.sWo = padded(L * blk_elems(d, d), 2);
        w.Wob = (bf16_t *)take(w.sWo, 2, K); w.WoTb = (bf16_t *)take(w.sWo, 2, K);
    }
    if (total) *total = off;
    return w;
}

size_t resmlp_workspace_bytes(const ModelDims &d)
{
    size_t total = 0;
    carve(d, nullptr, &total);
    return total;
}

// ---------------------------------------------------------------------------------------------
// layout / conversion kernels
// ---------------------------------------------------------------------------------------------

// bf16 copies of fp32 matrices [R][C] (R and C multiples of 64, rows contiguous) in the blocked layout of
// gemm_bf16.h, as they are (optional) and transposed: all weights of all blocks and workers, and the
// teacher map, in one launch.  HBM-bound (4 B read, 4 written per weight): a workgroup takes a 64 x 64 tile, 128-bit
// loads all in flight at once, 128-bit stores both ways, the transposed ones through LDS.  Timed on MI355X:
// 12 blocks 768/3072 with attention x 8 workers 1047 us (5.2 TB/s), 2 x 192/768 with attention x 2 workers 5.3 us (one launch
// per kind of matrix, one element per lane: 1430 and 58 us).
struct CvtMat {
    const float *in; long long s_in, l_in;           // worker and block strides
    bf16_t *out, *outT; long long s_out;             // worker stride of both; the blocks' copies are R*C padded apart
    int R, C, n_l, n_z;                              // blocks and workers
    int first;                                       // first workgroup
};
struct CvtList { CvtMat m[5]; int n; };

__global__ __launch_bounds__(256) void cvt_transpose_kernel(CvtList list)
{
    __shared__ bf16_t tile[64][66];
    int e = 0;
    while (e + 1 < list.n && (int)blockIdx.x >= list.m[e + 1].first) ++e;
    const CvtMat &q = list.m[e];
    const int R = q.R, C = q.C, tx = C >> 6, per = tx * (R >> 6);
    int b = blockIdx.x - q.first;
    const int zl = b / per;
    b -= zl * per;
    const int z = zl / q.n_l, l = zl - z * q.n_l;
    const int r0 = (b / tx) * 64, c0 = (b % tx) * 64;
    const int t = threadIdx.x, row = t >> 3, c = (t & 7) * 8;
    const float *src = q.in + (long long)z * q.s_in + (long long)l * q.l_in + (long long)(r0 + row) * C + c0 + c;
    float4 v[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int u = 0; u < 2; ++u) v[i][u] = *(const float4 *)(src + (long long)i * 32 * C + u * 4);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const bf16x8 w = {(bf16_t)v[i][0].x, (bf16_t)v[i][0].y, (bf16_t)v[i][0].z, (bf16_t)v[i][0].w,
                          (bf16_t)v[i][1].x, (bf16_t)v[i][1].y, (bf16_t)v[i][1].z, (bf16_t)v[i][1].w};
        if (q.out)
            *(bf16x8 *)(q.out + (long long)z * q.s_out + l * blk_elems(R, C) + blk_off(r0 + row + i * 32, c0 + c, C)) = w;
#pragma unroll
        for (int k = 0; k < 8; ++k) tile[row + i * 32][c + k] = w[k];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        bf16x8 w;
#pragma unroll
        for (int k = 0; k < 8; ++k) w[k] = tile[c + k][row + i * 32];
        *(bf16x8 *)(q.outT + (long long)z * q.s_out + l * blk_elems(C, R) + blk_off(c0 + row + i * 32, r0 + c, R)) = w;
    }
}

// ---------------------------------------------------------------------------------------------
// LayerNorm
// ---------------------------------------------------------------------------------------------
template <int LPR>
__device__ __forceinline__ float row_sum(float v)      // over the LPR lanes of a row
{
#pragma unroll
    for (int o = LPR / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// A token row lies in the registers of LPR lanes as VPL float4 each (d <= 4 LPR VPL, d a multiple of 64): narrow rows share a
// wavefront.  Statistics in fp32, output u = gamma*xhat + beta in bf16 (64-bit stores) in the blocked layout.
template <int VPL, int LPR>
__device__ __forceinline__ void ln_row(const float4 (&xv)[VPL], const float *gam, bf16_t *u, float *mu_out, float *rstd_out,
                                       int row, int d)
{
    const int lane = threadIdx.x & (LPR - 1);
    const float *bet = gam + d;
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < VPL; ++c) s += (xv[c].x + xv[c].y) + (xv[c].z + xv[c].w);
    const float mean = row_sum<LPR>(s) / (float)d;
    float q = 0.f;
#pragma unroll
    for (int c = 0; c < VPL; ++c) {
        const int j = (lane + c * LPR) * 4;
        if (j < d) {
            float a = xv[c].x - mean, b = xv[c].y - mean, e = xv[c].z - mean, f = xv[c].w - mean;
            q = fmaf(a, a, q); q = fmaf(b, b, q); q = fmaf(e, e, q); q = fmaf(f, f, q);
        }
    }
    const float rstd = 1.0f / sqrtf(row_sum<LPR>(q) / (float)d + LN_EPS);
#pragma unroll
    for (int c = 0; c < VPL; ++c) {
        const int j = (lane + c * LPR) * 4;
        if (j < d) {
            const float4 gv = *(const float4 *)(gam + j), bv = *(const float4 *)(bet + j);
            bf16x4 o = {(bf16_t)fmaf(gv.x, (xv[c].x - mean) * rstd, bv.x), (bf16_t)fmaf(gv.y, (xv[c].y - mean) * rstd, bv.y),
                        (bf16_t)fmaf(gv.z, (xv[c].z - mean) * rstd, bv.z), (bf16_t)fmaf(gv.w, (xv[c].w - mean) * rstd, bv.w)};
            *(bf16x4 *)(u + blk_off(row, j, d)) = o;
        }
    }
    if (lane == 0) { *mu_out = mean; *rstd_out = rstd; }
}

// The residual stream and its gradient are streamed where they are beyond the caches, so that these keep the bf16 arrays that the
// products read: 8 x 12608 rows of 768 with attention, backward pass 253 -> 233 us (6.0 TB/s), 12 blocks 74.2 -> 72.5 ms of
// kernels (72.9 without the forward pass's loads).
static bool ln_stream(long long K, long long M, long long d) { return K * M * d >= 16000000; }
template <bool NT> __device__ __forceinline__ float4 load4f(const float *p) { return NT ? ld_nt4((const float4 *)p) : *(const float4 *)p; }
template <bool NT> __device__ __forceinline__ float4 load4f(const bf16_t *p)
{
    const bf16x4 v = NT ? __builtin_nontemporal_load((const bf16x4 *)p) : *(const bf16x4 *)p;
    return make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
}

template <int VPL, int LPR, bool NT>
__global__ __launch_bounds__(256) void ln_fwd_kernel(const float *__restrict__ X, long long sX,
                                                     const float *__restrict__ theta, long long sTh,
                                                     long long off_gamma, bf16_t *__restrict__ U,
                                                     long long sU, float *__restrict__ MU,
                                                     float *__restrict__ RSTD, long long sStat, int M, int d)
{
    const int z = blockIdx.y;
    const int row = blockIdx.x * (256 / LPR) + threadIdx.x / LPR, lane = threadIdx.x & (LPR - 1);
    if (row >= M) return;
    const float *x = X + (long long)z * sX + (long long)row * d;
    float4 xv[VPL];
#pragma unroll
    for (int c = 0; c < VPL; ++c) {
        const int j = (lane + c * LPR) * 4;
        xv[c] = j < d ? load4f<NT>(x + j) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    ln_row<VPL, LPR>(xv, theta + (long long)z * sTh + off_gamma, U + (long long)z * sU, MU + (long long)z * sStat + row,
                     RSTD + (long long)z * sStat + row, row, d);
}

// Sample() and the first LayerNorm: tokens x_0 ~ N(0,1), [M][d] per worker, the draws of a bulk fill of the flat array,
// stored in fp32 and in bf16 (blocked; the teacher map's operand), and normalized while the row is at hand.  Bound by the
// draws' arithmetic.  The first workgroup also clears the 256 bytes that stand in for missing rows in the weight-gradient
// GEMMs.
template <int VPL, int LPR>
__global__ __launch_bounds__(256) void sample_ln_kernel(float *__restrict__ X, long long sX, bf16_t *__restrict__ X0,
                                                        long long sX0, const float *__restrict__ theta, long long sTh,
                                                        long long off_gamma, bf16_t *__restrict__ U, long long sU,
                                                        float *__restrict__ MU, float *__restrict__ RSTD, long long sStat,
                                                        int M, int d, uint64_t seed, const DevState *__restrict__ st,
                                                        bf16_t *__restrict__ zero)
{
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 128) zero[threadIdx.x] = (bf16_t)0.0f;
    const int z = blockIdx.y;
    const int row = blockIdx.x * (256 / LPR) + threadIdx.x / LPR, lane = threadIdx.x & (LPR - 1);
    if (row >= M) return;
    const uint32_t t = (uint32_t)st->t;
    const long long i0 = (long long)row * (d >> 2);
    float4 *x = (float4 *)(X + (long long)z * sX) + i0;
    bf16_t *x0 = X0 + (long long)z * sX0;
    float4 xv[VPL];
#pragma unroll
    for (int c = 0; c < VPL; ++c) {
        const int q = lane + c * LPR;
        xv[c] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (q * 4 < d) {
            xv[c] = normal4(seed, STREAM_X, (uint32_t)z, t, (uint32_t)(i0 + q));
            st_nt4(x + q, xv[c]);
            const bf16x4 b = {(bf16_t)xv[c].x, (bf16_t)xv[c].y, (bf16_t)xv[c].z, (bf16_t)xv[c].w};
            *(bf16x4 *)(x0 + blk_off(row, q * 4, d)) = b;
        }
    }
    ln_row<VPL, LPR>(xv, theta + (long long)z * sTh + off_gamma, U + (long long)z * sU, MU + (long long)z * sStat + row,
                     RSTD + (long long)z * sStat + row, row, d);
}

// Backward of LayerNorm plus the residual path, rows shared out as in ln_rows.h, VPL float4 per lane:
//   dn = du*gamma; dx_out = dx_in + rstd*(dn - mean(dn) - xhat*mean(dn*xhat))
// dx_out may be dx_in (each element is read and then written by the same lane): the launcher does
// that, so the update of dx is one stream of addresses instead of two.
// and partial sums of dgamma = sum_m du*xhat, dbeta = sum_m du (reduced by
// colsum_final_kernel) of each workgroup's W wavefronts together.  TODX: the first sub-block's input is data, whose gradient nobody
// reads: only the sums then.
// NT: all but the bf16 gradient, which the next products read, with streaming accesses (ln_stream).
// W = 1: a wavefront's sums are a partial row by themselves, four wavefronts a workgroup.
template <int VPL, int LPR, int R, bool NT, typename TDU, bool TODX, int W>
__global__ __launch_bounds__(W == 1 ? 256 : 64 * W) void ln_bwd_kernel(const TDU *__restrict__ DU, long long sDU,
                                                     const float *__restrict__ X, long long sX,
                                                     const float *__restrict__ MU,
                                                     const float *__restrict__ RSTD, long long sStat,
                                                     const float *__restrict__ theta, long long sTh,
                                                     long long off_gamma, const float *DXin,
                                                     float *DXout, long long sDX,
                                                     bf16_t *__restrict__ DXb, long long sDXb,
                                                     float *__restrict__ PART, long long sPART,
                                                     int part_rows, int M, int d)
{
    constexpr int G = 64 / LPR;                          // rows side by side
    __shared__ float sums[W == 1 ? 1 : W][W == 1 ? 1 : 2][W == 1 ? 1 : 4 * VPL * LPR];
    const int z = blockIdx.y, wave = threadIdx.x >> 6, wave_rows = part_rows * W;
    const int wr = blockIdx.x * (W == 1 ? 4 : W) + wave, lane = threadIdx.x & (LPR - 1), grp = (threadIdx.x & 63) / LPR;
    if (W == 1 && wr >= wave_rows) return;
    const float *gam = theta + (long long)z * sTh + off_gamma;
    const TDU *du_z = DU + (long long)z * sDU;
    const float *x_z = X + (long long)z * sX, *di_z = DXin + (long long)z * sDX;
    const float *mu_z = MU + (long long)z * sStat, *rs_z = RSTD + (long long)z * sStat;
    float g[VPL][4], dg[VPL][4], db[VPL][4];
#pragma unroll
    for (int c = 0; c < VPL; ++c) {
        const int j = (lane + c * LPR) * 4;
        const float4 gv = j < d ? *(const float4 *)(gam + j) : make_float4(0.f, 0.f, 0.f, 0.f);
        g[c][0] = gv.x; g[c][1] = gv.y; g[c][2] = gv.z; g[c][3] = gv.w;
#pragma unroll
        for (int e = 0; e < 4; ++e) { dg[c][e] = 0.f; db[c][e] = 0.f; }
    }
    // wavefronts take groups of R * G rows in turn, so that the launch is at one stretch of each array at a time (runs of rows
    // of their own: 265 us against 256 at 8 x 12608 rows of 768)
    for (int n = wr; (long long)n * (G * R) + grp < M; n += wave_rows) {
        const int row0 = n * (G * R) + grp, r_end = M;
        float4 duv[R][VPL], xv[R][VPL], di[R][VPL];
        float mean[R], rstd[R];
        // all loads of R rows first; a row beyond the run is read again as the first one and counts for nothing
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int row = u == 0 || row0 + u * G < r_end ? row0 + u * G : row0;
            const long long o = (long long)row * d;
            mean[u] = mu_z[row]; rstd[u] = rs_z[row];
#pragma unroll
            for (int c = 0; c < VPL; ++c) {
                const int j = (lane + c * LPR) * 4;
                if (j < d) {
                    duv[u][c] = load4f<NT>(du_z + o + j);    // row-major in either type: no GEMM reads it
                    xv[u][c] = load4f<NT>(x_z + o + j);
                    if (TODX) di[u][c] = load4f<NT>(di_z + o + j);
                }
            }
        }
        float s1[R], s2[R];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const bool in = u == 0 || row0 + u * G < r_end;
            s1[u] = 0.f; s2[u] = 0.f;
#pragma unroll
            for (int c = 0; c < VPL; ++c) {
                const int j = (lane + c * LPR) * 4;
                if (j >= d || !in) { duv[u][c] = make_float4(0.f, 0.f, 0.f, 0.f); xv[u][c] = make_float4(mean[u], mean[u], mean[u], mean[u]); }
                const float du[4] = {duv[u][c].x, duv[u][c].y, duv[u][c].z, duv[u][c].w};
                const float xx[4] = {xv[u][c].x, xv[u][c].y, xv[u][c].z, xv[u][c].w};
                float xh[4], dn[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    xh[e] = (xx[e] - mean[u]) * rstd[u];
                    dn[e] = du[e] * g[c][e];
                    s1[u] += dn[e]; s2[u] = fmaf(dn[e], xh[e], s2[u]);
                    dg[c][e] = fmaf(du[e], xh[e], dg[c][e]); db[c][e] += du[e];
                }
                xv[u][c] = make_float4(xh[0], xh[1], xh[2], xh[3]);
                duv[u][c] = make_float4(dn[0], dn[1], dn[2], dn[3]);
            }
        }
        if (!TODX) continue;
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const float m1 = row_sum<LPR>(s1[u]) / (float)d, m2 = row_sum<LPR>(s2[u]) / (float)d;
            const int row = row0 + u * G;
            if (u > 0 && row >= r_end) continue;
            const long long o = (long long)row * d;
#pragma unroll
            for (int c = 0; c < VPL; ++c) {
                const int j = (lane + c * LPR) * 4;
                if (j < d) {
                    float4 v;
                    v.x = di[u][c].x + rstd[u] * (duv[u][c].x - m1 - xv[u][c].x * m2);
                    v.y = di[u][c].y + rstd[u] * (duv[u][c].y - m1 - xv[u][c].y * m2);
                    v.z = di[u][c].z + rstd[u] * (duv[u][c].z - m1 - xv[u][c].z * m2);
                    v.w = di[u][c].w + rstd[u] * (duv[u][c].w - m1 - xv[u][c].w * m2);
                    if (NT) st_nt4((float4 *)(DXout + (long long)z * sDX + o + j), v);
                    else *(float4 *)(DXout + (long long)z * sDX + o + j) = v;
                    bf16x4 b = {(bf16_t)v.x, (bf16_t)v.y, (bf16_t)v.z, (bf16_t)v.w};
                    *(bf16x4 *)(DXb + (long long)z * sDXb + o + j) = b;
                }
            }
        }
    }
    // rows side by side are added up across the wavefront
    if (G > 1) {
#pragma unroll
        for (int c = 0; c < VPL; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int o = LPR; o < 64; o <<= 1) { dg[c][e] += __shfl_xor(dg[c][e], o, 64); db[c][e] += __shfl_xor(db[c][e], o, 64); }
        if (W == 1 && grp > 0) return;
    }
    if constexpr (W > 1) {                               // the wavefronts' sums, in order
        if (grp == 0) {
#pragma unroll
            for (int c = 0; c < VPL; ++c) {
                const int j = (lane + c * LPR) * 4;
                *(float4 *)&sums[wave][0][j] = make_float4(dg[c][0], dg[c][1], dg[c][2], dg[c][3]);
                *(float4 *)&sums[wave][1][j] = make_float4(db[c][0], db[c][1], db[c][2], db[c][3]);
            }
        }
        __syncthreads();
        for (int i = threadIdx.x; i < 2 * d; i += 64 * W) {
            const int beta = i >= d, j = i - beta * d;
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < W; ++w) s += sums[w][beta][j];
            PART[(long long)z * sPART + ((long long)beta * part_rows + blockIdx.x) * d + j] = s;
        }
        return;
    }
    float *pg = PART + (long long)z * sPART + (long long)wr * d;
    float *pb = PART + (long long)z * sPART + ((long long)part_rows + wr) * d;
#pragma unroll
    for (int c = 0; c < VPL; ++c) {
        const int j = (lane + c * LPR) * 4;
        if (j < d) {
            *(float4 *)(pg + j) = make_float4(dg[c][0], dg[c][1], dg[c][2], dg[c][3]);
            *(float4 *)(pb + j) = make_float4(db[c][0], db[c][1], db[c][2], db[c][3]);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// column sums: final stage of the LayerNorm parameter gradients
// ---------------------------------------------------------------------------------------------
// Column sums of the partial rows that the wavefronts of a LayerNorm backward pass leave, and (last entry of blockIdx.z) the
// loss from its partial sums.  A workgroup owns 64 columns of dgamma or dbeta of one worker and LayerNorm; its 16
// wavefronts each sum a contiguous run of the chunks in ascending order, eight loads in flight, and the partial sums are
// added in wavefront order (fixed order: deterministic).  (Four wavefronts: 11.8 us for 505 chunks, a chain of loads.)
struct ColsumArgs {
    const float *part; long long s_part; int chunks, cols;      // [worker][LayerNorm][dgamma, dbeta][chunks][cols]
    float *out; long long s_out;                                // a worker's gradient
    long long off[2], l_out; int nsub;                          // LayerNorm i: at off[i % nsub] + i / nsub * l_out
    int sums;                                                   // LayerNorms times two
    const float *lpart; long long s_lpart; int n_lpart; float scale; float *loss;
};
constexpr int COLSUM_WAVES = 16;
__global__ __launch_bounds__(64 * COLSUM_WAVES) void colsum_final_kernel(ColsumArgs q)
{
    __shared__ float red[COLSUM_WAVES][64];
    const int z = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if ((int)blockIdx.z == q.sums) {                     // the loss (256 lanes took 17 us for 9456 parts, one load after the other)
        if (blockIdx.x > 0) return;
        const float *p = q.lpart + (long long)z * q.s_lpart;
        float acc = 0.f;
        for (int i = threadIdx.x; i < q.n_lpart; i += 4096) {
            float r[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) r[u] = i + u * 1024 < q.n_lpart ? p[i + u * 1024] : 0.f;
            acc += (r[0] + r[1]) + (r[2] + r[3]);
        }
        acc = row_sum<64>(acc);
        if (lane == 0) red[wave][0] = acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < COLSUM_WAVES; ++w) s += red[w][0];
            q.loss[z] = s * q.scale;
        }
        return;
    }
    const int j = blockIdx.x * 64 + lane, ln = blockIdx.z >> 1, beta = blockIdx.z & 1;
    const float *p = q.part + (long long)z * q.s_part + (long long)blockIdx.z * q.chunks * q.cols;
    const int per = (q.chunks + COLSUM_WAVES - 1) / COLSUM_WAVES;
    const int c0 = wave * per, c1 = min(q.chunks, c0 + per);
    float a8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (j < q.cols) {
        for (int c = c0; c < c1; c += 8) {               // a short last run is filled up with zeros
            float r[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) r[u] = p[(long long)min(c + u, c1 - 1) * q.cols + j];
#pragma unroll
            for (int u = 0; u < 8; ++u) a8[u] += c + u < c1 ? r[u] : 0.f;
        }
    }
    red[wave][lane] = ((a8[0] + a8[1]) + (a8[2] + a8[3])) + ((a8[4] + a8[5]) + (a8[6] + a8[7]));
    __syncthreads();
    if (wave == 0 && j < q.cols) {
        float s = red[0][lane];
#pragma unroll
        for (int w = 1; w < COLSUM_WAVES; ++w) s += red[w][lane];
        q.out[(long long)z * q.s_out + (q.nsub > 1 && (ln & 1) ? q.off[1] : q.off[0]) + (q.nsub > 1 ? ln >> 1 : ln) * q.l_out + beta * q.cols + j] = s;
    }
}

// ---------------------------------------------------------------------------------------------
// GEMM epilogues
// ---------------------------------------------------------------------------------------------
// Phi(h) and phi(h) of the standard normal, for GELU(h) = h Phi(h) and its derivative
// Phi(h) + h phi(h).  erf by the rational-times-Gaussian formula 7.1.26 of Abramowitz & Stegun
// (|error| <= 1.5e-7, far below the bf16 rounding of the outputs); its exp(-x^2) with
// x = |h|/sqrt(2) is exactly the Gaussian factor phi needs, so one exponential serves both.
// Written to be cheap on the vector ALU (this runs in GEMM epilogues over 3e8 elements per
// launch): x is never formed (its scale is folded into the constants), the factors 1/2 and t of
// the tail are folded into the polynomial, the exponential is one exp2 of h*h times a constant,
// and the reflection for h < 0 is a sign copy.
__device__ __forceinline__ void gelu_parts(float h, float &cdf, float &pdf)
{
    // t = 1 / (1 + p x), p x = (0.3275911 / sqrt(2)) |h|
    const float t = __builtin_amdgcn_rcpf(fmaf(0.23164189f, fabsf(h), 1.0f));
    // exp(-x^2) = exp(-h^2/2) = 2^(h*h * (-log2(e)/2))
    const float ex = __builtin_amdgcn_exp2f(h * h * -0.72134752f);
    // (1 - erf(x))/2 = ex * t * (a1/2 + t (a2/2 + t (a3/2 + t (a4/2 + t a5/2))))
    float q = fmaf(0.5307027145f, t, -0.7265760135f);
    q = fmaf(q, t, 0.7107068705f);
    q = fmaf(q, t, -0.142248368f);
    q = fmaf(q, t, 0.127414796f);
    const float half_tail = q * t * ex;
    // Phi(h) = 1/2 + sign(h) (1/2 - half_tail)
    cdf = 0.5f + copysignf(0.5f - half_tail, h);
    pdf = 0.3989422804014327f * ex;
}

// (All outputs of the GEMMs are stored non-temporally: written back through L2 they evicted the operands the
// other tiles share, 493 against 445 us for a bf16 output of 12608 x 3072 per worker, K = 768.)
__device__ __forceinline__ bf16x8 pack8(const float (&v)[8])
{
    bf16x8 r;
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = (bf16_t)v[i];
    return r;
}

struct EpiLoss {                 // y = scale * acc; r = x_L - y; dx = inv * r in fp32 and bf16; sums of r^2
    // The targets never exist in memory (written and read again by a kernel of its own: 155 + 178 us at 8 x 12608 x 768).
    const float *X; long long sX; float *DX; long long sDX; bf16_t *DXb; long long sDXb; float *LPART; long long sLPART;
    long long ld; float scale, inv;
    static constexpr int VEC = 4;
    static constexpr NtOut OUT = NT_LOSS;
    typedef float4 Aux;
    struct Lane { EpiPtr<const float, false> x; EpiPtr<float, false> o; EpiPtr<bf16_t, false> b; mutable double sum; };
    __device__ Lane lane(int z, int row, int col, int r, int c) const
    {
        return Lane{EpiPtr<const float, false>(X + (long long)z * sX, ld, row, col, r, c),
                    EpiPtr<float, false>(DX + (long long)z * sDX, ld, row, col, r, c),
                    EpiPtr<bf16_t, false>(DXb + (long long)z * sDXb, ld, row, col, r, c), 0.0};
    }
    __device__ Aux pre(const Lane &l, int dr) const { return ld_nt4((const float4 *)l.x.at(dr)); }
    __device__ void operator()(const Lane &l, int dr, const float (&v)[4], const Aux &x) const
    {
        const float r[4] = {x.x - v[0] * scale, x.y - v[1] * scale, x.z - v[2] * scale, x.w - v[3] * scale};
        l.sum += (double)fmaf(r[0], r[0], r[1] * r[1]) + (double)fmaf(r[2], r[2], r[3] * r[3]);
        const float g[4] = {r[0] * inv, r[1] * inv, r[2] * inv, r[3] * inv};
        st_nt4((float4 *)l.o.at(dr), make_float4(g[0], g[1], g[2], g[3]));
        const bf16x4 b = {(bf16_t)g[0], (bf16_t)g[1], (bf16_t)g[2], (bf16_t)g[3]};
        __builtin_nontemporal_store(b, (bf16x4 *)l.b.at(dr));
    }
    __device__ void finish(const Lane &l, int z, int unit) const
    {
        double s = l.sum;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if ((threadIdx.x & 63) == 0) LPART[(long long)z * sLPART + unit] = (float)s;
    }
};
struct EpiScaleF32 {             // C = scale * acc
    float *C; long long ldc, sC; float scale;
    static constexpr int VEC = 4;
    static constexpr NtOut OUT = NT_F32;
    typedef NoAux Aux;
    typedef EpiPtr<float, false> Lane;
    __device__ Lane lane(int z, int row, int col, int r, int c) const { return Lane(C + (long long)z * sC, ldc, row, col, r, c); }
    __device__ Aux pre(const Lane &, int) const { return Aux{}; }
    __device__ void operator()(const Lane &l, int dr, const float (&v)[4], const Aux &) const
    {
        st_nt4((float4 *)l.at(dr), make_float4(v[0] * scale, v[1] * scale, v[2] * scale, v[3] * scale));
    }
};
template <bool BLK>
struct EpiBf16 {                 // C = bf16(acc), row-major or blocked
    bf16_t *C; long long ldc, sC;
    static constexpr int VEC = 8;
    static constexpr NtOut OUT = NT_BF16;
    typedef NoAux Aux;
    typedef EpiPtr<bf16_t, BLK> Lane;
    __device__ Lane lane(int z, int row, int col, int r, int c) const { return Lane(C + (long long)z * sC, ldc, row, col, r, c); }
    __device__ Aux pre(const Lane &, int) const { return Aux{}; }
    __device__ void operator()(const Lane &l, int dr, const float (&v)[8], const Aux &) const
    {
        __builtin_nontemporal_store(pack8(v), (bf16x8 *)l.at(dr));
    }
};
// the lane's VEC bias values, the same for all its rows
template <int VEC>
struct EpiBias {
    float b[VEC];
    __device__ EpiBias(const float *p)
    {
#pragma unroll
        for (int u = 0; u < VEC; u += 4) {
            const float4 t = *(const float4 *)(p + u);
            b[u] = t.x; b[u + 1] = t.y; b[u + 2] = t.z; b[u + 3] = t.w;
        }
    }
};
struct EpiBiasBf16 {             // C = bf16(acc + bias)
    const float *bias; long long sBias; bf16_t *C; long long ldc, sC; int N;
    static constexpr int VEC = 8;
    static constexpr NtOut OUT = NT_BF16;
    typedef NoAux Aux;
    struct Lane { EpiPtr<bf16_t, false> o; EpiBias<8> b; };
    __device__ Lane lane(int z, int row, int col, int r, int c) const
    {
        return Lane{EpiPtr<bf16_t, false>(C + (long long)z * sC, ldc, row, col, r, c),
                    EpiBias<8>(bias + (long long)z * sBias + min(col + c, N - 8))};
    }
    __device__ Aux pre(const Lane &, int) const { return Aux{}; }
    __device__ void operator()(const Lane &l, int dr, const float (&v)[8], const Aux &) const
    {
        float r[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] = v[i] + l.b.b[i];
        __builtin_nontemporal_store(pack8(r), (bf16x8 *)l.o.at(dr));
    }
};
struct EpiBiasGelu {             // h = acc + b1; H = bf16(gelu'(h)); A = bf16(gelu(h)), both blocked
    // The backward pass needs h only through gelu'(h) = Phi(h) + h phi(h), and both factors are at
    // hand here: storing the derivative instead of h costs two instructions per element now and
    // saves the whole GELU evaluation in the data-gradient epilogue.
    const float *bias; long long sBias; bf16_t *H; long long sH; bf16_t *A; long long sA; long long ld;
    static constexpr int VEC = 8;
    static constexpr NtOut OUT = NT_GELU;
    typedef NoAux Aux;
    struct Lane { EpiPtr<bf16_t, true> h, a; EpiBias<8> b; };
    __device__ Lane lane(int z, int row, int col, int r, int c) const
    {
        return Lane{EpiPtr<bf16_t, true>(H + (long long)z * sH, ld, row, col, r, c),
                    EpiPtr<bf16_t, true>(A + (long long)z * sA, ld, row, col, r, c),
                    EpiBias<8>(bias + (long long)z * sBias + min(col + c, (int)ld - 8))};
    }
    __device__ Aux pre(const Lane &, int) const { return Aux{}; }
    __device__ void operator()(const Lane &l, int dr, const float (&v)[8], const Aux &) const
    {
        float a[8], dg[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float h = v[i] + l.b.b[i];
            float c, pdf;
            gelu_parts(h, c, pdf);
            a[i] = h * c;
            dg[i] = fmaf(h, pdf, c);
        }
        __builtin_nontemporal_store(pack8(dg), (bf16x8 *)l.h.at(dr));
        __builtin_nontemporal_store(pack8(a), (bf16x8 *)l.a.at(dr));
    }
};
struct EpiBiasResidual {         // x_out = x_in + acc + b2
    const float *bias; long long sBias; const float *Xin; float *Xout; long long sX; long long ld;
    static constexpr int VEC = 4;
    static constexpr NtOut OUT = NT_RESIDUAL;
    typedef float4 Aux;
    struct Lane { EpiPtr<const float, false> x; EpiPtr<float, false> o; EpiBias<4> b; };
    __device__ Lane lane(int z, int row, int col, int r, int c) const
    {
        return Lane{EpiPtr<const float, false>(Xin + (long long)z * sX, ld, row, col, r, c),
                    EpiPtr<float, false>(Xout + (long long)z * sX, ld, row, col, r, c),
                    EpiBias<4>(bias + (long long)z * sBias + min(col + c, (int)ld - 4))};
    }
    __device__ Aux pre(const Lane &l, int dr) const { return ld_nt4((const float4 *)l.x.at(dr)); }
    __device__ void operator()(const Lane &l, int dr, const float (&v)[4], const Aux &x) const
    {
        st_nt4((float4 *)l.o.at(dr), make_float4(x.x + v[0] + l.b.b[0], x.y + v[1] + l.b.b[1], x.z + v[2] + l.b.b[2], x.w + v[3] + l.b.b[3]));
    }
};
struct EpiGeluBwd {              // dh = acc * gelu'(h), H holding gelu'(h) from the forward pass; both blocked
    const bf16_t *H; long long sH; bf16_t *DH; long long sDH; long long ld;
    static constexpr int VEC = 8;
    static constexpr NtOut OUT = NT_FACTOR;
    typedef bf16x8 Aux;
    struct Lane { EpiPtr<const bf16_t, true> h; EpiPtr<bf16_t, true> o; };
    __device__ Lane lane(int z, int row, int col, int r, int c) const
    {
        return Lane{EpiPtr<const bf16_t, true>(H + (long long)z * sH, ld, row, col, r, c),
                    EpiPtr<bf16_t, true>(DH + (long long)z * sDH, ld, row, col, r, c)};
    }
    __device__ Aux pre(const Lane &l, int dr) const { return __builtin_nontemporal_load((const bf16x8 *)l.h.at(dr)); }
    __device__ void operator()(const Lane &l, int dr, const float (&v)[8], const Aux &hb) const
    {
        float r[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] = v[i] * (float)hb[i];
        __builtin_nontemporal_store(pack8(r), (bf16x8 *)l.o.at(dr));
    }
};

// The shapes of nt_plan.h with their wavefronts along M and N and the wavefronts per SIMD that the registers are budgeted for.
// BLKA: the activation operand is blocked (the weights always are).
template <bool BLKA, class Epi>
static hipError_t gemm_nt(const GemmNT &p, const Epi &epi, int batch, hipStream_t s)
{
    const NtShape shape = nt_shape(Epi::OUT, p.M, p.N, p.K, batch, gemm_cu_count());
#define CASE(SHAPE, WM, WN, WPS) if constexpr (nt_allowed(SHAPE, Epi::OUT)) \
        if (shape == SHAPE) return launch_gemm_nt<SHAPE, WM, WN, WPS, BLKA>(p, epi, batch, s)
    CASE(NT_256x256, 2, 4, 2);
    CASE(NT_128x256, 1, 4, 2);
    CASE(NT_128x128_LONG, 2, 2, 2);
    CASE(NT_128x128, 2, 2, 3);
    CASE(NT_64x64_LONG, 2, 2, 2);
    CASE(NT_64x64, 2, 2, 4);
#undef CASE
    return hipErrorInvalidValue;
}
// wavefronts of all tiles of a batch entry
template <class Epi>
static int nt_units(const GemmNT &p, int batch)
{
    const NtShape shape = nt_shape(Epi::OUT, p.M, p.N, p.K, batch, gemm_cu_count());
    return (int)nt_tiles(shape, p.M, p.N, 1) * (shape == NT_256x256 ? 8 : 4);
}
#define TRY(expr) do { hipError_t e_ = (expr); if (e_ != hipSuccess) return e_; } while (0)

// out[z][i] = part[z][0][i] + part[z][1][i] + ... (ascending: a fixed order) for the n elements from `first` on of each
// block (blockIdx.z, l_out apart), n a multiple of 4
__global__ __launch_bounds__(256) void splitk_sum_kernel(const float *__restrict__ part, long long span, int split,
                                                         float *__restrict__ out, long long sOut, long long l_out,
                                                         long long first, long long n)
{
    const long long j = ((long long)blockIdx.x * 256 + threadIdx.x) * 4;
    if (j >= n) return;
    const int z = blockIdx.y;
    const long long i = blockIdx.z * l_out + first + j;
    const float *p = part + (long long)z * split * span + i;
    float4 a = *(const float4 *)p;
    for (int s = 1; s < split; ++s) {
        const float4 b = *(const float4 *)(p + (long long)s * span);
        a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
    }
    *(float4 *)(out + (long long)z * sOut + i) = a;
}

// Weight gradients dW = A^T B with the bias gradients (column sums of B) as by-products, collected into one launch: of
// n_l blocks whose gradients lie l_out apart in a worker's gradient, the first one's at [lo, hi) of it.  Widths are multiples of 64 and a block of
// zeros stands in for ragged token counts, so every weight gradient of this model qualifies.
// Tile shape and token ranges: wgrad_plan.h.
struct WgradLaunch {
    TnGroup t{};
    long long lo = 0, hi = 0;                            // what a block's part of the launch covers of its gradient
    long long lo2 = 0, hi2 = 0;                          // a second range, where all sub-blocks share the launch
    void add(const bf16_t *A, bool blkA, long long lda, long long sA, long long lA, const bf16_t *B, bool blkB, long long ldb,
             long long sB, long long lB, int M, int N, long long off, long long off_b)
    {
        TnProblem &p = t.p[t.n++];
        p.A = A; p.B = B; p.lda = lda; p.ldb = ldb; p.sA = sA; p.sB = sB; p.lA = lA; p.lB = lB;
        p.off = off; p.off_colsum = off_b; p.M = M; p.N = N; p.blkA = blkA; p.blkB = blkB;
    }
};
static hipError_t launch_wgrad(WgradLaunch q, const WgradCover &cover, float *g, long long P, int tokens, const ResWs &w, int batch, hipStream_t s)
{
    TnGroup &t = q.t;
    t.zeros = w.ZERO; t.K = tokens;
    const long long span = (t.n_l - 1) * t.l_out + (q.hi2 > q.hi ? q.hi2 : q.hi) - q.lo;
    if (span != cover.floats) return hipErrorInvalidValue;
    const WgradPlan plan = wgrad_plan_load(cover.load, tokens, gemm_cu_count(), w.split_floats, batch * span);
    t.split = plan.split; t.k_chunk = plan.k_chunk;
    t.out = g + q.lo; t.s_out = P;
    if (plan.split > 1) {
        if (batch * plan.split * span > w.split_floats) return hipErrorInvalidValue;
        t.out = w.SPLITK; t.s_out = span;
    }
    for (int e = 0; e < t.n; ++e) { t.p[e].off -= q.lo; t.p[e].off_colsum -= q.lo; }
    switch (plan.tile) {
    case WGRAD_192x384: TRY((launch_gemm_tn<192, 384, 2, 4, 1, 2, 4>(t, batch, s))); break;
    case WGRAD_128x128: TRY((launch_gemm_tn<128, 128, 2, 2, 1, 3, 3>(t, batch, s))); break;
    case WGRAD_128x128_2GROUPS: TRY((launch_gemm_tn<128, 128, 2, 2, 2, 2, 4>(t, batch, s))); break;
    default: TRY((launch_gemm_tn<64, 64, 2, 2, 4, 4, 3>(t, batch, s))); break;
    }
    if (plan.split > 1) {
        const long long first[2] = {0, q.lo2 - q.lo}, n[2] = {q.hi - q.lo, q.hi2 - q.lo2};
        for (int r = 0; r < 2; ++r)
            if (n[r] > 0) {
                splitk_sum_kernel<<<dim3((unsigned)((n[r] / 4 + 255) / 256), (unsigned)batch, (unsigned)t.n_l), 256, 0, s>>>(
                    w.SPLITK, span, plan.split, g + q.lo, P, t.l_out, first[r], n[r]);
                TRY(hipGetLastError());
            }
    }
    return hipSuccess;
}

hipError_t launch_resmlp_grad(const ModelDims &dm, const float *theta, float *g, const float *teacher,
                              void *ws, float *loss, const DevState *st, hipStream_t s)
{
    const int K = dm.K, M = (int)dm.B, d = (int)dm.d_in, dh = (int)dm.d_hidden, L = dm.n_blocks;
    const int heads = dm.n_heads, S = (int)dm.seq_len;
    const int nsub = heads > 0 ? 2 : 1;           // residual sub-blocks per block
    const long long P = dm.P;
    const long long dd = (long long)d * d;
    const long long per_attn = heads > 0 ? 2LL * d + 3 * dd + 3LL * d + dd + d : 0;
    const long long per_block = per_attn + 2LL * d + (long long)d * dh + dh + (long long)dh * d + d;
    if (heads > 0 && !attn_supports(d, heads, S, M)) return hipErrorInvalidValue;
    const long long oWq = 2LL * d, obq = oWq + 3 * dd, oWo = obq + 3LL * d, obo = oWo + dd;      // inside a block
    const long long oW1 = per_attn + 2LL * d, ob1 = oW1 + (long long)d * dh, oW2 = ob1 + dh, ob2 = oW2 + (long long)dh * d;
    ResWs w = carve(dm, ws, nullptr);
    const long long Md = (long long)M * d;            // a row-major [M][d] array (fp32 state and its relatives)
    const long long MdB = w.mdB, MdhB = w.mdhB;       // a blocked [M][d] / [M][dh] bf16 array
    const LnBwdPlan ln_plan = ln_bwd_plan(K, M, d);
    const int part_rows = (int)ln_plan.waves;

    AttnArgs att{};
    if (heads > 0) {
        att.sQKV = w.sQKV; att.sO = w.sO; att.sLSE = w.sLSE; att.DO = w.DO; att.sDO = w.sDO;
        att.DQKV = w.DQKV; att.sDQKV = w.sDQKV;
        att.M = M; att.d = d; att.S = S; att.nb = (S + 31) / 32;
        att.scale = 1.0f / sqrtf((float)ATT_DK);
        att.c2 = 1.4426950408889634f * att.scale;
    }

    const bool stream = ln_stream(K, M, d);
    // LayerNorm of residual state number `sub` with the parameters at off_gamma
    auto ln_fwd = [&](int sub, long long off_gamma) -> hipError_t {
#define LN_FWD_NT(VPL, LPR, NT) ln_fwd_kernel<VPL, LPR, NT><<<dim3((unsigned)((M + 256 / LPR - 1) / (256 / LPR)), (unsigned)K), 256, 0, s>>>( \
                        w.X + (long long)sub * Md, w.sX, theta, P, off_gamma, \
                        w.U + (long long)sub * MdB, w.sU, w.MU + (long long)sub * M, w.RSTD + (long long)sub * M, w.sStat, M, d)
#define LN_FWD(VPL, LPR) do { if (stream) LN_FWD_NT(VPL, LPR, true); else LN_FWD_NT(VPL, LPR, false); } while (0)
        LN_BY_WIDTH(d, LN_FWD);
#undef LN_FWD_NT
#undef LN_FWD
        return hipGetLastError();
    };
    // The gradient with respect to a LayerNorm's output comes out of a bf16 GEMM.  In the MLP-only
    // model it is stored in bf16, like the activations (2 B instead of 4 written by the GEMM and
    // read by the pass below: 2-3 % of an iteration at the benchmark size).  With attention
    // sub-blocks it stays in fp32: the query-weight gradients, sums of small softmax-gradient
    // terms, sit at the tested error bound already, and this one more rounding (in the MLP
    // sub-block alone) moved an entry past it.  The buffer is the same.
    const bool du16 = heads == 0;
    bf16_t *const DU16 = (bf16_t *)w.DU;
    const long long sDU16 = 2 * w.sDU;
    // its backward pass plus the residual path: DX (d loss / d state sub+1) and DU -> DX in place
    // (d loss / d state sub, also in bf16), and the LayerNorm parameter gradients
    int loss_parts = 0;
    auto ln_bwd = [&](int sub, long long off_gamma) -> hipError_t {
        dim3 grid((unsigned)(ln_plan.few ? part_rows : (part_rows + 3) / 4), (unsigned)K);
        bf16_t *const dxb_to = w.DXb + (long long)(w.defer && sub > 0 ? sub - 1 : 0) * Md;   // of the sub-block before, if there is one
#define LN_BWD_ARGS w.X + (long long)sub * Md, w.sX, w.MU + (long long)sub * M, w.RSTD + (long long)sub * M, w.sStat, theta, P, off_gamma, \
                    w.DX, w.DX, w.sDX, dxb_to, w.sDXb, w.PART + (w.defer ? 2LL * sub * part_rows * d : 0), w.sPART, part_rows, M, d
#define LN_BWD_R(VPL, LPR, R, NT, W) do { \
            const unsigned threads = W == 1 ? 256 : 64 * W; \
            if (du16 && sub > 0) ln_bwd_kernel<VPL, LPR, R, NT, bf16_t, true, W><<<grid, threads, 0, s>>>(DU16, sDU16, LN_BWD_ARGS); \
            else if (du16) ln_bwd_kernel<VPL, LPR, R, NT, bf16_t, false, W><<<grid, threads, 0, s>>>(DU16, sDU16, LN_BWD_ARGS); \
            else if (sub > 0) ln_bwd_kernel<VPL, LPR, R, NT, float, true, W><<<grid, threads, 0, s>>>(w.DU, w.sDU, LN_BWD_ARGS); \
            else ln_bwd_kernel<VPL, LPR, R, NT, float, false, W><<<grid, threads, 0, s>>>(w.DU, w.sDU, LN_BWD_ARGS); } while (0)
#define LN_BWD(VPL, LPR) do { if (ln_plan.few) LN_BWD_R(VPL, LPR, 1, false, LN_FEW_WAVES); \
                              else if (!stream) LN_BWD_R(VPL, LPR, ln_bwd_rows(VPL), false, 1); \
                              else LN_BWD_R(VPL, LPR, ln_bwd_rows(VPL), true, 1); } while (0)
        LN_BY_WIDTH(d, LN_BWD);
#undef LN_BWD
#undef LN_BWD_R
#undef LN_BWD_ARGS
        TRY(hipGetLastError());
        // the sums over wavefronts: after each pass, or after the last one for all where the partial rows are kept
        if (w.defer && sub > 0) return hipSuccess;
        ColsumArgs q{w.PART, w.sPART, part_rows, d, g, P, {0, per_attn}, per_block, nsub, w.defer ? 2 * nsub * L : 2,
                     w.LPART, w.sLPART, loss_parts, 0.5f / ((float)M * (float)d), loss};
        if (!w.defer || nsub == 1) { q.off[0] = off_gamma; q.nsub = 1; }
        colsum_final_kernel<<<dim3((unsigned)((d + 63) / 64), (unsigned)K, (unsigned)(q.sums + (sub == 0 ? 1 : 0))), 64 * COLSUM_WAVES, 0, s>>>(q);
        return hipGetLastError();
    };

    // bf16 copies of the weights in both orientations (the master weights changed last step), and the teacher map
    {
        CvtList list{};
        long long first = 0;
        auto add = [&](const float *in, long long s_in, bf16_t *out, bf16_t *outT, long long s_out, int R, int C, int n_l, int n_z) {
            list.m[list.n++] = CvtMat{in, s_in, per_block, out, outT, s_out, R, C, n_l, n_z, (int)first};
            first += (long long)(R / 64) * (C / 64) * n_l * n_z;
        };
        add(theta + oW1, P, w.W1b, w.W1Tb, w.sW, d, dh, L, K);
        add(theta + oW2, P, w.W2b, w.W2Tb, w.sW, dh, d, L, K);
        if (heads > 0) {
            add(theta + oWq, P, w.Wqb, w.WqTb, w.sWq, d, 3 * d, L, K);
            add(theta + oWo, P, w.Wob, w.WoTb, w.sWo, d, d, L, K);
        }
        add(teacher, 0, nullptr, w.WTt, 0, d, d, 1, 1);
        if (first > 0x7FFFFFFFll) return hipErrorInvalidValue;
        cvt_transpose_kernel<<<(unsigned)first, 256, 0, s>>>(list);
        TRY(hipGetLastError());
    }
    // elements of one block's blocked weight copies: as stored ([rows][cols]) and transposed
    const long long wW1 = w.wB[0], wW1T = w.wB[1], wW2 = w.wB[1], wW2T = w.wB[0];
    const long long wWq = blk_elems(d, 3 * d), wWqT = blk_elems(3 * d, d), wWo = blk_elems(d, d);

    // Sample(): tokens x_0 (fp32 in X[0], bf16 in DU), and the first sub-block's LayerNorm
    bf16_t *const X0 = (bf16_t *)w.DU;
    const long long sX0 = 2 * w.sDU;
#define SAMPLE_LN(VPL, LPR) sample_ln_kernel<VPL, LPR><<<dim3((unsigned)((M + 256 / LPR - 1) / (256 / LPR)), (unsigned)K), 256, 0, s>>>( \
                        w.X, w.sX, X0, sX0, theta, P, heads > 0 ? 0 : per_attn, w.U, w.sU, w.MU, w.RSTD, w.sStat, M, d, dm.seed, st, w.ZERO)
    LN_BY_WIDTH(d, SAMPLE_LN);
#undef SAMPLE_LN
    TRY(hipGetLastError());

    // forward
    for (int l = 0; l < L; ++l) {
        int sub = nsub * l;
        if (heads > 0) {
            const long long oga = l * per_block, obq = oga + 2LL * d + 3 * dd, obo = obq + 3LL * d + dd;
            bf16_t *QKVl = w.QKV + (long long)l * M * 3 * d, *Ol = w.O + (long long)l * Md;
            if (sub > 0) TRY(ln_fwd(sub, oga));
            {
                GemmNT p{w.U + (long long)sub * MdB, w.WqTb + l * wWqT, M, 3 * d, d, d, d, w.sU, w.sWq};
                EpiBiasBf16 epi{theta + obq, P, QKVl, 3LL * d, w.sQKV, 3 * d};
                TRY(gemm_nt<true>(p, epi, K, s));
            }
            att.QKV = QKVl; att.O = Ol; att.LSE = w.LSE + (long long)l * heads * M;
            TRY(launch_attn_fwd(att, heads, K, s));
            {
                GemmNT p{Ol, w.WoTb + l * wWo, M, d, d, d, d, w.sO, w.sWo};
                EpiBiasResidual epi{theta + obo, P, w.X + (long long)sub * Md, w.X + (long long)(sub + 1) * Md, w.sX, d};
                TRY(gemm_nt<false>(p, epi, K, s));
            }
            ++sub;
        }
        const long long og = l * per_block + per_attn, ob1 = og + 2LL * d + (long long)d * dh,
                        ob2 = ob1 + dh + (long long)dh * d;
        const float *Xl = w.X + (long long)sub * Md;
        float *Xn = w.X + (long long)(sub + 1) * Md;
        bf16_t *Ul = w.U + (long long)sub * MdB, *Al = w.A + (long long)l * MdhB;
        if (sub > 0) TRY(ln_fwd(sub, og));
        {
            GemmNT p{Ul, w.W1Tb + l * wW1T, M, dh, d, d, d, w.sU, w.sW};
            EpiBiasGelu epi{theta + ob1, P, w.H + (long long)l * MdhB, w.sH, Al, w.sA, dh};
            TRY(gemm_nt<true>(p, epi, K, s));
        }
        {
            GemmNT p{Al, w.W2Tb + l * wW2T, M, d, dh, dh, dh, w.sA, w.sW};
            EpiBiasResidual epi{theta + ob2, P, Xl, Xn, w.sX, d};
            TRY(gemm_nt<true>(p, epi, K, s));
        }
    }

    // targets y = x_0 W_T / sqrt(d), loss and d loss / d x_L
    {
        const float inv = 1.0f / ((float)M * (float)d);
        GemmNT p{X0, w.WTt, M, d, d, d, d, sX0, 0};
        EpiLoss epi{w.X + (long long)(nsub * L) * Md, w.sX, w.DX, w.sDX, w.DXb + (long long)(w.defer ? nsub * L - 1 : 0) * Md, w.sDXb,
                    w.LPART, w.sLPART, d, 1.0f / sqrtf((float)d), inv};
        TRY(gemm_nt<true>(p, epi, K, s));
        loss_parts = nt_units<EpiLoss>(p, K);                     // summed up with the last LayerNorm gradients
    }

    // The weight gradients of one block's MLP half and of its attention half (w.defer: as the first of all blocks')
    const int kept = w.defer ? 1 : 0;                    // copies of the gradients w.r.t. activations: one, or one for each block
    auto wgrad_mlp = [&](WgradLaunch &q, int l) {
        const long long sub = (long long)nsub * l + nsub - 1, lo = l * per_block;
        // W1 and b1:  dW1 = u^T dh, db1 = column sums of dh
        q.add(w.U + sub * MdB, true, d, w.sU, nsub * MdB, w.DH + kept * l * MdhB, true, dh, w.sDH, kept * MdhB, d, dh, lo + oW1, lo + ob1);
        // W2 and b2:  dW2 = a^T dx, db2 = column sums of dx
        q.add(w.A + l * MdhB, true, dh, w.sA, MdhB, w.DXb + kept * sub * Md, false, d, w.sDXb, kept * nsub * Md, dh, d, lo + oW2, lo + ob2);
        q.lo = lo + oW1; q.hi = lo + ob2 + d;
    };
    auto wgrad_attn = [&](WgradLaunch &q, int l) {
        const long long sub = (long long)nsub * l, lo = l * per_block;
        // Wqkv and bqkv:  dWqkv = u^T dqkv, dbqkv = column sums of dqkv
        q.add(w.U + sub * MdB, true, d, w.sU, nsub * MdB, w.DQKV + (long long)kept * l * M * 3 * d, false, 3LL * d, w.sDQKV,
              (long long)kept * M * 3 * d, d, 3 * d, lo + oWq, lo + obq);
        // Wo and bo:  dWo = o^T dx, dbo = column sums of dx
        q.add(w.O + l * Md, false, d, w.sO, Md, w.DXb + kept * sub * Md, false, d, w.sDXb, kept * nsub * Md, d, d, lo + oWo, lo + obo);
        q.lo = lo + oWq; q.hi = lo + obo + d;
    };
    auto one_block = [&](WgradLaunch &q, bool mlp) -> hipError_t {
        q.t.n_l = 1; q.t.l_out = per_block;
        return launch_wgrad(q, wgrad_cover(mlp, false, K, d, dh, heads > 0, L), g, P, M, w, K, s);
    };

    // backward; DX (and its bf16 copy DXb) holds d loss / d (output of the sub-block at hand)
    for (int l = L - 1; l >= 0; --l) {
        int sub = nsub * l + nsub - 1;
        const long long og = l * per_block + per_attn;
        bf16_t *DHl = w.DH + kept * l * MdhB;
        const bf16_t *dxb = w.DXb + (long long)kept * sub * Md;
        // dh = (dx W2^T) * gelu'(h)
        {
            GemmNT p{dxb, w.W2b + l * wW2, M, dh, d, d, d, w.sDXb, w.sW};
            EpiGeluBwd epi{w.H + (long long)l * MdhB, w.sH, DHl, w.sDH, dh};
            TRY(gemm_nt<false>(p, epi, K, s));
        }
        if (!w.defer) {
            WgradLaunch q;
            wgrad_mlp(q, l);
            TRY(one_block(q, true));
        }
        // du = dh W1^T, then LayerNorm backward + residual
        {
            GemmNT p{DHl, w.W1b + l * wW1, M, d, dh, dh, dh, w.sDH, w.sW};
            if (du16) {
                EpiBf16<false> epi{DU16, d, sDU16};
                TRY(gemm_nt<true>(p, epi, K, s));
            } else {
                EpiScaleF32 epi{w.DU, d, w.sDU, 1.0f};
                TRY(gemm_nt<true>(p, epi, K, s));
            }
        }
        TRY(ln_bwd(sub, og));
        if (heads > 0) {
            --sub;
            const long long oga = l * per_block;
            bf16_t *QKVl = w.QKV + (long long)l * M * 3 * d, *Ol = w.O + (long long)l * Md;
            bf16_t *DQKVl = w.DQKV + (long long)kept * l * M * 3 * d;
            const bf16_t *dxa = w.DXb + (long long)kept * sub * Md;
            // do = dx Wo^T
            {
                GemmNT p{dxa, w.Wob + l * wWo, M, d, d, d, d, w.sDXb, w.sWo};
                EpiBf16<false> epi{w.DO, d, w.sDO};
                TRY(gemm_nt<false>(p, epi, K, s));
            }
            att.QKV = QKVl; att.O = Ol; att.LSE = w.LSE + (long long)l * heads * M; att.DQKV = DQKVl;
            TRY(launch_attn_bwd(att, heads, K, s));
            if (!w.defer) {
                WgradLaunch q;
                wgrad_attn(q, l);
                TRY(one_block(q, false));
            }
            // du = dqkv Wqkv^T, then LayerNorm backward + residual
            {
                GemmNT p{DQKVl, w.Wqb + l * wWq, M, d, 3 * d, 3LL * d, 3LL * d, w.sDQKV, w.sWq};
                EpiScaleF32 epi{w.DU, d, w.sDU, 1.0f};
                TRY(gemm_nt<false>(p, epi, K, s));
            }
            TRY(ln_bwd(sub, oga));
        }
    }
    if (w.defer) {                                       // all weight gradients of all blocks
        WgradLaunch q;
        wgrad_mlp(q, 0);
        if (heads > 0) {
            const long long lo = q.lo, hi = q.hi;
            wgrad_attn(q, 0);
            q.lo2 = lo; q.hi2 = hi;
        }
        q.t.n_l = L; q.t.l_out = per_block;
        TRY(launch_wgrad(q, wgrad_cover(true, true, K, d, dh, heads > 0, L), g, P, M, w, K, s));
    }
    return hipSuccess;
}

}  // namespace qsr
