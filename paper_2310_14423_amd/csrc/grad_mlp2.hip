// grad_mlp2.hip -- local gradient (Eq. (1) of arXiv 2310.14423) of the two-layer perceptron
// workload for all K workers in batched launches.  Parameters of one worker are packed as
// W1 [d_in][d_hidden], b1 [d_hidden], W2 [d_hidden][d_out], b2 [d_out]; the gradient uses the
// same packing.  hidden = relu(x W1 + b1); logits = hidden W2 + b2; loss = mean softmax
// cross-entropy.  Inputs: label_i uniform over the classes, x_i = mean[label_i] + sigma*N(0,I),
// drawn per (worker, iteration) from Philox4x32-10.
#include "philox.h"
#include "qsr_internal.h"
#include "sgemm.h"

namespace qsr {

// Rows of X, hid, dhid and, with more than 16 classes, logit are padded to a multiple of 4 floats, so that every product reads
// them with 128-bit accesses whatever the widths (the padding is read and never counts).
struct Mlp2Ws {
    float *X, *hid, *dhid, *logit;
    long long ldx, ldh, ldz;
    float *part;           // [K][tiles of 16 rows][17]: column sums of dlogit and the summed loss of a tile
                           // (more than 16 classes: [K][B], the samples' losses)
    int *label;
};

static size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

static Mlp2Ws carve(const ModelDims &d, void *ws, size_t *total)
{
    char *p = (char *)ws;
    size_t off = 0;
    Mlp2Ws w;
    size_t K = (size_t)d.K, B = (size_t)d.B;
    w.ldx = (d.d_in + 3) / 4 * 4; w.ldh = (d.d_hidden + 3) / 4 * 4; w.ldz = d.d_out > 16 ? (d.d_out + 3) / 4 * 4 : d.d_out;
    w.X = (float *)(p + off);     off += up256(K * B * w.ldx * sizeof(float));
    w.hid = (float *)(p + off);   off += up256(K * B * w.ldh * sizeof(float));
    w.dhid = (float *)(p + off);  off += up256(K * B * w.ldh * sizeof(float));
    w.logit = (float *)(p + off); off += up256(K * B * w.ldz * sizeof(float));
    w.part = (float *)(p + off);  off += up256(K * ((B + 15) / 16) * 17 * sizeof(float));
    w.label = (int *)(p + off);   off += up256(K * B * sizeof(int));
    if (total) *total = off;
    return w;
}

size_t mlp2_workspace_bytes(const ModelDims &d)
{
    size_t total = 0;
    carve(d, nullptr, &total);
    return total;
}

// Sample() in one pass: label c_i uniform over the classes, x_i = mu_{c_i} + sigma z.  One thread
// per group of four consecutive elements of a worker's [B][d_in] batch (the group is the Philox
// counter of the normal draws); the label of a row comes from word i % 4 of the label stream's
// group i / 4 and is recomputed by every thread that needs it, which is cheaper than a kernel of
// its own; the thread that holds a row's first element also stores the label for the loss.
__global__ __launch_bounds__(64) void mlp2_sample_kernel(float *__restrict__ X, int *__restrict__ label,
                                                         const float *__restrict__ means, long long B,
                                                         long long d_in, long long ldx, uint32_t classes, float sigma,
                                                         uint64_t seed, const DevState *__restrict__ st)
{
    const uint32_t t = (uint32_t)st->t;
    const uint32_t k = blockIdx.y;
    const long long n = B * d_in, groups = (n + 3) / 4;
    float *x = X + (long long)k * B * ldx;
    int *lab = label + (long long)k * B;
    auto label_of = [&](long long i) {
        const U4 r = draw4(seed, STREAM_LABEL, k, t, (uint32_t)(i >> 2));
        const uint32_t w = (i & 3) == 0 ? r.x : (i & 3) == 1 ? r.y : (i & 3) == 2 ? r.z : r.w;
        return (int)index_from_word(w, classes);
    };
    const long long stride = (long long)gridDim.x * 64;
    for (long long q = (long long)blockIdx.x * 64 + threadIdx.x; q < groups; q += stride) {
        const float4 z4 = normal4(seed, STREAM_X, k, t, (uint32_t)q);
        const float z[4] = {z4.x, z4.y, z4.z, z4.w};
        const long long p = q * 4;
        long long i = p / d_in, j = p - i * d_in;
        int c = label_of(i);
        if (ldx == d_in) {                               // four columns of one row
            const float *mu = means + (long long)c * d_in + j;
            if (j == 0) lab[i] = c;
            const float4 o = make_float4(z[0] * sigma + mu[0], z[1] * sigma + mu[1], z[2] * sigma + mu[2], z[3] * sigma + mu[3]);
            *(float4 *)(x + p) = o;
            continue;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (p + e < n) {
                if (j == 0) lab[i] = c;
                x[i * ldx + j] = z[e] * sigma + means[(long long)c * d_in + j];
                if (++j == d_in) {
                    j = 0; ++i;
                    if (e < 3 && p + e + 1 < n) c = label_of(i);
                }
            }
        }
    }
}

// More than 16 classes: logits -> (softmax - onehot)/B in place, and the sample's cross-entropy.  One wavefront per
// sample, the classes across its lanes (as one lane per sample and one workgroup per worker it took 43 us for
// 5 x 50 samples of 100 classes).
__global__ __launch_bounds__(256) void mlp2_softmax_ce_kernel(float *__restrict__ z_dz,
                                                              const int *__restrict__ label,
                                                              float *__restrict__ sample_loss, long long B, int C, long long ldz)
{
    const int k = blockIdx.y, lane = threadIdx.x & 63;
    const long long i = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= B) return;
    const float invB = 1.0f / (float)B;
    float *z = z_dz + ((long long)k * B + i) * ldz;
    const int y = label[(long long)k * B + i];
    float v[16];                                         // C <= 1024
    float mx = -INFINITY;
#pragma unroll
    for (int u = 0; u < 16; ++u)
        if (u * 64 < C) {
            v[u] = u * 64 + lane < C ? z[u * 64 + lane] : -INFINITY;
            mx = fmaxf(mx, v[u]);
        }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    float se = 0.f, zy = 0.f;
#pragma unroll
    for (int u = 0; u < 16; ++u)
        if (u * 64 < C) {
            if (u * 64 + lane == y) zy = v[u] - mx;
            v[u] = u * 64 + lane < C ? expf(v[u] - mx) : 0.f;
            se += v[u];
        }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { se += __shfl_xor(se, o, 64); zy += __shfl_xor(zy, o, 64); }
    const float inv = 1.0f / se;
#pragma unroll
    for (int u = 0; u < 16; ++u)
        if (u * 64 + lane < C) z[u * 64 + lane] = (v[u] * inv - (u * 64 + lane == y ? 1.f : 0.f)) * invB;
    if (lane == 0) sample_loss[(long long)k * B + i] = logf(se) - zy;
}

// Exchanges inside a row of 16 lanes: with lane ^ 1, ^ 2, ^ 7, ^ 8 (in a sum or a maximum ^ 7 stands for ^ 4: the four
// lanes of a group already hold the same)
template <int CTRL> __device__ __forceinline__ float row_get(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL> __device__ __forceinline__ double row_get(double v)
{
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float row_sum(float v)
{
    v += row_get<0xb1>(v); v += row_get<0x4e>(v); v += row_get<0x141>(v);
    return v + row_get<0x128>(v);
}
__device__ __forceinline__ double row_max(double v)
{
    double t = row_get<0xb1>(v); v = t > v ? t : v;
    t = row_get<0x4e>(v); v = t > v ? t : v;
    t = row_get<0x141>(v); v = t > v ? t : v;
    t = row_get<0x128>(v);
    return t > v ? t : v;
}

// Output layer forward and loss for at most 16 classes, one workgroup per 16 samples of a worker:
// logits = hid W2 + b2 with products and sums in double precision on the fp64 matrix cores (one
// 16x16x4 instruction covers 16 samples x 16 classes x 4 hidden units; each of the WAVES wavefronts takes its
// share of the hidden units, and the first four add up the partial results, in order, of four samples each), then
// the softmax of each row across the 16 lanes that hold it: the maximum is subtracted in double
// before anything is rounded to fp32.  At the workload's step size the logits grow into the hundreds
// within a few iterations, where one fp32 ulp of a logit (6e-5 at 600) would be the relative error
// of the probability computed from it; the difference to the largest logit is small and rounds
// harmlessly.  Written: dlogit = (softmax - onehot)/B, and per tile the column sums of dlogit and
// the summed cross-entropy (mlp2_out_bwd_kernel adds the tiles up).
// Bound by latency, 64 workgroups at 8 x 128 samples: 8.2 us with 1024 hidden units, 10 classes (10.8 with eight wavefronts, the
// softmax of all sixteen samples in the first one and exchanges through LDS).  Sixteen wavefronts while each workgroup has a
// compute unit to itself, eight beyond (us, 16 / 8, at 64, 1024 and 3000 units):
//   128 workgroups 4.0 / 3.8, 8.5 / 9.4, 18.0 / 20.4;  256 4.0 / 3.9, 9.4 / 9.8, 19.6 / 21.6;  264 5.7 / 4.2, 15.5 / 14.1, 33.6 / 30.7;
//   512 6.0 / 4.4, 16.7 / 15.1, 36.9 / 33.0;  2048 17.8 / 9.3, 58 / 44, 171 / 147
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void mlp2_logits_ce_kernel(const float *__restrict__ hid,
                                                             const float *__restrict__ theta, long long P,
                                                             long long oW2, long long ob2,
                                                             const int *__restrict__ label,
                                                             float *__restrict__ dlogit,
                                                             float *__restrict__ part,
                                                             int B, int dh, int ldh, int C)
{
    __shared__ double dpart[WAVES][4][64];
    __shared__ float2 row_out[4][64];                    // a lane's dlogit and its row's loss
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r = lane & 15, q = lane >> 4;
    const int k = blockIdx.y, row0 = blockIdx.x * 16;
    const float *A = hid + (long long)k * B * ldh;
    const float *W = theta + (long long)k * P + oW2;
    const int ng = (dh + 15) / 16, ngw = (ng + WAVES - 1) / WAVES;
    const int g0 = w * ngw, g1 = min(ng, g0 + ngw);
    const int arow = row0 + r;

    // lane l supplies A[row l%16][k l/16] and B[k l/16][column l%16] of an instruction; a float4 of a
    // row of hid along k feeds four instructions, with the matching four rows of W2
    struct Frag { float a[4], b[4]; };
    auto gload = [&](int g, Frag &f) {
        const int kk = g * 16 + 4 * q;
        const float *ar = A + (long long)arow * ldh + kk;
        if (arow < B && kk + 3 < dh) {
            const float4 v = *(const float4 *)ar;
            f.a[0] = v.x; f.a[1] = v.y; f.a[2] = v.z; f.a[3] = v.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) f.a[j] = (arow < B && kk + j < dh) ? ar[j] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) f.b[j] = (r < C && kk + j < dh) ? W[(long long)(kk + j) * C + r] : 0.f;
    };
    f64x4_t acc;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = 0.0;
    constexpr int PF = 4;
    Frag fr[PF];
#pragma unroll
    for (int u = 0; u < PF; ++u)
        if (g0 + u < g1) gload(g0 + u, fr[u]);
    for (int gb = g0; gb < g1; gb += PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int g = gb + u;                   // uniform over the wavefront
            if (g < g1) {
                const Frag f = fr[u];
                if (g + PF < g1) gload(g + PF, fr[u]);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)f.a[j], (double)f.b[j], acc, 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) dpart[w][e][lane] = acc[e];
    __syncthreads();
    // accumulator element e of lane l is the logit of sample row0 + 4e + l/16, class l%16; wavefront e < 4 goes on with it
    if (w < 4) {
        double z = dpart[0][w][lane];
#pragma unroll
        for (int g = 1; g < WAVES; ++g) z += dpart[g][w][lane];
        const bool cin = r < C;
        const int row = row0 + 4 * w + q;
        const bool rin = row < B;
        z = cin ? z + (double)theta[(long long)k * P + ob2 + r] : -1.7e308;
        const double mx = row_max(z);
        const float zs = cin ? (float)(z - mx) : 0.f;
        const float ex = cin ? expf(zs) : 0.f;
        const float se = row_sum(ex);
        const int y = rin ? label[(long long)k * B + row] : -1;
        const float zy = row_sum(r == y ? zs : 0.f);
        const float dz = (ex * (1.0f / se) - (r == y ? 1.f : 0.f)) * (1.0f / (float)B);
        if (rin && cin) dlogit[((long long)k * B + row) * C + r] = dz;
        row_out[w][lane] = make_float2(rin && cin ? dz : 0.f, rin ? logf(se) - zy : 0.f);
    }
    __syncthreads();
    if (w > 0) return;
    float cs = 0.f, ls = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) { cs += row_out[e][lane].x; ls += row_out[e][lane].y; }
    cs += __shfl_xor(cs, 16, 64); cs += __shfl_xor(cs, 32, 64);
    ls += __shfl_xor(ls, 16, 64); ls += __shfl_xor(ls, 32, 64);
    float *pt = part + ((long long)k * gridDim.x + blockIdx.x) * 17;
    if (lane < 16) pt[lane] = cs;
    if (lane == 0) pt[16] = ls;
}

// Output layer backward for at most 16 classes, one workgroup per UNITS hidden units of a worker:
// gW2[j][c] = sum_i hid[i][j] dlogit[i][c], dhid[i][j] = [hid[i][j] > 0] sum_c dlogit[i][c] W2[j][c],
// gb1[j] = sum_i dhid[i][j]; a thread owns a hidden unit and every SHARES-th sample (its loads of hid go
// out eight at a time before the first is used), the SHARES partial sums are added pairwise
// through LDS.  The first workgroup of a worker also adds up the tiles of
// mlp2_logits_ce_kernel: gb2 and the mean cross-entropy.  (These were three launches of the tiled
// GEMM and a column-sum kernel, 5 to 9 us each whatever they did.)  32 units while each workgroup has a compute unit to itself, 64
// beyond: every workgroup stages all of dlogit, and two on a compute unit do so one behind the other (us, 32 / 64, 10 classes):
//   8 x 1024 units, 128 samples (256 workgroups of 32) 8.2 / 9.4;  8 x 1056 (264) 12.0 / 10.4;  16 x 1024 (512) 15.4 / 10.8;
//   4 x 2048, 512 samples 22.5 / 29.2;  16 x 4096, 512 samples 120 / 101;  16 classes, 16 x 1024, 32 samples 15.4 / 10.0
template <int UNITS>
__global__ __launch_bounds__(512) void mlp2_out_bwd_kernel(const float *__restrict__ hid,
                                                           const float *__restrict__ dlogit,
                                                           const float *__restrict__ theta,
                                                           float *__restrict__ dhid, float *__restrict__ g,
                                                           long long P, long long oW2, long long ob1, long long ob2,
                                                           const float *__restrict__ part, int tiles,
                                                           float *__restrict__ loss, int B, int dh, int ldh, int C)
{
    __shared__ __attribute__((aligned(16))) float dl_s[128][16];
    constexpr int SHARES = 512 / UNITS;
    __shared__ float red[SHARES][UNITS][17];
    const int tid = threadIdx.x, tj = tid % UNITS, ti = tid / UNITS;
    const int k = blockIdx.y, j0 = blockIdx.x * UNITS, j = j0 + tj;
    const bool jin = j < dh;
    float w2[16], gw[16], cs = 0.f;
#pragma unroll
    for (int c = 0; c < 16; ++c) {
        w2[c] = (jin && c < C) ? theta[(long long)k * P + oW2 + (long long)j * C + c] : 0.f;
        gw[c] = 0.f;
    }
    const float *hk = hid + (long long)k * B * ldh;
    float *dk = dhid + (long long)k * B * ldh;
    for (int i0 = 0; i0 < B; i0 += 128) {
        __syncthreads();
        for (int idx = tid; idx < 128 * 16; idx += 512) {
            const int rr = idx >> 4, c = idx & 15;
            dl_s[rr][c] = (i0 + rr < B && c < C) ? dlogit[((long long)k * B + i0 + rr) * C + c] : 0.f;
        }
        __syncthreads();
#pragma unroll 1
        for (int part8 = 0; part8 < 128 / SHARES; part8 += 8) {
            float hv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + ti + SHARES * (part8 + u);
                hv[u] = (jin && i < B) ? hk[(long long)i * ldh + j] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int rr = ti + SHARES * (part8 + u), i = i0 + rr;
                const float4 *dl4 = (const float4 *)dl_s[rr];
                const float4 x0 = dl4[0], x1 = dl4[1], x2 = dl4[2], x3 = dl4[3];
                const float dl[16] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w,
                                      x2.x, x2.y, x2.z, x2.w, x3.x, x3.y, x3.z, x3.w};
                float d = 0.f;
#pragma unroll
                for (int c = 0; c < 16; ++c) d = fmaf(dl[c], w2[c], d);
                d = hv[u] > 0.f ? d : 0.f;
                if (jin && i < B) dk[(long long)i * ldh + j] = d;
                cs += d;
#pragma unroll
                for (int c = 0; c < 16; ++c) gw[c] = fmaf(hv[u], dl[c], gw[c]);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < 16; ++c) red[ti][tj][c] = gw[c];
    red[ti][tj][16] = cs;
    __syncthreads();
    float *gk = g + (long long)k * P;
    for (int idx = tid; idx < UNITS * 17; idx += 512) {
        const int jj = idx / 17, c = idx - jj * 17;
        float v[SHARES];
#pragma unroll
        for (int t = 0; t < SHARES; ++t) v[t] = red[t][jj][c];
#pragma unroll
        for (int n = SHARES / 2; n >= 1; n >>= 1)
#pragma unroll
            for (int t = 0; t < n; ++t) v[t] += v[t + n];
        if (j0 + jj < dh) {
            if (c == 16) gk[ob1 + j0 + jj] = v[0];
            else if (c < C) gk[oW2 + (long long)(j0 + jj) * C + c] = v[0];
        }
    }
    if (blockIdx.x == 0 && tid < 17) {
        float v = 0.f;
        for (int t = 0; t < tiles; ++t) v += part[((long long)k * tiles + t) * 17 + tid];
        if (tid == 16) loss[k] = v * (1.0f / (float)B);
        else if (tid < C) gk[ob2 + tid] = v;
    }
}

hipError_t launch_mlp2_grad(const ModelDims &d, const float *theta, float *g, const float *means,
                            void *ws, float *loss, const DevState *st, hipStream_t s)
{
    const long long B = d.B, di = d.d_in, dh = d.d_hidden, dz = d.d_out, P = d.P;
    const int K = d.K;
    Mlp2Ws w = carve(d, ws, nullptr);
    const long long oW1 = 0, ob1 = di * dh, oW2 = ob1 + dh, ob2 = oW2 + dh * dz;
    hipError_t e;

    // Sample(): labels and inputs
    {
        long long bx = ((B * di + 3) / 4 + 63) / 64;
        if (bx > 0x7FFFFFFFll) bx = 0x7FFFFFFFll;
        mlp2_sample_kernel<<<dim3((unsigned)bx, (unsigned)K), 64, 0, s>>>(w.X, w.label, means, B, di, w.ldx, (uint32_t)dz,
                                                                        (float)d.data_sigma, d.seed, st);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    // forward
    GemmArgs a{};
    a.A = w.X; a.lda = w.ldx; a.sA = B * w.ldx;
    a.B = theta + oW1; a.ldb = dh; a.sB = P;
    a.C = w.hid; a.ldc = w.ldh; a.sC = B * w.ldh;
    a.M = (int)B; a.N = (int)dh; a.Kd = (int)di; a.bias = theta + ob1; a.sBias = P;
    if ((e = launch_dgemm_nn<EPI_BIAS_RELU>(a, K, s)) != hipSuccess) return e;   // double accumulation

    if (dz <= 16) {
        // logits, softmax and loss in one launch; gW2, dhid, gb1 (and the sums that finish gb2 and
        // the loss) in a second
        const int tiles = (int)((B + 15) / 16);
        const bool many = (long long)tiles * K > 256;
        auto logits = many ? mlp2_logits_ce_kernel<8> : mlp2_logits_ce_kernel<16>;
        logits<<<dim3((unsigned)tiles, (unsigned)K), many ? 512 : 1024, 0, s>>>(
            w.hid, theta, P, oW2, ob2, w.label, w.logit, w.part, (int)B, (int)dh, (int)w.ldh, (int)dz);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        const bool small = (dh + 31) / 32 * K <= 256;
        auto back = small ? mlp2_out_bwd_kernel<32> : mlp2_out_bwd_kernel<64>;
        back<<<dim3((unsigned)(small ? (dh + 31) / 32 : (dh + 63) / 64), (unsigned)K), 512, 0, s>>>(
            w.hid, w.logit, theta, w.dhid, g, P, oW2, ob1, ob2, w.part, tiles, loss, (int)B, (int)dh, (int)w.ldh, (int)dz);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    } else {
        a = GemmArgs{};
        a.A = w.hid; a.lda = w.ldh; a.sA = B * w.ldh;
        a.B = theta + oW2; a.ldb = dz; a.sB = P;
        a.C = w.logit; a.ldc = w.ldz; a.sC = B * w.ldz;
        a.M = (int)B; a.N = (int)dz; a.Kd = (int)dh; a.bias = theta + ob2; a.sBias = P;
        if ((e = launch_dgemm_nn<EPI_BIAS>(a, K, s)) != hipSuccess) return e;
        mlp2_softmax_ce_kernel<<<dim3((unsigned)((B + 3) / 4), (unsigned)K), 256, 0, s>>>(w.logit, w.label, w.part, B, (int)dz, w.ldz);
        if ((e = hipGetLastError()) != hipSuccess) return e;

        // backward; w.logit now holds d loss / d logits
        a = GemmArgs{};                                        // gW2 = hid^T dlogits
        a.A = w.hid; a.lda = w.ldh; a.sA = B * w.ldh;
        a.B = w.logit; a.ldb = w.ldz; a.sB = B * w.ldz;
        a.C = g + oW2; a.ldc = dz; a.sC = P;
        a.M = (int)dh; a.N = (int)dz; a.Kd = (int)B;
        a.colsum = g + ob2; a.sCol = P;                        // gb2, and the mean cross-entropy
        a.part = w.part; a.n_part = (int)B; a.part_out = loss; a.part_scale = 1.0f / (float)B;
        GemmArgs h{};                                          // dhid = (dlogits W2^T) * [hid > 0]
        h.A = w.logit; h.lda = w.ldz; h.sA = B * w.ldz;
        h.B = theta + oW2; h.ldb = dz; h.sB = P;               // (b2 lies behind W2's last row)
        h.C = w.dhid; h.ldc = w.ldh; h.sC = B * w.ldh;
        h.M = (int)B; h.N = (int)dh; h.Kd = (int)dz; h.aux = w.hid;
        if ((e = launch_sgemm_pair<EPI_MASK_POS>(a, h, K, s)) != hipSuccess) return e;
    }

    a = GemmArgs{};                                        // gW1 = X^T dhid
    a.A = w.X; a.lda = w.ldx; a.sA = B * w.ldx;
    a.B = w.dhid; a.ldb = w.ldh; a.sB = B * w.ldh;
    a.C = g + oW1; a.ldc = dh; a.sC = P;
    a.M = (int)di; a.N = (int)dh; a.Kd = (int)B;
    if (dz > 16) { a.colsum = g + ob1; a.sCol = P; }       // gb1 (else the output layer's backward kernel has done it)
    return launch_sgemm_tn(a, K, s);
}

}  // namespace qsr
