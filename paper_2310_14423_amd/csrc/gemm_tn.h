// gemm_tn.h -- batched bf16 "TN" GEMM for gfx950: the weight gradients of the residual-MLP workload,
//
//     C[z][m][n] = sum_k A[z][k][m] * B[z][k][n]      (both operands stored [k][feature], k = token)
//
// so the 8 consecutive k a lane of the MFMA needs lie in 8 different rows.  The stages are kept in
// LDS as they are in memory (tokens x features) and the fragments are fetched with the gfx950 LDS
// transpose read (ds_read_b64_tr_b16): within each group of 16 lanes, lane j receives element
// j%4 of the 64-bit words addressed by lanes j/4, j/4+4, j/4+8, j/4+12 of the group (checked on
// the hardware).  Pointing lane r = q + 4e of a group at token e, features 4q..4q+3 of a
// 4-token x 16-feature block therefore hands lane j feature j and the 4 tokens in order; two
// such reads give the 8 k values of an MFMA operand, and the four groups of a wavefront cover
// 16 features x 32 tokens in exactly the operand layout of v_mfma_f32_16x16x32_bf16 (gemm_bf16.h).
//
//  * Stages of 32 tokens are copied global -> LDS directly (global_load_lds_dwordx4) into a ring of NS
//    buffers, NS ahead, LDS keeping [32-feature column block][32 tokens][32 features], with the two halves of a token's
//    64 bytes exchanged in every second group of 8 tokens: two groups of lanes read 8 tokens apart at the same time,
//    which are a multiple of all banks apart.  Token rows beyond K are read from a block of zeros.
//  * The order of the main loop is pinned as in gemm_bf16.h: LDS reads and copies go out one or two at
//    a time between MFMAs, one barrier per stage.  (Two wavefront groups a phase apart, one
//    multiplying while the other fetches, with two barriers per stage: 468 us against 407 us at 8 x 12608
//    tokens x 768 x 3072, same box, both with 32x32x16 instructions; 386 with 16x16x32, which take less of the chip's power.)
//  * Large problems: tiles of 192 x 384 (wavefront 96 x 96).  768 x 3072 outputs per worker are 32
//    such tiles, so 8 workers fill the 256 compute units exactly once.  The reduction of
//    problems with fewer tiles can be cut into ranges (TnGroup::split): each (tile, range) is a
//    workgroup of its own; the caller adds the partial results up in a fixed order.
//  * Small problems: tiles of 64 x 64 whose reduction is shared by KG = 4 groups of four wavefronts in one
//    workgroup, each with its own ring on a quarter of the tokens; the groups' results are added in
//    order through LDS, with no second launch.
//  * Tile order: worker, block of the model, problem, panels of 4 N-tiles, M-tile, N-tile inside the panel; each XCD (workgroup id
//    mod 8) takes a contiguous eighth of that order: one XCD's L2 sees one worker's activations.
//  * Bias gradients (column sums of B over the tokens) come from the B fragments the wavefronts of the
//    first tile row already hold for their MFMAs: one bf16 dot product with ones per register pair.
//
// lda/ldb must be multiples of 8 elements, M and N multiples of 64 (ragged against the tile: operand
// columns are clamped on load, the epilogue is bounds-checked); K may be ragged.
#pragma once
#include <type_traits>

#include "gemm_bf16.h"
#include "qsr_internal.h"

namespace qsr {

struct EpiF32 {                  // C = acc, rows of ldc
    float *C; long long ldc;
    static constexpr int VEC = 4;
    typedef NoAux Aux;
    typedef EpiPtr<float, false> Lane;
    __device__ Lane lane(int, int row, int col, int r, int c) const { return Lane(C, ldc, row, col, r, c); }
    __device__ Aux pre(const Lane &, int) const { return Aux{}; }
    __device__ void operator()(const Lane &l, int dr, const float (&v)[4], const Aux &) const
    {
        st_nt4((float4 *)l.at(dr), make_float4(v[0], v[1], v[2], v[3]));
    }
};

// One weight gradient of a launch, of every block (l) and worker: A and B as above, block and worker strides in
// elements, blkA / blkB: the operand is stored in 32-token x 32-feature blocks (gemm_bf16.h); lda / ldb then hold
// its feature count.  A 1 KiB chunk of a stage (16 tokens x 32 features of one column block) is then 1 KiB of
// consecutive memory; row-major it is 16 pieces of 64 B a whole row apart.  Either way a stage lies 32 * ld elements
// behind the one before.
struct TnProblem {
    const bf16_t *A, *B;
    long long lda, ldb, sA, sB, lA, lB;
    long long off, off_colsum;             // of the product (rows of N) and of B's column sums in a worker's output
    int M, N, blkA, blkB;
    int first;                             // first tile among a block's
};
// A launch: out[worker * s_out + l * l_out + off + m * N + n].  split > 1: the reduction is cut into `split` ranges of
// k_chunk tokens (a multiple of 32), and range s of worker z takes the place of worker z * split + s.
// Several weight gradients share a launch because most leave a last round of the chip half empty by themselves:
// 8 x 12608 tokens, q|k|v projection (192 tiles of 192 x 384 for 256 compute units) and output projection (64).
constexpr int TN_PROBLEMS = 4;
struct TnGroup {
    TnProblem p[TN_PROBLEMS];
    int n, n_l, per_l;                     // problems, blocks, tiles of a block
    int K, split, k_chunk;                 // tokens and their ranges
    const bf16_t *zeros;                   // 64 bytes of zeros, read in place of token rows beyond a range
    float *out; long long s_out, l_out;
};

template <int BM, int BN, int WM, int WN, int KG, int WPS, int NS>
__global__ __launch_bounds__(WM * WN * KG * 64, WPS) void gemm_tn_kernel(TnGroup g, int Z)
{
    constexpr int BK = 32, NW = WM * WN;                          // wavefronts of a group
    constexpr int TM = BM / WM / 16, TN = BN / WN / 16, MM = TM * TN;
    constexpr int HA = TM / 2, HB = TM - HA;                      // rows of the tile's blocks on either side of a stage's barrier
    constexpr int PANEL = 4;                                      // N-tiles per panel of the tile order
    constexpr int STAGE = (BM + BN) * BK;                         // elements
    constexpr int CA = BM / 16, CHUNKS = (BM + BN) / 16;          // 1 KiB chunks per stage
    constexpr int CPW = (CHUNKS + NW - 1) / NW;                   // ... and wavefront (the last ones may have one less)
    extern __shared__ __attribute__((aligned(1024))) unsigned char gemm_smem[];

    const int tid = threadIdx.x, lane = tid & 63, wave_wg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave_wg / NW, wave = wave_wg % NW;
    const int wm = wave / WN, wn = wave % WN;
    const int split = g.split > 1 ? g.split : 1;                  // ranges of the reduction, each a work item
    const int per_z = g.per_l * g.n_l;
    int f = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    if (f >= Z * split * per_z) return;
    const int zz = f / per_z;                                     // worker * split + range
    f -= zz * per_z;
    const int l = f / g.per_l;
    f -= l * g.per_l;
    int e = 0;
    while (e + 1 < g.n && f >= g.p[e + 1].first) ++e;
    const TnProblem &p = g.p[e];
    f -= p.first;
    const int nx = (p.N + BN - 1) / BN, ny = (p.M + BM - 1) / BM;
    const int pn = f / (ny * PANEL);
    f -= pn * ny * PANEL;
    const int bw = min(PANEL, nx - pn * PANEL);
    const int my = f / bw;
    const int m0 = my * BM, n0 = (pn * PANEL + f - my * bw) * BN;
    float *out = g.out + (long long)zz * g.s_out + l * g.l_out;

    // this group's tokens [k_begin, k_end), and the stages every group walks (a group that runs out
    // multiplies zeros)
    const int z = zz / split, r0 = (zz - z * split) * (split > 1 ? g.k_chunk : 0);
    const int r1 = split > 1 ? min(g.K, r0 + g.k_chunk) : g.K;
    const int nk = ((r1 - r0 + BK - 1) / BK + KG - 1) / KG;
    const int k_begin = r0 + grp * nk * BK, k_end = min(r1, k_begin + nk * BK);

    // ---- copies: chunk c of a stage is 1 KiB of LDS (16 tokens x 32 features of one column block)
    bf16_t *ring = (bf16_t *)gemm_smem + grp * NS * STAGE;
    const bf16_t *src[CPW];
    const bf16_t *A = p.A + (long long)z * p.sA + l * p.lA + (long long)k_begin * p.lda;    // k_begin is a multiple of 32:
    const bf16_t *B = p.B + (long long)z * p.sB + l * p.lB + (long long)k_begin * p.ldb;    // the first block row of the range
    const bool blkA = p.blkA != 0, blkB = p.blkB != 0;
    const int tok = lane >> 2;
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        const int c = i * NW + wave;
        const bool isA = c < CA;
        const int cc = isA ? c : c - CA, t = (cc & 1) * 16 + tok;                // token inside the stage
        const int fc = min((isA ? m0 : n0) + (cc >> 1) * 32, (isA ? p.M : p.N) - 32) + ((lane & 3) ^ ((tok >> 3) << 1)) * 8;
        if (isA) src[i] = blkA ? A + (long long)(fc >> 5) * 1024 + t * 32 + (fc & 31) : A + (long long)t * p.lda + fc;
        else src[i] = blkB ? B + (long long)(fc >> 5) * 1024 + t * 32 + (fc & 31) : B + (long long)t * p.ldb + fc;
    }
    const long long stepA = (long long)BK * p.lda, stepB = (long long)BK * p.ldb;   // elements per stage
    const unsigned lds_ring = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)ring;
    int d_stage = 0, d_row = k_begin;                 // buffer and first token of the next stage to copy
    auto issue = [&](int i) {
        const int c = i * NW + wave;
        if (CHUNKS % NW == 0 || c < CHUNKS) {
            const bf16_t *q = src[i];
            if (d_row + BK > k_end) {                 // the range's last stage, or one beyond it
                const int cc = c < CA ? c : c - CA;
                if (d_row + (cc & 1) * 16 + tok >= k_end) q = g.zeros + (lane & 3) * 8;
            }
            // as asm: behind the builtin, the compiler takes every transpose read for a possible reader of the copies
            // in flight and waits for all of them first.  The s_nop is the wait state that such a copy needs behind a
            // write of m0 (the compiler sets m0 right before the statement, and counts wait states for its own copies only).
            const unsigned dst = __builtin_amdgcn_readfirstlane(lds_ring + d_stage * (STAGE * 2) + c * 1024);
            asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "{m0}"(dst), "v"(q) : "memory");
            src[i] += c < CA ? stepA : stepB;
        }
    };
    auto issued = [&]() { d_stage = d_stage + 1 == NS ? 0 : d_stage + 1; d_row += BK; };
    const bool short_wave = CHUNKS % NW != 0 && (CPW - 1) * NW + wave >= CHUNKS;

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float csum[TN];                                   // column sums of B: lane l has 8 tokens of column l % 16 per fragment
#pragma unroll
    for (int j = 0; j < TN; ++j) csum[j] = 0.f;
    const bool colsum_wg = m0 == 0;
    const bool do_colsum = colsum_wg && wm == 0;

    bf16x8 fa[TM], fb[TN];                            // fragments of a stage: 16 features x 32 tokens
    // lane's place in the transpose reads inside a 32-token x 32-feature block, for either half of the features
    const int g16 = lane >> 4, r16 = lane & 15;
    const int lane_tok = (g16 * 8 + (r16 >> 2)) * 32 + (r16 & 3) * 4;
    const int lane_half[2] = {lane_tok + (g16 & 1) * 16, lane_tok + ((g16 & 1) ^ 1) * 16};
    auto frag = [&](const bf16_t *side, int i) {      // side: a wavefront's column blocks of a stage, 32 features each
        typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
        const bf16_t *q0 = side + (i >> 1) * 1024 + lane_half[i & 1];
        union { struct { s16x4 a, b; } s; bf16x8 v; } u;
        u.s.a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)q0);
        u.s.b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(q0 + 4 * 32));
        return u.v;
    };
    auto read_a = [&](int stage, int i) { fa[i] = frag(ring + stage * STAGE + wm * TM * 512, i); };
    auto read_b = [&](int stage, int j) { fb[j] = frag(ring + stage * STAGE + BM * BK + wn * TN * 512, j); };
    auto multiply = [&](int i, int j) { acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0); };
    auto add_columns = [&]() {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bf16x2 two = {fb[j][2 * e], fb[j][2 * e + 1]};
                csum[j] = __builtin_amdgcn_fdot2_f32_bf16(two, ones, csum[j], false);
            }
    };
    auto barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // waits until at most `stages` of this wavefront's stage copies are outstanding, and for its LDS reads
    auto wait = [&](auto stages) {
        constexpr int FULL = CPW * decltype(stages)::value, SHORT = (CPW - 1) * decltype(stages)::value;
        if (short_wave) __builtin_amdgcn_s_waitcnt(0x0070 | (SHORT & 15) | ((SHORT >> 4) << 14));
        else __builtin_amdgcn_s_waitcnt(0x0070 | (FULL & 15) | ((FULL >> 4) << 14));
    };

#pragma unroll
    for (int s = 0; s < NS; ++s)
        if (s < nk) {
#pragma unroll
            for (int i = 0; i < CPW; ++i) issue(i);
            issued();
        }
    if (nk >= NS) wait(std::integral_constant<int, NS - 1>{});
    else wait(std::integral_constant<int, 0>{});
    barrier();
    int cur = 0;
#pragma unroll
    for (int i = 0; i < HA; ++i) read_a(0, i);
#pragma unroll
    for (int j = 0; j < TN - 1; ++j) read_b(0, j);
    // With scalar loads (the epilogue's arguments) in flight at its top, which complete in any order, the loop would wait for all
    // LDS reads at its first MFMA.
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F);
    auto stage = [&](auto last_c, auto issue_c, auto left) {      // the order of gemm_bf16.h
        constexpr bool LAST = decltype(last_c)::value, ISSUE = decltype(issue_c)::value;
        constexpr int MA = HA * TN, MB = HB * TN;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < MA; ++m) {
            const int j = m / HA, i = j & 1 ? HA - 1 - m % HA : m % HA;
            multiply(i, j);
            if (m == 0) read_b(cur, TN - 1);
            else if (m <= HB) read_a(cur, HA + m - 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (do_colsum) add_columns();
        if (!LAST) {
            wait(left);
            barrier();
            cur = cur + 1 == NS ? 0 : cur + 1;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            const int j = m / HB, i = HA + (j & 1 ? HB - 1 - m % HB : m % HB);
            multiply(i, j);
            if (!LAST) {
                if (m < HA) read_a(cur, m);
                if (m % HB == HB - 1 && j < TN - 1) read_b(cur, j);
            }
#pragma unroll
            for (int c = 0; c < CPW; ++c)
                if (!LAST && ISSUE && (CPW <= MB ? MB - CPW + c : c * MB / CPW) == m) issue(c);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!LAST && ISSUE) issued();
    };
    // stages outstanding at a wait: kt + 2 .. kt + NS - 1 while that many exist
    int kt = 0;
    for (; kt + NS < nk; ++kt) stage(std::false_type{}, std::true_type{}, std::integral_constant<int, NS - 2>{});
    if (kt + NS == nk && kt + 1 < nk) { stage(std::false_type{}, std::false_type{}, std::integral_constant<int, NS - 2>{}); ++kt; }
    for (; kt + 1 < nk; ++kt) stage(std::false_type{}, std::false_type{}, std::integral_constant<int, 0>{});
    stage(std::true_type{}, std::false_type{}, std::integral_constant<int, 0>{});
    __syncthreads();                                  // everyone is through with the rings

    // The ring's memory from here on: epilogue staging, column sums [group][token quarter][column], the other groups'
    // accumulators
    constexpr int STAGING = NW * StagedTile<TN * 16>::FLOATS;
    constexpr int COLS = KG * 4 * BN, ACCS = (KG - 1) * NW * MM * 4 * 64;
    static_assert((STAGING + COLS + ACCS) * 4 <= KG * NS * STAGE * 2, "epilogue inside the rings");
    float *cols = (float *)gemm_smem + STAGING, *accs = cols + COLS;
    if (do_colsum) {
#pragma unroll
        for (int j = 0; j < TN; ++j) cols[(grp * 4 + (lane >> 4)) * BN + wn * (BN / WN) + j * 16 + (lane & 15)] = csum[j];
    }
    if (KG > 1 && grp > 0) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    accs[((((grp - 1) * NW + wave) * MM + i * TN + j) * 4 + e) * 64 + lane] = acc[i][j][e];
    }
    __syncthreads();
    if (colsum_wg && tid < BN && n0 + tid < p.N) {
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < KG * 4; ++q) s += cols[q * BN + tid];
        out[p.off_colsum + n0 + tid] = s;
    }
    if (KG > 1) {
        if (grp > 0) return;
#pragma unroll
        for (int gg = 0; gg < KG - 1; ++gg)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[i][j][e] += accs[(((gg * NW + wave) * MM + i * TN + j) * 4 + e) * 64 + lane];
    }
    const EpiF32 epi{out + p.off, p.N};
    epilogue_via_lds<TM, TN>(acc, (float *)gemm_smem + wave * StagedTile<TN * 16>::FLOATS, lane,
                             m0 + wm * TM * 16, n0 + wn * TN * 16, p.M, p.N, 0, 0, epi, []() {});
}

// Whether launch_gemm_tn can take the group (blocked operands: 32-column blocks; the ranges of a split reduction
// start at multiples of 32 tokens).
inline bool gemm_tn_supports(const TnGroup &g)
{
    if (g.n < 1 || g.n > TN_PROBLEMS || g.n_l < 1 || g.K < 1 || g.zeros == nullptr) return false;
    if (g.split > 1 && (g.k_chunk < 32 || g.k_chunk % 32 != 0 || (long long)(g.split - 1) * g.k_chunk >= g.K)) return false;
    for (int e = 0; e < g.n; ++e) {
        const TnProblem &p = g.p[e];
        if (p.lda % (p.blkA ? 32 : 8) != 0 || p.ldb % (p.blkB ? 32 : 8) != 0) return false;
        if (p.M % 64 != 0 || p.N % 64 != 0 || p.M < 64 || p.N < 64) return false;
    }
    return true;
}

// compute units of the current device
inline int gemm_cu_count()
{
    static int n_cu = 0;                      // contexts are not thread-safe; one GPU per process
    if (n_cu == 0) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 8)
            n_cu = 256;
    }
    return n_cu;
}

template <int BM, int BN, int WM, int WN, int KG, int WPS, int NS>
inline hipError_t launch_gemm_tn(TnGroup g, int batch, hipStream_t s)
{
    if (!gemm_tn_supports(g)) return hipErrorInvalidValue;
    constexpr size_t smem = (size_t)KG * NS * (BM + BN) * 32 * 2;
    static_assert(smem <= 160 * 1024, "rings do not fit the 160 KB LDS");
    auto kern = gemm_tn_kernel<BM, BN, WM, WN, KG, WPS, NS>;
    static bool lds_limit_raised = false;     // per instantiation; contexts are not thread-safe
    if (smem > 64 * 1024 && !lds_limit_raised) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        lds_limit_raised = true;
    }
    long long per_l = 0;
    for (int e = 0; e < g.n; ++e) {
        g.p[e].first = (int)per_l;
        per_l += (long long)((g.p[e].M + BM - 1) / BM) * ((g.p[e].N + BN - 1) / BN);
    }
    g.per_l = (int)per_l;
    const long long items = per_l * g.n_l * batch * (g.split > 1 ? g.split : 1);
    if ((items + 7) / 8 * 8 * (WM * WN * KG * 64) >= 1ll << 32) return hipErrorInvalidValue;   // threads of a launch
    kern<<<(unsigned)((items + 7) / 8 * 8), WM * WN * KG * 64, smem, s>>>(g, batch);
    return hipGetLastError();
}

}  // namespace qsr
