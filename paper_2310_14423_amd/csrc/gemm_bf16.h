// gemm_bf16.h -- batched bf16 x bf16 -> fp32 GEMM on the gfx950 matrix cores, "NT" form:
//
//     C[z][m][n] = sum_k A[z][m][k] * B[z][n][k]        (both operands K-contiguous)
//
// which is the operand order the MFMA instruction wants: v_mfma_f32_32x32x16_bf16 takes, per
// lane, 8 consecutive k of one row of A and 8 consecutive k of one column of B.  Lane layout
// (checked on the hardware): lane l holds A[row l%32][k (l/32)*8 .. +7], B[k (l/32)*8 .. +7]
// [col l%32], and accumulator element i is D[(i/4)*8 + (l/32)*4 + i%4][l%32].
//
// Tiling: a workgroup of WM x WN wavefronts computes a BM x BN tile; K is walked in stages of
// 32 through a ring of NS LDS buffers.  The stages are copied global -> LDS directly
// (global_load_lds_dwordx4: no register staging, no LDS store instructions), NS of them ahead (a buffer is
// requested again as soon as its stage has been read); a wavefront waits for its share of the next stage only (a
// counted vmcnt, not 0).  That
// instruction writes 64 lanes x 16 B to 1 KiB of consecutive LDS, so rows are stored unpadded
// (4 pieces of 16 B) and bank conflicts are avoided by an XOR swizzle instead: slot s of row r
// holds piece s ^ ((r >> 2) & 3), which spreads the 128-bit fragment reads of 16 consecutive rows
// over all 64 banks (measured: no conflicts).
// M and N may be ragged: out-of-range rows are clamped to the last valid row on load (they
// only feed accumulator rows that are never stored) and the epilogue is bounds-checked.
// K must be a multiple of 32, N of 64, and lda a multiple of 8 elements (16-byte rows).
//
// The two operands are handed to the instruction in swapped roles (the B rows as its "A", the A
// rows as its "B"), so that it produces the transposed tile: lane l then owns, for token row
// m = l%32, four consecutive output columns n, which is what the epilogue's LDS staging writes
// with 128-bit stores (see epilogue_via_lds).
//
// Operand layout.  Besides plain row-major, a bf16 matrix [R][C] (C a multiple of 32) can be stored
// in blocks of 32 rows x 32 columns, each block 2 KiB contiguous, blocks ordered [row block]
// [column block] (blk_off below).  Both kinds of GEMM then copy consecutive memory: a 256-row x
// 32-deep stage of this kernel's operands is 8 pieces of 2 KiB (one block each) instead of
// 256 pieces of 64 B a whole row (1.5 - 6 KiB) apart, and a 32-token x 192- or 384-feature slab of
// the weight-gradient kernel (gemm_tn.h), which walks the same arrays along their rows, is 12 or
// 24 KiB in one piece instead of 32 pieces; every global -> LDS copy instruction moves 1 KiB of
// consecutive memory.  (Blocks of 256 rows x 32 columns, 32 KiB per slab here, were timed first:
// this kernel gained 3-4 %, the weight-gradient kernel, whose slab was then 2 KiB pieces exactly
// 16 KiB apart, lost 8 %.)  All weights (B operands) are blocked; activations are blocked where
// their producers write them that way (BLKA), row-major otherwise.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace qsr {

// element offset of (r, c) in the blocked layout of an [R][C] matrix; R is padded to 256 rows (the
// tiles of this kernel read whole 256-row panels)
__host__ __device__ __forceinline__ long long blk_off(long long r, long long c, long long C)
{
    return ((r >> 5) * (C >> 5) + (c >> 5)) * 1024 + (r & 31) * 32 + (c & 31);
}
// elements a blocked [R][C] matrix occupies
__host__ __device__ __forceinline__ long long blk_elems(long long R, long long C) { return ((R + 255) >> 8) * 256 * C; }

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct GemmNT {
    const bf16_t *A, *B;
    int M, N, K;
    long long lda, ldb;
    long long sA, sB;      // per-batch strides (elements)
};

// Epilogue.  The MFMA leaves lane l with 4 consecutive columns of row l%32, i.e. one store
// instruction would touch 32 different rows.  Each wavefront therefore passes its tile, 32 rows
// at a time, through a private LDS area (the ring is free by then) and re-reads it so that
// consecutive lanes hold one row's consecutive columns: whole 128- or 256-byte row segments per
// global instruction.  Rows are padded by 16 B: conflict-free both ways.  A lane takes VEC = 8
// consecutive columns where the outputs are bf16 (16-byte accesses) and 4 where they are fp32.
//
// Addresses: an element of a lane is a wavefront-uniform base (worker, tile, row within the tile:
// scalar registers) plus a 32-bit lane offset that is the same for all rows of the tile, so a row
// costs no vector instruction.  (Written with 64-bit element offsets per access, the address
// arithmetic was 8 vector slots per element of the GELU epilogue's 32.)
// The functor provides
//     VEC, Aux
//     Lane lane(z, row, col, r, c)   -- r, c: the lane's row and column relative to the uniform
//                                       (row, col); called once
//     Aux  pre(Lane, dr)             -- loads for the lane's columns, dr rows further down (may be empty);
//                                       requested one 32-row block ahead of their use
//     void operator()(Lane, dr, v[VEC], aux)
// with dr a compile-time constant after unrolling; EpiPtr below does the offsets.
// and, if it has such a member,
//     void finish(Lane, z, unit)     -- at the end; unit: the wavefront's number among the tiles of batch entry z
struct NoAux {};
template <class Epi, class = void> struct EpiHasFinish : std::false_type {};
template <class Epi> struct EpiHasFinish<Epi, std::void_t<decltype(&Epi::finish)>> : std::true_type {};

// One array as the epilogue sees it: uniform base and lane offset.  T elements, row-major with row
// stride ld, or in 32 x 32 blocks (ld the number of columns).  dr, the rows further down, must not
// carry the lane's row over the edge of a 32-row block except in whole blocks: row (uniform) is a
// multiple of 32 and r + dr % 32 < 32 holds for every access.
template <class T, bool BLK>
struct EpiPtr {
    T *base; unsigned off; long long ld;
    __device__ __forceinline__ EpiPtr(T *p, long long ld_, int row, int col, int r, int c) : ld(ld_)
    {
        if (BLK) {
            base = p + ((long long)(row >> 5) * (ld >> 5) + (col >> 5)) * 1024;
            off = (unsigned)((c >> 5) * 1024 + r * 32 + (c & 31));
        } else {
            base = p + (long long)row * ld + col;
            off = (unsigned)(r * (int)ld + c);
        }
    }
    __device__ __forceinline__ T *at(int dr) const
    {
        return base + (BLK ? (long long)(dr >> 5) * (ld >> 5) * 1024 + (dr & 31) * 32 : (long long)dr * ld) + off;
    }
};

// `compute` leaves the tile in acc and says whether this wavefront stores it.  A wavefront with one block of 32 x 32 asks for
// what its epilogue reads ahead of that: with few tiles in flight nothing else hides the latency.
template <int TM, int TN, class Epi, class Compute>
__device__ __forceinline__ void epilogue_via_lds(f32x16 (&acc)[TM][TN], float *stage, int lane,
                                                 int row0, int col0, int M, int N, int z, int unit, const Epi &epi, Compute compute)
{
    constexpr bool EARLY = TM * TN == 1;
    if constexpr (!EARLY) if (!compute()) return;
    constexpr int W = TN * 32, LD = W + 4;             // floats per staged row
    constexpr int VEC = Epi::VEC;
    constexpr int LPR = W / VEC;                       // lanes per row on the way out
    constexpr int RPI = 64 / LPR;                      // rows per read instruction
    constexpr int ITERS = (32 + RPI - 1) / RPI;
    static_assert(32 % RPI == 0, "rows per instruction must divide the block");
    const bool active = 64 % LPR == 0 || lane < RPI * LPR;   // TN = 3: some of the last lanes are idle
    const int r0 = active ? lane / LPR : 0, c = (lane % LPR) * VEC;
    const auto lp = epi.lane(z, row0, col0, r0, c);
    typename Epi::Aux aux[2][ITERS];
    if constexpr (EARLY) {
#pragma unroll
        for (int it = 0; it < ITERS; ++it)
            if (active && row0 + it * RPI + r0 < M && col0 + c < N) aux[0][it] = epi.pre(lp, it * RPI);
        if (!compute()) return;
    }
    auto block = [&](auto full_c, int i) {
        constexpr bool FULL = decltype(full_c)::value;
        auto request = [&](int ib, int buf) {
#pragma unroll
            for (int it = 0; it < ITERS; ++it)
                if (active && (FULL || (row0 + ib * 32 + it * RPI + r0 < M && col0 + c < N)))
                    aux[buf][it] = epi.pre(lp, ib * 32 + it * RPI);
        };
        // What the functor reads from global memory is requested one block ahead, before the stores of
        // the block in between: vector memory operations complete in order, so a wait for loads issued
        // after a block's stores would also wait for those stores.
        if (i == 0 && !EARLY) request(0, 0);
        if (i + 1 < TM) request(i + 1, (i + 1) & 1);
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int eg = 0; eg < 4; ++eg)
                *(float4 *)(stage + (lane & 31) * LD + j * 32 + eg * 8 + (lane >> 5) * 4) =
                    make_float4(acc[i][j][eg * 4 + 0], acc[i][j][eg * 4 + 1], acc[i][j][eg * 4 + 2],
                                acc[i][j][eg * 4 + 3]);
        __builtin_amdgcn_wave_barrier();               // LDS executes a wavefront's accesses in order
        float4 t[ITERS][VEC / 4];                      // all reads of a block go out before the first use
#pragma unroll
        for (int it = 0; it < ITERS; ++it)
#pragma unroll
            for (int u = 0; u < VEC / 4; ++u) t[it][u] = *(const float4 *)(stage + (it * RPI + r0) * LD + c + u * 4);
#pragma unroll
        for (int it = 0; it < ITERS; ++it)
            if (active && (FULL || (row0 + i * 32 + it * RPI + r0 < M && col0 + c < N))) {
                float v[VEC];
#pragma unroll
                for (int u = 0; u < VEC / 4; ++u) {
                    v[u * 4] = t[it][u].x; v[u * 4 + 1] = t[it][u].y; v[u * 4 + 2] = t[it][u].z; v[u * 4 + 3] = t[it][u].w;
                }
                epi(lp, i * 32 + it * RPI, v, aux[i & 1][it]);
            }
        __builtin_amdgcn_wave_barrier();
    };
    // a tile inside the matrix takes no test per row
    if (row0 + TM * 32 <= M && col0 + W <= N) {
#pragma unroll
        for (int i = 0; i < TM; ++i) block(std::true_type{}, i);
    } else {
#pragma unroll
        for (int i = 0; i < TM; ++i) block(std::false_type{}, i);
    }
    if constexpr (EpiHasFinish<Epi>::value) epi.finish(lp, z, unit);
}

// BLKA: A is stored in 32 x 32 blocks (see above); B always is.  In LDS a stage is [BM rows][32 k] of
// A, then [BN rows][32 k] of B, rows of 64 B, slot s of row r holding piece s ^ ((r >> 2) & 3).
// WPS: wavefronts per SIMD the registers are budgeted for.  KG: groups of wavefronts that share a tile's contraction, each
// with a ring of its own on a KG-th of it (K a multiple of 32 KG); the results are added in order through LDS.
template <int BM, int BN, int WM, int WN, int KG, int WPS, int NS, bool BLKA, class Epi>
__global__ __launch_bounds__(WM * WN * KG * 64, WPS) void gemm_nt_bf16_kernel(GemmNT p, Epi epi, int batch)
{
    constexpr int BK = 32, NW = WM * WN;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32, NF = TM + TN, MM = TM * TN;
    constexpr int CA = BM / 16, CB = BN / 16;           // 1 KiB chunks (16 rows x 64 B) per stage
    constexpr int CPW = (CA + CB) / NW;                 // ... and wavefront
    static_assert((CA + CB) % NW == 0 && BM % 32 == 0 && BN % 32 == 0, "chunks / waves");
    constexpr int STAGE = (BM + BN) * BK;
    extern __shared__ __attribute__((aligned(1024))) unsigned char gemm_smem[];

    const int lane = threadIdx.x & 63, wave_wg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = wave_wg / NW, wave = wave_wg % NW;
    bf16_t *smem = (bf16_t *)gemm_smem + grp * NS * STAGE;
    const int wm = wave / WN, wn = wave % WN;
    // Workgroups go to the 8 XCDs round-robin by linear id (the grid's x extent is a multiple of
    // 8).  Tile order: batch entry (worker), then panels of 4 N-tiles, then M-tile, then N-tile
    // inside the panel; each XCD takes a contiguous eighth of that order.  One XCD's L2 then sees
    // one worker's B operand (for 8 workers), and the tiles that run together share their A rows
    // and B rows: 30-45 % fewer bytes fetched into L2 than with the batch as a grid dimension.
    // (Panels of 2, 3, 6 or 12 tiles: the same to 3 %, the narrow ones slower at N = 768.)
    const int nx = (p.N + BN - 1) / BN, ny = (p.M + BM - 1) / BM;
    int tile = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    if (tile >= batch * nx * ny) return;
    const int z = tile / (nx * ny);
    tile -= z * nx * ny;
    constexpr int PANEL = 4;
    const int pn = tile / (ny * PANEL);
    tile -= pn * ny * PANEL;
    const int bw = min(PANEL, nx - pn * PANEL);
    const int by = tile / bw, bx = pn * PANEL + tile - by * bw;
    const int m0 = by * BM, n0 = bx * BN;
    const int nk = p.K / (BK * KG);                    // stages of a group
    const bf16_t *A = p.A + (long long)z * p.sA + (long long)grp * nk * (BLKA ? 1024 : BK);
    const bf16_t *B = p.B + (long long)z * p.sB + (long long)grp * nk * 1024;

    // Per-lane global source of each 1 KiB chunk this wave copies: chunk c is 16 rows, LDS slot
    // (row, s) holds the global piece s ^ ((row >> 2) & 3) of that row.  Blocked operand: half of a
    // 32 x 32 block, consecutive in memory up to that permutation; rows beyond the matrix inside the
    // last 256-row panel are allocated (their values only reach accumulator rows never stored), and
    // every tile shape divides 256.  Row-major A: 16 pieces of 64 B, rows clamped.
    const bf16_t *src[CPW];
    const int piece = ((lane & 3) ^ ((lane >> 4) & 3)) * 8;
    const int blk_lane = (lane >> 2) * 32 + piece;
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        const int c = wave * CPW + i;
        if (c < CA) {
            if (BLKA) src[i] = A + ((long long)((m0 >> 5) + (c >> 1)) * (p.K >> 5)) * 1024 + (c & 1) * 512 + blk_lane;
            else src[i] = A + (long long)min(m0 + c * 16 + (lane >> 2), p.M - 1) * p.lda + piece;
        } else {
            src[i] = B + ((long long)((n0 >> 5) + ((c - CA) >> 1)) * (p.K >> 5)) * 1024 + (c & 1) * 512 + blk_lane;
        }
    }
    typedef __attribute__((address_space(3))) void lds_void;
    typedef __attribute__((address_space(1))) const void glb_void;
    int d_stage = 0;                                    // stage the next copy goes to
    auto issue = [&](int i) {
        const int c = wave * CPW + i;
        __builtin_amdgcn_global_load_lds((glb_void *)src[i], (lds_void *)(smem + d_stage * STAGE + c * 512), 16, 0, 0);
        src[i] += BLKA || c >= CA ? 1024 : BK;
    };
    auto issued = [&]() { d_stage = d_stage + 1 == NS ? 0 : d_stage + 1; };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    bf16x8 fa[2][TM], fb[2][TN];
    int offA[2], offB[2];                               // the lane's place in a stage, per 16-wide k-step
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int pc = ks * 2 + (lane >> 5), r = lane & 31, sw = (pc ^ ((r >> 2) & 3)) * 8;
        offA[ks] = (wm * TM * 32 + r) * 32 + sw;
        offB[ks] = BM * BK + (wn * TN * 32 + r) * 32 + sw;
    }
    // fragment q of a k-step, in the order the multiplications need them: b0, a0, the other b, the other a
    auto read = [&](int stage, int ks, int q) {
        const bf16_t *s = smem + stage * STAGE;
        if (q == 0) fb[ks][0] = *(const bf16x8 *)(s + offB[ks]);
        else if (q == 1) fa[ks][0] = *(const bf16x8 *)(s + offA[ks]);
        else if (q <= TN) fb[ks][q - 1] = *(const bf16x8 *)(s + offB[ks] + (q - 1) * 1024);
        else fa[ks][q - TN] = *(const bf16x8 *)(s + offA[ks] + (q - TN) * 1024);
    };
    auto multiply = [&](int ks, int m) {                // serpentine: neighbours share an operand
        const int i = m / TN, j = (i & 1) ? TN - 1 - m % TN : m % TN;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ks][j], fa[ks][i], acc[i][j], 0, 0, 0);
    };
    // a barrier that no memory access is moved across
    auto barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // vmcnt(left), lgkmcnt(0)
    auto wait = [&](auto left) {
        constexpr int n = decltype(left)::value;
        __builtin_amdgcn_s_waitcnt(0x0070 | (n & 15) | ((n >> 4) << 14));
    };

    // Main loop.  A stage is two k-steps.  While step 0's MFMAs issue, the fragments of step 1 are
    // read; then comes the barrier (everyone's copies of the next stage have landed, everyone is
    // through reading this one); while step 1's MFMAs issue, the fragments of the next stage's step
    // 0 are read and the stage NS further on is requested into the buffer just freed.  The order is
    // pinned instruction by instruction (sched_barrier after every MFMA): one LDS read or one copy
    // between two MFMAs.  Left to the compiler, a k-step's six reads go out in one burst in front
    // of its eight MFMAs and both wavefronts of a SIMD do so together.  Timed on MI355X at
    // 12608 x 768 x 3072, batch 8, same box: bf16 output 465 -> 393 us (K = 3072), main loop alone
    // 430 -> 371 us = 1.28 PFLOP/s; the loop without its copies runs at 1.5-1.6 PFLOP/s, and bare
    // MFMAs on random operands at 1.84 (2.28 on zeros: the clock drops with the power they draw).
    // Neither 3, 4 or 5 stages nor raised wave priority around the MFMAs make a difference; four
    // wavefronts of 128 x 128 (a third fewer LDS reads) ran the same loop in 361-393 us on the same
    // boxes, and lost it again in the epilogues, where one wavefront per SIMD has nothing to hide
    // its waits behind (751 against 631 us with the GELU epilogue).
    auto compute = [&]() -> bool {
#pragma unroll
    for (int s = 0; s < NS; ++s)
        if (s < nk) {
#pragma unroll
            for (int i = 0; i < CPW; ++i) issue(i);
            issued();
        }
    if (nk >= NS) wait(std::integral_constant<int, CPW * (NS - 1)>{});
    else wait(std::integral_constant<int, 0>{});
    barrier();
    int cur = 0;
#pragma unroll
    for (int q = 0; q < NF; ++q) read(0, 0, q);
    auto stage = [&](auto last_c, auto issue_c, auto left) {
        constexpr bool LAST = decltype(last_c)::value, ISSUE = decltype(issue_c)::value;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < MM; ++m) {
            multiply(0, m);
#pragma unroll
            for (int q = 0; q < NF; ++q)
                if ((NF <= MM ? q : q * MM / NF) == m) read(cur, 1, q);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!LAST) {
            wait(left);
            barrier();
            cur = cur + 1 == NS ? 0 : cur + 1;
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int m = 0; m < MM; ++m) {
            multiply(1, m);
#pragma unroll
            for (int q = 0; q < NF; ++q)
                if (!LAST && (NF <= MM ? q : q * MM / NF) == m) read(cur, 0, q);
#pragma unroll
            for (int i = 0; i < CPW; ++i)
                if (!LAST && ISSUE && (CPW <= MM ? MM - CPW + i : i * MM / CPW) == m) issue(i);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!LAST && ISSUE) issued();
    };
    // copies outstanding at a stage's wait: stages kt + 2 .. kt + NS - 1 while that many exist
    int kt = 0;
    for (; kt + NS < nk; ++kt) stage(std::false_type{}, std::true_type{}, std::integral_constant<int, CPW * (NS - 2)>{});
    if (kt + NS == nk && kt + 1 < nk) { stage(std::false_type{}, std::false_type{}, std::integral_constant<int, CPW * (NS - 2)>{}); ++kt; }
    for (; kt + 1 < nk; ++kt) stage(std::false_type{}, std::false_type{}, std::integral_constant<int, 0>{});
    stage(std::true_type{}, std::false_type{}, std::integral_constant<int, 0>{});

        __syncthreads();                               // every wavefront is done with the rings
        if constexpr (KG > 1) {
            constexpr int STAGING = NW * 32 * (TN * 32 + 4);   // floats
            float *accs = (float *)gemm_smem + STAGING;
            if (grp > 0) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int e = 0; e < 16; ++e)
                            accs[((((grp - 1) * NW + wave) * MM + i * TN + j) * 16 + e) * 64 + lane] = acc[i][j][e];
            }
            __syncthreads();
            if (grp > 0) return false;
#pragma unroll
            for (int gg = 0; gg < KG - 1; ++gg)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int e = 0; e < 16; ++e) acc[i][j][e] += accs[(((gg * NW + wave) * MM + i * TN + j) * 16 + e) * 64 + lane];
        }
        return true;
    };
    epilogue_via_lds<TM, TN>(acc, (float *)gemm_smem + wave * (32 * (TN * 32 + 4)), lane, m0 + wm * TM * 32,
                             n0 + wn * TN * 32, p.M, p.N, z, (by * nx + bx) * NW + wave, epi, compute);
}

typedef short s16x4 __attribute__((ext_vector_type(4)));   // operand of the LDS transpose read

template <int BM, int BN, int WM, int WN, int KG, int WPS, int NS, bool BLKA, class Epi>
inline hipError_t launch_gemm_nt(const GemmNT &p, const Epi &epi, int batch, hipStream_t s)
{
    static_assert(256 % BM == 0 && 256 % BN == 0, "blocked operands are allocated in panels of 256 rows");
    if (p.K % (32 * KG) != 0 || p.K < 32 || p.N % 64 != 0) return hipErrorInvalidValue;
    const unsigned tiles = (unsigned)((p.N + BN - 1) / BN) * (unsigned)((p.M + BM - 1) / BM) * (unsigned)batch;
    dim3 grid((tiles + 7) / 8 * 8, 1, 1);
    constexpr size_t ring = (size_t)KG * NS * (BM + BN) * 32 * sizeof(bf16_t);
    constexpr size_t staging = ((size_t)WM * WN * 32 * (BN / WN + 4) + (size_t)(KG - 1) * BM * BN) * sizeof(float);
    constexpr size_t smem = ring > staging ? ring : staging;
    static_assert(smem <= 160 * 1024, "tile does not fit the 160 KB LDS");
    auto kern = gemm_nt_bf16_kernel<BM, BN, WM, WN, KG, WPS, NS, BLKA, Epi>;
    static bool lds_limit_raised = false;     // per instantiation; contexts are not thread-safe
    if (smem > 64 * 1024 && !lds_limit_raised) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        lds_limit_raised = true;
    }
    kern<<<grid, WM * WN * KG * 64, smem, s>>>(p, epi, batch);
    return hipGetLastError();
}

}  // namespace qsr
