// gemm_bf16.h -- batched bf16 x bf16 -> fp32 GEMM on the gfx950 matrix cores, "NT" form:
//
//     C[z][m][n] = sum_k A[z][m][k] * B[z][n][k]        (both operands K-contiguous)
//
// which is the operand order the MFMA instruction wants: v_mfma_f32_16x16x32_bf16 takes, per
// lane, 8 consecutive k of one row of A and 8 consecutive k of one column of B.  Lane layout
// (checked on the hardware): lane l holds A[row l%16][k (l/16)*8 .. +7], B[k (l/16)*8 .. +7]
// [col l%16], and accumulator element i is D[(l/16)*4 + i][l%16].
// The chip runs these products at its power limit, and this instruction takes less of it than
// v_mfma_f32_32x32x16_bf16, which moves twice the accumulators through the registers for half the
// operands: bare on random operands 2120 TFLOP/s against 1830 on MI355X (2440 and 2480 on zeros).
//
// Tiling: a workgroup of WM x WN wavefronts computes a BM x BN tile; K is walked in stages of
// 32 through a ring of NS LDS buffers.  The stages are copied global -> LDS directly
// (global_load_lds_dwordx4: no register staging, no LDS store instructions), NS of them ahead (a buffer is
// requested again as soon as its stage has been read); a wavefront waits for its share of the next stage only (a
// counted vmcnt, not 0).  That
// instruction writes 64 lanes x 16 B to 1 KiB of consecutive LDS, so rows are stored unpadded
// (4 pieces of 16 B) and bank conflicts are avoided by exchanging the halves of every second group of 8 rows: slot s of row r
// holds piece s ^ ((r >> 3) & 1) * 2.  A 128-bit read takes the lanes of a half wavefront in two turns, 0-3, 12-15, 20-27 and
// 4-11, 16-19, 28-31, and so covers all 64 banks in each (measured: no conflicts; with s ^ ((r >> 2) & 3), which suits
// fragments of 32 rows x 16 k, every read conflicts).
// M and N may be ragged: out-of-range rows are clamped to the last valid row on load (they
// only feed accumulator rows that are never stored) and the epilogue is bounds-checked.
// K must be a multiple of 32, N of 64, and lda a multiple of 8 elements (16-byte rows).
//
// The two operands are handed to the instruction in swapped roles (the B rows as its "A", the A
// rows as its "B"), so that it produces the transposed tile: lane l then owns, for token row
// m = l%16, four consecutive output columns n, which is what the epilogue's LDS staging writes
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

#include "nt_plan.h"

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
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct GemmNT {
    const bf16_t *A, *B;
    int M, N, K;
    long long lda, ldb;
    long long sA, sB;      // per-batch strides (elements)
};

// Epilogue.  The MFMA leaves lane l with 4 consecutive columns of row l%16, i.e. one store
// instruction would touch 16 different rows.  Each wavefront therefore passes its tile, 32 rows
// at a time, through a private LDS area (the ring is free by then) and re-reads it so that
// consecutive lanes hold one row's consecutive columns: whole 128- or 256-byte row segments per
// global instruction.  A lane takes VEC = 8 consecutive columns where the outputs are bf16 (16-byte accesses) and 4 where
// they are fp32.  StagedTile says where a row's columns lie, so that there are no bank conflicts either way.
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

// 32 rows of W floats in LDS.  The 16-byte units of rows of 32 or 64 are permuted by the row, which is conflict-free in the
// turns that 128-bit accesses are made in (see the top; with rows padded by 16 bytes instead, a quarter of the LDS cycles of
// the GELU kernel were conflicts); rows of other widths are padded.
template <int W>
struct StagedTile {
    static constexpr bool PERMUTED = W == 32 || W == 64;
    static constexpr int LD = PERMUTED ? W : W + 4, FLOATS = 32 * LD;
    // of the unit of column c (a multiple of 4)
    static __device__ __forceinline__ int at(int row, int c)
    {
        if (!PERMUTED) return row * LD + c;
        return row * LD + ((c >> 2) ^ (W == 64 ? row & 15 : (row >> 1) & 7)) * 4;
    }
};

// `compute` leaves the tile in acc.  A wavefront with one block of 32 x 32 asks for
// what its epilogue reads ahead of that: with few tiles in flight nothing else hides the latency.
// TM x TN blocks of 16 x 16.
template <int TM, int TN, class Epi, class Compute>
__device__ __forceinline__ void epilogue_via_lds(f32x4 (&acc)[TM][TN], float *stage, int lane,
                                                 int row0, int col0, int M, int N, int z, int unit, const Epi &epi, Compute compute)
{
    constexpr bool EARLY = TM * TN == 4;
    if constexpr (!EARLY) compute();
    constexpr int W = TN * 16;                         // floats per staged row
    typedef StagedTile<W> Staged;
    constexpr int VEC = Epi::VEC;
    constexpr int LPR = W / VEC;                       // lanes per row on the way out
    constexpr int RPI = 64 / LPR;                      // rows per read instruction
    constexpr int ITERS = (32 + RPI - 1) / RPI;
    static_assert(32 % RPI == 0, "rows per instruction must divide the block");
    const bool active = 64 % LPR == 0 || lane < RPI * LPR;   // W = 96: some of the last lanes are idle
    const int r0 = active ? lane / LPR : 0, c = (lane % LPR) * VEC;
    const auto lp = epi.lane(z, row0, col0, r0, c);
    typename Epi::Aux aux[2][ITERS];
    if constexpr (EARLY) {
#pragma unroll
        for (int it = 0; it < ITERS; ++it)
            if (active && row0 + it * RPI + r0 < M && col0 + c < N) aux[0][it] = epi.pre(lp, it * RPI);
        compute();
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
        if (i + 1 < TM / 2) request(i + 1, (i + 1) & 1);
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                *(f32x4 *)(stage + Staged::at(h * 16 + (lane & 15), j * 16 + (lane >> 4) * 4)) = acc[2 * i + h][j];
        __builtin_amdgcn_wave_barrier();               // LDS executes a wavefront's accesses in order
        float4 t[ITERS][VEC / 4];                      // all reads of a block go out before the first use
#pragma unroll
        for (int it = 0; it < ITERS; ++it)
#pragma unroll
            for (int u = 0; u < VEC / 4; ++u) t[it][u] = *(const float4 *)(stage + Staged::at(it * RPI + r0, c + u * 4));
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
    if (row0 + TM * 16 <= M && col0 + W <= N) {
#pragma unroll
        for (int i = 0; i < TM / 2; ++i) block(std::true_type{}, i);
    } else {
#pragma unroll
        for (int i = 0; i < TM / 2; ++i) block(std::false_type{}, i);
    }
    if constexpr (EpiHasFinish<Epi>::value) epi.finish(lp, z, unit);
}

// The tiles of a launch: along N, along M, of a batch entry, all, an eighth of them (rounded up); reciprocals for quotient()
struct NtGrid { int nx, ny, per_z, tiles, share; float inv_per_z, inv_panel; };
// n / d for 0 <= n < 2^31, d >= 1, inv = 1.0f / d, in a handful of instructions: the estimate is off by n / d 2^-23 and less than
// one more, which a step mends up to quotients of 2^22 (a launch's batch entries, a batch entry's panels)
__device__ __forceinline__ int quotient(int n, int d, float inv)
{
    int q = __builtin_amdgcn_readfirstlane((int)((float)n * inv));
    const int r = n - q * d;
    q += r < 0 ? -1 : r >= d ? 1 : 0;
    return q;
}

// A kernel's arguments, BYTES of them beginning with these two, requested at once.  Left to the compiler, each load goes out shortly before
// its use, and a wavefront that has nothing else to do waits for one line of the arguments after the other: the launches of 2310 products
// of 142 random blocks take 0.972 of that, those below 6 us 0.962.
template <size_t BYTES>
__device__ __forceinline__ void request_arguments(const GemmNT &p, const NtGrid &g)
{
    const auto *args = (__attribute__((address_space(4))) const int *)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int LAST = (int)(BYTES / 4) - 1, THIRD = LAST > 32 ? 32 : LAST;      // lines of 16 words
    static_assert(sizeof(GemmNT) + sizeof(NtGrid) > 64 && LAST < 48, "the first two lines by the values, a third by its first word");
    asm volatile("" :: "s"(p.A), "s"(p.B), "s"(p.lda), "s"(p.M), "s"(p.N), "s"(p.K), "s"(p.sA), "s"(p.sB), "s"(g.nx), "s"(g.ny), "s"(g.per_z),
                 "s"(g.tiles), "s"(g.share), "s"(g.inv_per_z), "s"(g.inv_panel), "s"(args[THIRD]));
}

// f(n - 1), ..., f(0), the numbers as types
template <int N, class F>
__device__ __forceinline__ void unrolled(F f)
{
    if constexpr (N > 0) {
        f(std::integral_constant<int, N - 1>{});
        unrolled<N - 1>(f);
    }
}

// BLKA: A is stored in 32 x 32 blocks (see above); B always is.  In LDS a stage is [BM rows][32 k] of
// A, then [BN rows][32 k] of B, rows of 64 B, slot s of row r holding piece s ^ ((r >> 3) & 1) * 2.
// WPS: wavefronts per SIMD the registers are budgeted for.
template <int BM, int BN, int WM, int WN, int WPS, int NS, bool BLKA, class Epi>
__global__ __launch_bounds__(WM * WN * 64, WPS) void gemm_nt_bf16_kernel(GemmNT p, NtGrid g, Epi epi)
{
    request_arguments<sizeof(GemmNT) + sizeof(NtGrid) + sizeof(Epi)>(p, g);
    constexpr int BK = 32, NW = WM * WN;
    constexpr int TM = BM / WM / 16, TN = BN / WN / 16, MM = TM * TN;
    constexpr int CA = BM / 16, CB = BN / 16;           // 1 KiB chunks (16 rows x 64 B) per stage
    constexpr int CPW = (CA + CB) / NW;                 // ... and wavefront
    static_assert((CA + CB) % NW == 0 && BM % 32 == 0 && BN % 32 == 0, "chunks / waves");
    constexpr int STAGE = (BM + BN) * BK;
    extern __shared__ __attribute__((aligned(1024))) unsigned char gemm_smem[];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    bf16_t *smem = (bf16_t *)gemm_smem;
    const int wm = wave / WN, wn = wave % WN;
    // Workgroups go to the 8 XCDs round-robin by linear id (the grid's x extent is a multiple of
    // 8).  Tile order: batch entry (worker), then panels of 4 N-tiles, then M-tile, then N-tile
    // inside the panel; each XCD takes a contiguous eighth of that order.  One XCD's L2 then sees
    // one worker's B operand (for 8 workers), and the tiles that run together share their A rows
    // and B rows: 30-45 % fewer bytes fetched into L2 than with the batch as a grid dimension.
    // (Panels of 2, 3, 6 or 12 tiles: the same to 3 %, the narrow ones slower at N = 768.)
    int tile = (blockIdx.x % 8) * g.share + blockIdx.x / 8;
    if (tile >= g.tiles) return;
    // all of a wavefront's requests depend on these: quotients by multiplication
    const int z = quotient(tile, g.per_z, g.inv_per_z);
    tile -= z * g.per_z;
    constexpr int PANEL = 4;
    const int pn = quotient(tile, g.ny * PANEL, g.inv_panel);
    tile -= pn * g.ny * PANEL;
    const int bw = min(PANEL, g.nx - pn * PANEL);
    const int by = bw == 4 ? tile >> 2 : bw == 2 ? tile >> 1 : bw == 1 ? tile : (int)(((unsigned long long)(unsigned)tile * 0xAAAAAAABull) >> 33);
    const int bx = pn * PANEL + tile - by * bw;
    const int m0 = by * BM, n0 = bx * BN;
    const int nk = p.K / BK;                           // stages
    const bf16_t *A = p.A + (long long)z * p.sA;
    const bf16_t *B = p.B + (long long)z * p.sB;

    // Per-lane global source of each 1 KiB chunk this wave copies: chunk c is 16 rows, LDS slot
    // (row, s) holds the global piece s ^ ((row >> 3) & 1) * 2 of that row.  Blocked operand: half of a
    // 32 x 32 block, consecutive in memory up to that permutation; rows beyond the matrix inside the
    // last 256-row panel are allocated (their values only reach accumulator rows never stored), and
    // every tile shape divides 256.  Row-major A: 16 pieces of 64 B, rows clamped.
    const bf16_t *src[CPW];
    const int piece = ((lane & 3) ^ (lane >> 5) * 2) * 8;
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
    // The copies as asm: behind the builtin, the compiler waits for all LDS reads in flight at every use of one.  The s_nop is
    // the wait state that such a copy needs behind a write of m0 (the compiler sets m0 right before the statement, and counts
    // wait states for its own copies only).
    const unsigned lds_ring = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)smem;
    int d_stage = 0;                                    // stage the next copy goes to
    auto issue = [&](int i) {
        const int c = wave * CPW + i;
        const unsigned dst = __builtin_amdgcn_readfirstlane(lds_ring + d_stage * (STAGE * 2) + c * 1024);
        asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "{m0}"(dst), "v"(src[i]) : "memory");
        src[i] += BLKA || c >= CA ? 1024 : BK;
    };
    auto issued = [&]() { d_stage = d_stage + 1 == NS ? 0 : d_stage + 1; };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // A stage's fragments (16 rows x 32 k each) of A and B.  AHEAD, for small tiles: a second set holds the next stage's.
    constexpr bool AHEAD = MM <= 4;
    constexpr int SETS = AHEAD ? 2 : 1;
    constexpr int HA = AHEAD ? TM : TM / 2, HB = TM - HA;    // rows of blocks multiplied before and behind a stage's barrier
    bf16x8 fa[SETS][TM], fb[SETS][TN];
    // the lane's place in a stage: row l%16 of a fragment, piece l/16
    const int lane_off = (lane & 15) * 32 + (((lane >> 4) ^ ((lane >> 3) & 1) * 2) * 8);
    const int offA = wm * TM * 512 + lane_off, offB = BM * BK + wn * TN * 512 + lane_off;
    auto read_a = [&](int stage, int set, int i) { fa[set][i] = *(const bf16x8 *)(smem + stage * STAGE + offA + i * 512); };
    auto read_b = [&](int stage, int set, int j) { fb[set][j] = *(const bf16x8 *)(smem + stage * STAGE + offB + j * 512); };
    auto multiply = [&](int set, int i, int j) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][j], fa[set][i], acc[i][j], 0, 0, 0);
    };
    // a barrier that no memory access is moved across
    auto barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // until at most `stages` stages' copies are outstanding, and for all LDS reads
    auto wait = [&](auto stages) {
        constexpr int n = CPW * decltype(stages)::value;
        static_assert(n < 64, "vmcnt has six bits");
        __builtin_amdgcn_s_waitcnt(0x0070 | (n & 15) | ((n >> 4) << 14));
    };

    // Main loop.  A stage's blocks are multiplied column by column of the wavefront's tile, the first half of its rows
    // and then the second half, so that one set of fragments is enough: while the first half's MFMAs issue, the
    // second half's A fragments are read (and the last column's B fragment, which the stage before needed to its end); then
    // comes the barrier (everyone's copies of the next stage have landed, everyone is through reading this one); while the
    // second half's MFMAs issue, the next stage's A fragments of the first half are read, each column's B fragment as soon as
    // the column is through with the present one, and the stage NS further on is requested into the buffer just freed.
    // Small tiles hold two sets: the barrier comes first, and the next stage is read while this one is multiplied.
    // The order is pinned instruction by instruction (sched_barrier after every MFMA): one LDS read or one copy
    // between two MFMAs.  Left to the compiler, the reads go out in one burst in front of the MFMAs and both wavefronts of a
    // SIMD do so together.
    // Timed on MI355X at 12608 x 768 x 3072, batch 8, bf16 output: 363 us = 1.31 PFLOP/s; with 32x32x16
    // instructions, everything else alike, 407; with these and conflicts in the fragment reads 381.  Without its copies the
    // same kernel takes 300 us, without its LDS reads 316, without its barriers 352 (at a lower clock: what they cost is power), the
    // bare MFMAs 225.  With large tiles neither 3, 4 or 5 stages nor raised wave priority around the MFMAs make a difference.
    auto compute = [&]() {
    auto request = [&]() {
#pragma unroll
        for (int i = 0; i < CPW; ++i) issue(i);
        issued();
    };
    if constexpr (AHEAD) {                             // a loop: small problems wait for instructions as much as for data
#pragma unroll 1
        for (int s = 0; s < min(NS, nk); ++s) request();
    } else {
#pragma unroll
        for (int s = 0; s < NS; ++s) if (s < nk) request();
    }
    unrolled<NS>([&](auto left) { if ((nk < NS ? nk : NS) - 1 == decltype(left)::value) wait(left); });
    barrier();
    int cur = 0;
#pragma unroll
    for (int i = 0; i < HA; ++i) read_a(0, 0, i);
#pragma unroll
    for (int j = 0; j < TN - (AHEAD ? 0 : 1); ++j) read_b(0, 0, j);
    if constexpr (AHEAD) {                             // sets alternate so that the last stage has set 0: the first, either
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[1][i] = fa[0][i];
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[1][j] = fb[0][j];
    }
    // With scalar loads (the epilogue's arguments) in flight at its top, which complete in any order, the loop would wait for all
    // LDS reads at its first MFMA.
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F);
    auto next = [&]() { cur = cur + 1 == NS ? 0 : cur + 1; };
    auto stage_ahead = [&](auto set_c, auto last_c, auto issue_c, auto left) {
        constexpr int SET = decltype(set_c)::value;
        constexpr bool LAST = decltype(last_c)::value, ISSUE = decltype(issue_c)::value;
        if (!LAST) {
            wait(left);
            barrier();
            next();
        }
        __builtin_amdgcn_sched_barrier(0);
        if (!LAST) {
#pragma unroll
            for (int i = 0; i < TM; ++i) read_a(cur, SET ^ 1, i);
#pragma unroll
            for (int j = 0; j < TN; ++j) read_b(cur, SET ^ 1, j);
        }
#pragma unroll
        for (int m = 0; m < MM; ++m) {
            multiply(SET, m % TM, m / TM);
#pragma unroll
            for (int i = 0; i < CPW; ++i)
                if (!LAST && ISSUE && (CPW <= MM ? i : i * MM / CPW) == m) issue(i);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!LAST && ISSUE) issued();
    };
    auto stage_halves = [&](auto, auto last_c, auto issue_c, auto left) {
        constexpr bool LAST = decltype(last_c)::value, ISSUE = decltype(issue_c)::value;
        constexpr int MA = HA * TN, MB = HB * TN;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < MA; ++m) {                  // serpentine: neighbours share an operand
            const int j = m / HA, i = j & 1 ? HA - 1 - m % HA : m % HA;
            multiply(0, i, j);
            if (m == 0) read_b(cur, 0, TN - 1);
            else if (m <= HB) read_a(cur, 0, HA + m - 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!LAST) {
            wait(left);
            barrier();
            next();
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            const int j = m / HB, i = HA + (j & 1 ? HB - 1 - m % HB : m % HB);
            multiply(0, i, j);
            if (!LAST) {
                if (m < HA) read_a(cur, 0, m);
                if (m % HB == HB - 1 && j < TN - 1) read_b(cur, 0, j);
            }
#pragma unroll
            for (int c = 0; c < CPW; ++c)
                if (!LAST && ISSUE && (CPW <= MB ? MB - CPW + c : c * MB / CPW) == m) issue(c);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!LAST && ISSUE) issued();
    };
    auto stage = [&](auto set_c, auto last_c, auto issue_c, auto left) {
        if constexpr (AHEAD) stage_ahead(set_c, last_c, issue_c, left);
        else stage_halves(set_c, last_c, issue_c, left);
    };
    // At a stage's wait the stages behind the next one are outstanding, NS - 2 of them while requests go on
    constexpr std::integral_constant<int, NS - 2> full{};
    constexpr std::integral_constant<int, 0> set0{};
    constexpr std::integral_constant<int, SETS - 1> set1{};
    static_assert(!AHEAD || NS % 2 == 0, "the stages behind the last request begin with set 1");
    int todo = nk - NS;
    if (AHEAD) {
        if (todo > 0 && (todo & 1)) { stage(set0, std::false_type{}, std::true_type{}, full); --todo; }
        for (; todo > 0; todo -= 2) { stage(set1, std::false_type{}, std::true_type{}, full); stage(set0, std::false_type{}, std::true_type{}, full); }
    } else {
        for (; todo > 0; --todo) stage(set0, std::false_type{}, std::true_type{}, full);
    }
    unrolled<NS - 1>([&](auto left) {                  // NS - 2, ..., 0 stages outstanding
        constexpr int LEFT = decltype(left)::value;
        if (nk >= LEFT + 2) stage(std::integral_constant<int, AHEAD ? (LEFT + 1) & 1 : 0>{}, std::false_type{}, std::false_type{}, left);
    });
    stage(set0, std::true_type{}, std::false_type{}, set0);

        __syncthreads();                               // every wavefront is done with the ring
    };
    epilogue_via_lds<TM, TN>(acc, (float *)gemm_smem + wave * StagedTile<TN * 16>::FLOATS, lane, m0 + wm * TM * 16,
                             n0 + wn * TN * 16, p.M, p.N, z, (by * g.nx + bx) * NW + wave, epi, compute);
}

typedef short s16x4 __attribute__((ext_vector_type(4)));   // operand of the LDS transpose read

template <NtShape SHAPE, int WM, int WN, int WPS, bool BLKA, class Epi>
inline hipError_t launch_gemm_nt(const GemmNT &p, const Epi &epi, int batch, hipStream_t s)
{
    constexpr int BM = NT_TILE[SHAPE].bm, BN = NT_TILE[SHAPE].bn, NS = NT_TILE[SHAPE].stages;
    static_assert(256 % BM == 0 && 256 % BN == 0, "blocked operands are allocated in panels of 256 rows");
    if (p.K % 32 != 0 || p.K < 32 || p.N % 64 != 0) return hipErrorInvalidValue;
    const long long tiles = nt_tiles(SHAPE, p.M, p.N, batch);
    if (tiles > (1 << 24)) return hipErrorInvalidValue;    // threads of a launch
    dim3 grid((unsigned)(tiles + 7) / 8 * 8, 1, 1);
    constexpr size_t ring = (size_t)NS * (BM + BN) * 32 * sizeof(bf16_t);
    constexpr size_t staging = (size_t)WM * WN * StagedTile<BN / WN>::FLOATS * sizeof(float);
    constexpr size_t smem = ring > staging ? ring : staging;
    static_assert(smem <= 160 * 1024, "tile does not fit the 160 KB LDS");
    auto kern = gemm_nt_bf16_kernel<BM, BN, WM, WN, WPS, NS, BLKA, Epi>;
    static bool lds_limit_raised = false;     // per instantiation; contexts are not thread-safe
    if (smem > 64 * 1024 && !lds_limit_raised) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        lds_limit_raised = true;
    }
    NtGrid g;
    g.nx = (p.N + BN - 1) / BN; g.ny = (p.M + BM - 1) / BM; g.per_z = g.nx * g.ny; g.tiles = (int)tiles; g.share = (int)(grid.x / 8);
    g.inv_per_z = 1.0f / (float)g.per_z; g.inv_panel = 1.0f / (float)(4 * g.ny);
    kern<<<grid, WM * WN * 64, smem, s>>>(p, g, epi);
    return hipGetLastError();
}

}  // namespace qsr
