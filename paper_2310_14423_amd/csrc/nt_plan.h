// nt_plan.h -- the tile shape of a forward or data-gradient product of the block models (gemm_bf16.h), from its sizes and the
// kind of its outputs.  Host arithmetic only, apart from the kernels, so that it can be checked without a GPU.
#pragma once

namespace qsr {

// Shapes: tile, stages of the ring (of 32 along the contraction), workgroups that a compute unit holds.  The two small tiles come
// with a short ring and more workgroups, or with a long ring for problems that do not fill the chip and wait for their loads.
enum NtShape { NT_64x64, NT_64x64_LONG, NT_128x128, NT_128x128_LONG, NT_128x256, NT_256x256 };
constexpr int NT_SHAPES = 6;
struct NtTileShape { int bm, bn, stages, resident; };
constexpr NtTileShape NT_TILE[NT_SHAPES] = {{64, 64, 4, 4}, {64, 64, 8, 2}, {128, 128, 3, 3}, {128, 128, 5, 2}, {128, 256, 3, 2}, {256, 256, 4, 1}};

// What an epilogue does: GELU and its derivative, two outputs; a factor read; fp32 read and written; bf16 written; fp32 written; fp32 read,
// fp32 and bf16 written and summed up
enum NtOut { NT_GELU, NT_FACTOR, NT_RESIDUAL, NT_BF16, NT_F32, NT_LOSS };
constexpr int NT_OUTS = 6;

// The loss's sums leave its wavefronts of the two large tiles without registers (8 x 11491 x 1024 x 1024 320 us, 295 in tiles of 128 x 128),
// and 128 x 128 with the long ring is hardly ever the shortest.
constexpr bool nt_allowed(NtShape s, NtOut out) { return out != NT_LOSS || s == NT_64x64 || s == NT_64x64_LONG || s == NT_128x128; }

inline long long nt_tiles(NtShape s, long long M, long long N, long long batch)
{
    return ((M + NT_TILE[s].bm - 1) / NT_TILE[s].bm) * ((N + NT_TILE[s].bn - 1) / NT_TILE[s].bn) * batch;
}

// Estimated time in us.  A compute unit takes its tiles in rounds of as many as it holds; a round lasts as long as a tile by
// itself (latency + per stage of 32 + epilogue) or as all its tiles' work (per stage + epilogue each), smoothed between them.
// Fitted to 508 products (1 to 8 workers, 64 to 12608 tokens, widths 64 to 1024, hidden to 4 times that, each kind of output)
// timed with every shape on MI355X, which it reproduces to 10-15 %, and to the sizes of a 12-block 768/3072 encoder.
// The loss's epilogues are fitted to what the choice costs over 523 other products, timed with every shape too: 0.8 % (2.7 % with those of
// the other fp32 epilogue that reads: 3 x 9159 x 704 x 704 62.0 us in tiles of 128 x 128, 72.8 in the 128 x 256 that these choose).
// (The wait of a lone 128 x 256 tile is that of operands that come from the other XCDs' products: 2 x 1251 tokens x 2112 x 704
// 17.8 us, 13.8 in tiles of 128 x 128.)
inline double nt_us(NtShape s, NtOut out, long long tiles, long long K, int n_cu)
{
    struct Fit { double latency, wait, work, epilogue[NT_OUTS]; };
    static constexpr Fit FIT[NT_SHAPES] = {
        {0.70, 0.107, 0.096, {0.70, 0.80, 1.13, 0.36, 0.78, 1.98}},
        {0.64, 0.043, 0.101, {1.02, 0.97, 1.26, 0.58, 0.91, 2.48}},
        {0.87, 0.124, 0.259, {2.67, 1.90, 2.96, 0.94, 1.37, 6.18}},
        {0.38, 0.058, 0.240, {3.07, 2.34, 2.97, 1.33, 1.81, 7.75}},
        {2.57, 0.450, 0.416, {5.20, 3.90, 4.90, 1.86, 2.43, 15.86}},
        {14.4, 0.000, 0.670, {7.70, 5.05, 6.37, 0.00, 0.97, 18.12}},
    };
    const Fit &f = FIT[s];
    const double st = (double)(K / 32), e = f.epilogue[out];
    auto round = [&](long long n) {
        const double a = f.latency + f.wait * st + e, b = (double)n * (e + f.work * st);
        const double a2 = a * a, b2 = b * b, q = a2 * a2 + b2 * b2;
        double r = a > b ? a : b;                      // fourth root by Newton's method, from above half of it
        for (int i = 0; i < 6; ++i) r -= (r * r * r * r - q) / (4.0 * r * r * r);
        return r;
    };
    const long long per_cu = (tiles + n_cu - 1) / n_cu, full = per_cu / NT_TILE[s].resident, rest = per_cu % NT_TILE[s].resident;
    return (double)full * round(NT_TILE[s].resident) + (rest > 0 ? round(rest) : 0.0);
}

// The shape with the least estimate, of those that the estimate is right for.  128 x 256 from a contraction of 256 on.  256 x 256 from 1024 on:
// its row is a fit of whole rounds on the bounds of its parameters, not of a tile's time, and promises too much below.  Where it would be
// taken at 768 to 1023 the launch is 6 % longer with GELU (31 products) and a residual (27) and 4 % with a factor (39).  With a plain output it is 1.7 %
// shorter by itself (66 products), but whole models of such products run no faster for it (12 of 3 to 6 blocks at 0.987 to 1.012 of the time,
// 0.999 on average): the chip runs them at its power limit.
// Over the products above its choices take 1.3 % longer than the best; the rule by tile counts that it replaces, with shapes for a
// full chip and two groups of wavefronts on a long contraction, 5.1 %.  E.g. (us; before) 2 x 1040 x 192 x 768 5.5 (6.1), 5 x 2945 x
// 256 x 1024 12.1 (15.8), 2 x 9381 x 448 x 1344 32.1 (39.9).
inline NtShape nt_shape(NtOut out, long long M, long long N, long long K, long long batch, int n_cu)
{
    NtShape best = NT_64x64;
    double us = 1e300;
    for (int i = 0; i < NT_SHAPES; ++i) {
        const NtShape s = (NtShape)i;
        if ((s == NT_128x256 && K < 256) || (s == NT_256x256 && K < 1024) || !nt_allowed(s, out)) continue;
        const double t = nt_us(s, out, nt_tiles(s, M, N, batch), K, n_cu);
        if (t < us) { us = t; best = s; }
    }
    return best;
}

}  // namespace qsr
