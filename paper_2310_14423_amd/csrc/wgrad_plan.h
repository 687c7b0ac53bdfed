// wgrad_plan.h -- how a weight gradient of the block models (M x N outputs per worker, a reduction over the
// tokens) is cut into tiles and token ranges, and the workspace that the ranges' partial results take.  Host
// arithmetic only, apart from the kernels, so that each can be checked against the other without a GPU.
#pragma once

namespace qsr {

constexpr int WGRAD_SPLIT = 4;          // most ranges a weight gradient's token reduction is cut into

// Floats of the partial products and of the partial bias gradients of one launch for K workers of a model of width d,
// hidden width dh: a launch holds the weights d x dh and dh x d or, with attention, d x 3d and d x d, of one block, or of
// all n_blocks; a bias is as long as its weight's second dimension.
struct WgradSpace { long long products, biases; };
inline WgradSpace wgrad_space(long long K, long long d, long long dh, bool attention, long long n_blocks = 1)
{
    const long long mlp = 2 * d * dh, attn = attention ? 4 * d * d : 0, mlp_b = d + dh, attn_b = attention ? 4 * d : 0;
    if (n_blocks > 1) return {K * WGRAD_SPLIT * n_blocks * (mlp + attn), K * WGRAD_SPLIT * n_blocks * (mlp_b + attn_b)};
    return {K * WGRAD_SPLIT * (mlp > attn ? mlp : attn), K * WGRAD_SPLIT * (mlp_b > attn_b ? mlp_b : attn_b)};
}

// Tile shape by the number of tiles and the length of the reduction, from timing on MI355X (us; batch x tokens x
// width x hidden: gradient of the second weight / of a width x width projection; s4: cut into four ranges, without
// the 6-16 us that adding them up takes):
//                              192x384          128x128, 3 WG/CU    128x128, 2 groups    64x64, 4 groups   before
//   8 x 12608 x 768 x 3072   407 / 297, s4 117   589 / 193           616 / 217              - / -          468 / 372 (s4 128)
//   2 x 12608 x 768 x 3072   271 / 269, s4 113   177 / 115, s4 51    192 / 97             236 / 99         375 / 357
//   1 x 12608 x 768 x 3072   291 / 275, s4 84    121 / 116, s4 35    101 / 97             131 / 47         374 / 360
//   8 x 1576 x 768 x 3072     61 / 43             68 / 28             84 / 32             148 / 42          68 / 53
//   4 x 2000 x 512 x 2048     53 / 50             26 / 22             25 / 20              43 / 11          67 / 65
//   2 x 400 x 768 x 3072      18 / 16             11 / 7.6            15 / 8.0             25 / 10.5        21 / 20
//   2 x 1040 x 192 x 768      32 / 30             13 / 13             12 / 12             8.0 / 7.7         39 / 38
// Hence: the large tile from 160 of them on; a long reduction (4096 tokens) with fewer is cut into up to WGRAD_SPLIT
// ranges, on the large tile while that makes about 200 workgroups, else on the small one; a short one goes to
// 128 x 128 (two groups per workgroup below 200 of them) and from 110 of those down to 64 x 64 with four groups.
enum WgradTile { WGRAD_192x384, WGRAD_128x128, WGRAD_128x128_2GROUPS, WGRAD_64x64_4GROUPS };
struct WgradPlan { WgradTile tile; int split, k_chunk; };    // split > 1: ranges of k_chunk tokens (a multiple of 32)
// whether a launch may be cut into token ranges; big: its tiles of 192 x 384
inline bool wgrad_may_split(long long big, long long tokens) { return big < 160 && tokens >= 4096; }
// big, mid: the launch's tiles of 192 x 384 and of 128 x 128
inline WgradPlan wgrad_plan_tiles(long long big, long long mid, int tokens, int n_cu)
{
    if (wgrad_may_split(big, tokens)) {
        const bool large = big >= 48;
        const long long want = large ? n_cu / big : 3LL * n_cu / mid;
        int split = (int)(want < 1 ? 1 : want > WGRAD_SPLIT ? WGRAD_SPLIT : want);
        const int k_chunk = ((tokens + split - 1) / split + 31) / 32 * 32;
        split = (tokens + k_chunk - 1) / k_chunk;
        if (split > 1) return {large ? WGRAD_192x384 : WGRAD_128x128, split, k_chunk};
    }
    return {big >= 160 ? WGRAD_192x384 : mid >= 200 ? WGRAD_128x128 : mid >= 110 ? WGRAD_128x128_2GROUPS : WGRAD_64x64_4GROUPS, 1, 0};
}
inline long long wgrad_tiles(int bm, int bn, int M, int N) { return (long long)((M + bm - 1) / bm) * ((N + bn - 1) / bn); }
// one weight gradient alone
inline WgradPlan wgrad_plan(int M, int N, int tokens, int batch, int n_cu)
{
    return wgrad_plan_tiles(wgrad_tiles(192, 384, M, N) * batch, wgrad_tiles(128, 128, M, N) * batch, tokens, n_cu);
}

#ifndef WGRAD_DEFER_TILES
#define WGRAD_DEFER_TILES 1024
#endif
// Whether the weight gradients of all blocks wait for one launch behind the backward pass (each block then keeps its
// operands) instead of two launches per block.
inline bool wgrad_defer(long long K, long long tokens, long long d, long long dh, bool attention, long long n_blocks)
{
    if (n_blocks < 2) return false;
    const long long tiles = K * (wgrad_tiles(128, 128, (int)d, (int)dh) + wgrad_tiles(128, 128, (int)dh, (int)d) +
                                 (attention ? wgrad_tiles(128, 128, (int)d, (int)(3 * d)) + wgrad_tiles(128, 128, (int)d, (int)d) : 0));
    const long long bytes = K * tokens * n_blocks * (d + dh + (attention ? 4 * d : 0)) * 2;
    return tiles < WGRAD_DEFER_TILES && bytes <= (1ll << 31);
}

}  // namespace qsr
