// wgrad_plan.h -- how a weight gradient of the block models (M x N outputs per worker, a reduction over the
// tokens) is cut into tiles and token ranges, and the workspace that the ranges' partial results take.  Host
// arithmetic only, apart from the kernels, so that each can be checked against the other without a GPU.
#pragma once

namespace qsr {

constexpr int WGRAD_SPLIT = 4;          // most ranges a weight gradient's token reduction is cut into

// Floats of the partial products and of the partial bias gradients for K workers of a model of width d, hidden
// width dh: the weights are d x dh, dh x d and, with attention, d x 3d and d x d; a bias is as long as its weight's
// second dimension.
struct WgradSpace { long long products, biases; };
inline WgradSpace wgrad_space(long long K, long long d, long long dh, bool attention)
{
    const long long weight = d * (attention && 3 * d > dh ? 3 * d : dh);
    long long bias = d > dh ? d : dh;
    if (attention && 3 * d > bias) bias = 3 * d;
    return {K * WGRAD_SPLIT * weight, K * WGRAD_SPLIT * bias};
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
inline WgradPlan wgrad_plan(int M, int N, int tokens, int batch, int n_cu)
{
    auto tiles = [&](int bm, int bn) { return (long long)((M + bm - 1) / bm) * ((N + bn - 1) / bn) * batch; };
    const long long big = tiles(192, 384), mid = tiles(128, 128);
    if (big < 160 && tokens >= 4096) {
        const bool large = big >= 48;
        const long long want = large ? n_cu / big : 3LL * n_cu / mid;
        int split = (int)(want < 1 ? 1 : want > WGRAD_SPLIT ? WGRAD_SPLIT : want);
        const int k_chunk = ((tokens + split - 1) / split + 31) / 32 * 32;
        split = (tokens + k_chunk - 1) / k_chunk;
        if (split > 1) return {large ? WGRAD_192x384 : WGRAD_128x128, split, k_chunk};
    }
    return {big >= 160 ? WGRAD_192x384 : mid >= 200 ? WGRAD_128x128 : mid >= 110 ? WGRAD_128x128_2GROUPS : WGRAD_64x64_4GROUPS, 1, 0};
}

}  // namespace qsr
