// wgrad_plan.h -- how a weight gradient of the block models (M x N outputs per worker, a reduction over the
// tokens) is cut into tiles and token ranges, and the workspace that the ranges' partial results take.  Host
// arithmetic only, apart from the kernels, so that each can be checked against the other without a GPU.
#pragma once
#include <initializer_list>

namespace qsr {

constexpr int WGRAD_SPLIT = 4;          // most ranges a weight gradient's token reduction is cut into
constexpr int WGRAD_SPLIT_TOKENS = 1024;   // ... from this length on

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

// Workspace for the partial results of a launch whose outputs span `span` floats: WGRAD_SPLIT of it, but not more than
// 256 MiB (a launch that large fills the chip without ranges: 8 x 5885 tokens x 832 x 2496 545 us, 448 in two ranges and
// 90 to add them up), nor anything below two ranges.
constexpr long long wgrad_part_floats(long long span)
{
    return 2 * span > (1ll << 26) ? 0 : WGRAD_SPLIT * span > (1ll << 26) ? 1ll << 26 : WGRAD_SPLIT * span;
}

// Tile shape and token ranges of a launch: the cheapest by estimated time.  The estimate is rounds of the chip times the
// time of a tile (a fixed part, for filling the ring and the epilogue, and a part per 32-token stage), fitted to 218 random
// launches of one or several weight gradients (1 to 8 workers, 1 to 4 blocks, widths 64 to 1024, 64 to 12608 tokens) timed with
// all shapes and ranges on MI355X, which it reproduces to 5-10 %; us per tile and stage:
//                      resident per compute unit   fixed   32 tokens
//   192 x 384                     1                 8.3      0.804
//   128 x 128                     3                 4.5      0.295 alone, 0.540 two, 0.785 three together
//   128 x 128, 2 groups           1                 4.7      0.519 for 64 tokens
//   64 x 64, 4 groups             1                 3.7      0.462 for 128 tokens
// Its choices took 0.8 % longer than the best ones (adding up ranges included); the rule by tile counts that it replaces
// 14.7 %.  E.g. (us; best of the others) 8 x 5885 tokens x 832 x 2496: 2240 tiles of 128 x 128 560 for 545 with two groups;
// 4 x 3350 x 704 x 1408: 128 tiles of 192 x 384 92, 528 of 128 x 128 72; 2 x 1060 x 192 x 768 and attention: 64 x 64 8.7, 128 x 128 11.5.
enum WgradTile { WGRAD_192x384, WGRAD_128x128, WGRAD_128x128_2GROUPS, WGRAD_64x64_4GROUPS };
constexpr int WGRAD_TILES = 4;
struct WgradPlan { WgradTile tile; int split, k_chunk; double us; };    // split > 1: ranges of k_chunk tokens (a multiple of 32)

// A launch: its tiles by shape, its outputs, and the stretches of memory that its partial results are added up in
struct WgradLoad {
    long long big = 0, mid = 0, small = 0, outputs = 0;
    int stretches = 1;
    void add(long long M, long long N, long long copies)
    {
        big += (M + 191) / 192 * ((N + 383) / 384) * copies;
        mid += (M + 127) / 128 * ((N + 127) / 128) * copies;
        small += M / 64 * (N / 64) * copies;
        outputs += M * N * copies;
    }
};
inline double wgrad_us(WgradTile tile, const WgradLoad &q, long long tokens, int split, int n_cu)
{
    const long long stages = ((tokens + split - 1) / split + 31) / 32;
    auto rounds = [&](long long tiles) { return (double)((tiles * split + n_cu - 1) / n_cu); };
    double us = 0.0;
    switch (tile) {
    case WGRAD_192x384: us = rounds(q.big) * (8.3 + 0.804 * (double)stages); break;
    case WGRAD_128x128: {
        const long long per_cu = (long long)rounds(q.mid), full = per_cu / 3, rest = per_cu % 3;
        us = (double)full * (4.5 + 0.785 * (double)stages) + (rest > 0 ? 4.5 + (0.295 + 0.245 * (double)(rest - 1)) * (double)stages : 0.0);
        break;
    }
    case WGRAD_128x128_2GROUPS: us = rounds(q.mid) * (4.7 + 0.519 * (double)((stages + 1) / 2)); break;
    default: us = 1.0 + rounds(q.small) * (3.7 + 0.462 * (double)((stages + 3) / 4)); break;
    }
    if (split > 1) us += 2.5 * q.stretches + (split + 1) * 4.0 * (double)q.outputs / 4.5e6;   // a launch each, 4.5 TB/s
    return us;
}
// part_floats: the workspace for partial results
inline WgradPlan wgrad_plan_load(const WgradLoad &q, int tokens, int n_cu, long long part_floats, long long span)
{
    WgradPlan best{WGRAD_128x128, 1, 0, 1e300};
    for (int want = 1; want <= WGRAD_SPLIT; ++want) {
        if (want > 1 && (tokens < WGRAD_SPLIT_TOKENS || want * span > part_floats)) break;
        const int k_chunk = ((tokens + want - 1) / want + 31) / 32 * 32, split = (tokens + k_chunk - 1) / k_chunk;
        if (split != want) continue;
        for (int t = 0; t < WGRAD_TILES; ++t) {
            const double us = wgrad_us((WgradTile)t, q, tokens, split, n_cu);
            if (us < best.us) best = {(WgradTile)t, split, split > 1 ? k_chunk : 0, us};
        }
    }
    return best;
}
// Whether the weight gradients of all blocks wait for one launch behind the backward pass (each block then keeps its
// operands, at most 2 GiB) instead of two launches per block: where the estimates say that it is faster.  Decided for the
// whole chip's 256 compute units, since it decides the workspace's layout.  The sums behind it take two workgroups along the
// grid's z extent for each LayerNorm and one more, of at most 65536.  2 x 1040 tokens x 192 x 768, two blocks with
// attention: 67 us of weight gradients in 8 launches, 13 in one.
inline bool wgrad_defer(long long K, long long tokens, long long d, long long dh, bool attention, long long n_blocks)
{
    const long long bytes = K * tokens * n_blocks * (d + dh + (attention ? 4 * d : 0)) * 2;
    if (n_blocks < 2 || bytes > (1ll << 31) || (attention ? 4 : 2) * n_blocks + 1 > 65536) return false;
    WgradLoad mlp, attn, all;
    for (WgradLoad *q : {&mlp, &all}) {
        const long long copies = q == &all ? K * n_blocks : K;
        q->add(d, dh, copies); q->add(dh, d, copies);
    }
    if (attention)
        for (WgradLoad *q : {&attn, &all}) {
            const long long copies = q == &all ? K * n_blocks : K;
            q->add(d, 3 * d, copies); q->add(d, d, copies);
        }
    all.stretches = attention ? 2 : 1;
    auto us = [&](const WgradLoad &q) {
        const long long span = q.outputs + q.outputs / 32;          // about: biases and LayerNorm parameters
        return wgrad_plan_load(q, (int)tokens, 256, wgrad_part_floats(span), span).us;
    };
    return us(all) < (double)n_blocks * (us(mlp) + (attention ? us(attn) : 0.0));
}


// The launches of a model of n_blocks: the MLP halves (mlp) or the attention halves of one block or, with `all`, both of every
// block.  What they cover of a worker's gradient, from the first weight to the last bias, and their load.
struct WgradCover { long long floats; WgradLoad load; };
inline WgradCover wgrad_cover(bool mlp, bool all, long long K, long long d, long long dh, bool attention, long long n_blocks)
{
    const long long w_mlp = 2 * d * dh + d + dh, w_attn = 4 * d * d + 4 * d;
    const long long per_block = 2 * d + w_mlp + (attention ? 2 * d + w_attn : 0), copies = all ? K * n_blocks : K;
    WgradCover q{mlp ? w_mlp : w_attn, {}};
    if (all) q.floats = n_blocks * per_block - 2 * d;            // (the first LayerNorm's parameters lie in front)
    if (mlp || all) { q.load.add(d, dh, copies); q.load.add(dh, d, copies); }
    if (attention && (!mlp || all)) { q.load.add(d, 3 * d, copies); q.load.add(d, d, copies); }
    q.load.stretches = all && attention ? 2 : 1;
    return q;
}

// Floats of workspace for the partial results of any launch of the model (deferred: wgrad_defer)
inline long long wgrad_split_floats(long long K, long long tokens, long long d, long long dh, bool attention, long long n_blocks, bool deferred)
{
    if (tokens < WGRAD_SPLIT_TOKENS) return 0;
    const WgradSpace parts = wgrad_space(K, d, dh, attention, deferred ? n_blocks : 1);      // (all blocks: the LayerNorm parameters as well)
    const long long norms = deferred ? K * 2 * (attention ? 2 : 1) * n_blocks * d : 0;
    return wgrad_part_floats((parts.products + parts.biases) / WGRAD_SPLIT + norms);
}

}  // namespace qsr
