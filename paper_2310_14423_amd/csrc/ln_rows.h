// ln_rows.h -- how the LayerNorm backward pass shares the token rows of a worker among wavefronts.  Host arithmetic only,
// apart from the kernels, so that it can be checked without a GPU.
#pragma once

namespace qsr {

// A row of d lies in the registers of LPR lanes as VPL float4 each (d <= 4 LPR VPL, d a multiple of 64): F(VPL, LPR)
#define LN_BY_WIDTH(d, F) do { if ((d) <= 64) F(1, 16); else if ((d) <= 128) F(1, 32); else if ((d) <= 256) F(1, 64); \
                               else if ((d) <= 512) F(2, 64); else if ((d) <= 768) F(3, 64); else F(4, 64); } while (0)

// Rows of a lane group in flight at once: what the registers hold where latency is all (few rows), one or two where the
// wavefronts beside it hide it.
constexpr int ln_bwd_rows(int vpl, bool few) { return few ? (vpl <= 2 ? 4 : 2) : (vpl == 1 ? 2 : 1); }

// The wavefronts of a worker take steps of `step` rows (64 / LPR side by side, ln_bwd_rows of each in flight) in turn.
// Few enough of them that all wavefronts of the launch are resident at once (a launch of 1.5 times the chip's wavefront slots
// runs as one full wave of workgroups and a half-empty one: 283 against 234 us at 8 x 12608 rows of 768), resident wavefronts
// per compute unit following from the kernel's registers; not fewer than four rows each, since each leaves a row of partial
// sums for the parameter gradients (two each: 7 x 852 tokens of 704, three blocks with attention, 1374 against 1357 us an
// iteration; at least 16, few tokens left most of the chip idle: 27 us a pass at 2 x 1040 rows of 192); and not fewer
// than a step, since a wavefront without rows leaves a row of zeros (with rows of 64, three of four did; 4 x 4000
// tokens of 128, three blocks with attention, 404 against 395 us).
struct LnBwdPlan { bool few; int step; long long waves; };
inline LnBwdPlan ln_bwd_plan(long long K, long long M, long long d)
{
    const int vpl = (int)((d + 255) / 256), side = d <= 64 ? 4 : d <= 128 ? 2 : 1;
    const long long slots = 256LL * (vpl <= 2 ? 20 : vpl == 3 ? 16 : 12);
    long long rows = (K * M + slots - 1) / slots;
    LnBwdPlan q;
    q.few = rows <= 4;
    q.step = side * ln_bwd_rows(vpl, q.few);
    if (rows < 4) rows = 4;
    if (rows < q.step) rows = q.step;
    q.waves = (M + rows - 1) / rows;
    return q;
}

}  // namespace qsr
