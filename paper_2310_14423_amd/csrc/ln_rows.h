// ln_rows.h -- how the LayerNorm backward pass shares the token rows of a worker among wavefronts.  Host arithmetic only,
// apart from the kernels, so that it can be checked without a GPU.
#pragma once

namespace qsr {

// A row of d lies in the registers of LPR lanes as VPL float4 each (d <= 4 LPR VPL, d a multiple of 64): F(VPL, LPR)
#define LN_BY_WIDTH(d, F) do { if ((d) <= 64) F(1, 16); else if ((d) <= 128) F(1, 32); else if ((d) <= 256) F(1, 64); \
                               else if ((d) <= 512) F(2, 64); else if ((d) <= 768) F(3, 64); else F(4, 64); } while (0)

// Rows of a lane group in flight at once
constexpr int ln_bwd_rows(int vpl) { return vpl == 1 ? 2 : 1; }
// Few rows: a step of one row a lane group for each wavefront, and the sums of a workgroup's wavefronts added up in LDS.
constexpr int LN_FEW_WAVES = 8;

// The wavefronts of a worker take steps of `step` rows (64 / LPR side by side, ln_bwd_rows of each in flight) in turn.
// Few enough of them that all wavefronts of the launch are resident at once (a launch of 1.5 times the chip's wavefront slots
// runs as one full wave of workgroups and a half-empty one: 283 against 234 us at 8 x 12608 rows of 768), resident wavefronts
// per compute unit following from the kernel's registers; not fewer than four rows each, since each leaves a row of partial
// sums for the parameter gradients (two each: 7 x 852 tokens of 704, three blocks with attention, 1374 against 1357 us an
// iteration; at least 16, few tokens left most of the chip idle: 27 us a pass at 2 x 1040 rows of 192).
// Where a launch has few rows, its time is a wavefront's instructions one after the other, so a wavefront takes one step of one
// row a lane group: 2 x 1040 rows of 192 4.3 us, 5.7 with four rows in flight and four times the code; 3 x 247 of 128 6.6 and 4.7
// with two of them.  The workgroup's sums are added up in LDS, so that the sums behind read fewer rows (4.0 -> 3.6 us).
// `waves`: what leaves a row of partial sums, of a worker: wavefronts or, with few rows, the workgroups that add theirs up.
struct LnBwdPlan { bool few; int step; long long waves; };
inline LnBwdPlan ln_bwd_plan(long long K, long long M, long long d)
{
    const int vpl = (int)((d + 255) / 256), side = d <= 64 ? 4 : d <= 128 ? 2 : 1;
    const long long slots = 256LL * (vpl <= 2 ? 20 : vpl == 3 ? 16 : 12);
    long long rows = (K * M + slots - 1) / slots;
    LnBwdPlan q;
    q.few = rows <= 4;
    if (q.few) {
        q.step = side;
        q.waves = (M + side * LN_FEW_WAVES - 1) / (side * LN_FEW_WAVES);
        return q;
    }
    q.step = side * ln_bwd_rows(vpl);
    if (rows < q.step) rows = q.step;
    q.waves = (M + rows - 1) / rows;
    return q;
}

}  // namespace qsr
