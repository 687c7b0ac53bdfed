// ln_rows.h -- how the LayerNorm backward pass shares the token rows of a worker among wavefronts.  Host arithmetic only,
// apart from the kernels, so that it can be checked without a GPU.
#pragma once

namespace qsr {

// A row of d lies in the registers of LPR lanes as VPL float4 each (d <= 4 LPR VPL, d a multiple of 64): F(VPL, LPR)
#define LN_BY_WIDTH(d, F) do { if ((d) <= 64) F(1, 16); else if ((d) <= 128) F(1, 32); else if ((d) <= 256) F(1, 64); \
                               else if ((d) <= 512) F(2, 64); else if ((d) <= 768) F(3, 64); else F(4, 64); } while (0)

// Rows of a lane group in flight at once
constexpr int ln_bwd_rows(int vpl) { return vpl == 1 ? 2 : 1; }
// Few rows: the wavefronts of a workgroup, whose sums are added up in LDS
constexpr int LN_FEW_WAVES = 8;

// The wavefronts of a worker take steps of `step` rows (64 / LPR side by side, ln_bwd_rows of each in flight) in turn.
// Many rows (more than four for each wavefront that the chip holds): as many wavefronts as are resident at once, which follows from the kernel's
// registers (a launch of 1.5 times the chip's wavefront slots runs as one full wave of workgroups and a half-empty one: 283 against
// 234 us at 8 x 12608 rows of 768).  Each leaves a row of partial sums for the parameter gradients.
// Few rows: one step of one row a lane group for each wavefront, up to four times as many wavefronts as the chip holds, eight of them to a row of
// partial sums.  A launch's time is then a wavefront's instructions one after the other: 2 x 1040 rows of 192 4.3 us, 5.7 with four rows in
// flight in four times the code; and the sums behind read fewer rows (4.0 -> 3.6 us).  Up to four rows a slot the two launches together are
// faster for it at all widths, against resident wavefronts of four rows or more each with a row of partial sums (us, this pass twice with one launch of sums):
//   2 x 10240 rows of 128 24.7 (25.8), of 192 32.1 (37.5), of 512 55.8 (69.5), 2 x 8192 of 768 71.0 (84.3), 2 x 6144 of 1024 76.5 (85.2);
//   at one row a slot, 2 x 2560 of 192 14.8 (18.4), of 512 23.1 (26.5), 2 x 2048 of 768 23.3 (31.9), 2 x 1536 of 1024 26.2 (35.5).
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
