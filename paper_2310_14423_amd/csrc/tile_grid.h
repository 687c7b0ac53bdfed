// tile_grid.h -- the grid of a launch whose workgroups number their tiles themselves (host arithmetic, and so apart from the
// kernels): x and y together hold at least `tiles`, and a kernel leaves workgroups beyond those alone.
#pragma once

namespace qsr {

struct TileGrid { unsigned x, y; };
// A launch takes fewer than 2^32 threads along x and at most 65536 workgroups along y.  x = 0: more than fit.
inline TileGrid tile_grid(long long tiles, int threads)
{
    const long long most = (1ll << 31) / threads, rows = (tiles + most - 1) / most;
    if (tiles < 1 || rows > 65536) return {0, 0};
    return {(unsigned)((tiles + rows - 1) / rows), (unsigned)rows};
}

}  // namespace qsr
