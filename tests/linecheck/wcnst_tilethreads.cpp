// Host build of the 1D step kernels' tiles (Tile1D in wcnst_device.hpp): what
// a stage forms, for every tile of a line, against the threads that form it.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "wcnst_device.hpp"

using namespace wcnst;

// Most positions that a stage of any tile forms.
template <int DIFF>
static int most(int nx, int bc, int w)
{
    int m = 0;
    for (int t = 0; t < (nx + w - 1) / w; ++t) {
        const Tile1D<DIFF> T(t, w, nx, bc);
        for (int s = 0; s < 2; ++s) m = std::max(m, T.out_hi(s) - T.out_lo(s));
        m = std::max(m, T.B(2) - T.A(2));
    }
    return m;
}

extern "C" {

int tt_threads() { return TILE_THREADS; }

int tt_most(int nx, int bc, int diff, int pair)
{
    if (pair) return most<DIFF_MND>(nx, bc, line_tile_width<DIFF_MND, true>(nx));
    if (diff == DIFF_MD) return most<DIFF_MD>(nx, bc, line_tile_width<DIFF_MD>(nx));
    if (diff == DIFF_HW) return most<DIFF_HW>(nx, bc, line_tile_width<DIFF_HW>(nx));
    return most<DIFF_MND>(nx, bc, line_tile_width<DIFF_MND>(nx));
}

// Positions of a line that is one tile (0 where it is several).
int tt_whole(int nx, int bc)
{
    const int w = line_tile_width<DIFF_MND>(nx);
    return w < nx ? 0 : Tile1D<DIFF_MND>(0, w, nx, bc).positions();
}

}  // extern "C"
