// Host build of the index geometry of the 1D step kernels (Tile1D in
// wcnst_device.hpp), checked for every tile of a line.
#include <hip/hip_runtime.h>

#include <vector>

#include "wcnst_device.hpp"

using namespace wcnst;

// 0 when the tiles own every cell once and, in every stage of every tile,
// every index the kernel forms stays inside the tile's positions and reads
// only what the stage's input holds; else a code naming the first violation.
template <int DIFF>
static int check(int nx, int bc, int w, int cap, int threads)
{
    const int nt = (nx + w - 1) / w;
    using T1 = Tile1D<DIFF>;
    std::vector<int> owned((size_t)nx, 0);
    for (int t = 0; t < nt; ++t) {
        const T1 T(t, w, nx, bc);
        const int base = T.base(), np = T.positions();
        if (T.c0 >= T.c1) return 1;
        for (int c = T.c0; c < T.c1; ++c) owned[(size_t)c] += 1;
        if (np > cap) return 2;
        // the load: every position has a source cell
        for (int p = base; p < base + np; ++p) {
            const int c = ghost_map(p, nx, bc);
            if (c < 0 || c >= nx) return 3;
            if (T.ghosts && (p < -T1::REACH || p >= nx + T1::REACH)) return 4;
        }
        int lo = base, hi = base + np;  // positions the stage's input holds
        for (int s = 0; s < 3; ++s) {
            const int a = T.A(s), b = T.B(s), nf = T.faces(s);
            // (a thread, or a pair of threads, for every midpoint)
            if (nf > cap || nf > threads || nf != b - a + 2 * T1::G - 1) return 5;
            for (int i = 0; i < nf; ++i)
                for (int m = 0; m < 6; ++m) {
                    const int p = a - T1::G - 2 + i + m;
                    if (p < lo || p >= hi) return 6;
                }
            if (DIFF == DIFF_HW)
                for (int i = 0; i < b - a + 4; ++i) {
                    const int p = a - 2 + i;
                    if (p < lo || p >= hi || i >= cap) return 7;
                }
            // (a tile of several writes only its own cells in the last stage)
            const bool own = s == 2 && nt > 1;
            for (int p = own ? a : T.out_lo(s); p < (own ? b : T.out_hi(s)); ++p) {
                const int c = T.source(p, bc);
                if (c < a || c >= b || c < lo || c >= hi) return 8;
                if (p < base || p >= base + np) return 9;
                if (!T.ghosts && c != p) return 10;
                // midpoints c - G .. c + G - 1, of thread i: a - G + i
                if (c - a + 2 * T1::G - 1 >= nf) return 11;
            }
            lo = T.out_lo(s);
            hi = T.out_hi(s);
        }
        if (T.A(2) != T.c0 || T.B(2) != T.c1) return 12;
    }
    for (int v : owned)
        if (v != 1) return 13;
    return 0;
}

extern "C" {

// pair: tiles of two threads a midpoint (MND)
int lc_check(int nx, int bc, int diff, int pair)
{
    constexpr int N = TILE_THREADS;
    if (pair) return check<DIFF_MND>(nx, bc, line_tile_width<DIFF_MND, true>(nx), PAIR_CAP, PAIR_FACES);
    if (diff == DIFF_MD) return check<DIFF_MD>(nx, bc, line_tile_width<DIFF_MD>(nx), LINE_CAP, N);
    if (diff == DIFF_HW) return check<DIFF_HW>(nx, bc, line_tile_width<DIFF_HW>(nx), LINE_CAP, N);
    return check<DIFF_MND>(nx, bc, line_tile_width<DIFF_MND>(nx), LINE_CAP, N);
}

}  // extern "C"
