// Host-side check of the candidate bytes of a one-wavefront tile: the interior
// cells' bytes, the marks' offsets from them and from the lanes' spares.
#include <cstdio>
#include <set>

#include "fmm_tile.h"

using namespace fmm;

template <int E> static int check()
{
    using Gm = Geo<E>;
    int bad = 0;
    std::set<int> cells;
    for (int p = 0; p < Gm::V; p++) cells.insert(Gm::cfi(p));
    bad += (int)cells.size() != Gm::V;
    const int off[6] = {-Gm::CX, Gm::CX, -Gm::CY, Gm::CY, -1, 1};
    for (int p = 0; p < Gm::V; p++) {
        const int c = Gm::cfi(p), i0 = p / (E * E), i1 = p / E % E, i2 = p % E;
        bad += c < 0 || c >= Gm::CFP;
        bad += i2 == 0 && c % E != 0;  // a row of E cells is aligned
        for (int k = 0; k < 6; k++) {
            const bool in[6] = {i0 > 0, i0 < E - 1, i1 > 0, i1 < E - 1, i2 > 0, i2 < E - 1};
            const int step[6] = {-E * E, E * E, -E, E, -1, 1};
            // a neighbour in the tile: its byte.  Across a face of axes 0 and 1
            // (the marks along axis 2 test their coordinate): a byte that is
            // nobody's, inside the array.
            if (in[k])
                bad += c + off[k] != Gm::cfi(p + step[k]);
            else if (k < 4)
                bad += cells.count(c + off[k]) != 0 || c + off[k] < 0 || c + off[k] >= Gm::CFB;
        }
    }
    for (int lane = 0; lane < 64; lane++)
        for (int k = 0; k < 7; k++) {
            const int s = Gm::spare(lane) + (k < 6 ? off[k] : 0);
            bad += cells.count(s) != 0 || s < 0 || s >= Gm::CFB;
        }
    if (bad) std::printf("E=%d: %d\n", E, bad);
    return bad;
}

int main()
{
    const int bad = check<4>() + check<8>();
    if (!bad) std::printf("ok\n");
    return bad != 0;
}
