// Rows that the LDS-staged band kernel stages, on the host: every row it copies
// lies in the lattice, and every row that a site of the tile reads is the right
// one, for every tile height and lattice height.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "mc_internal.hpp"

int main()
{
    long bad = 0, once = 0;
    for (int Ly = 1; Ly <= 140; ++Ly)
        for (int periodic = 0; periodic < 2; ++periodic)
            for (int ty = 1; ty <= 64; ++ty)
                for (int y0 = 0; y0 < Ly; y0 += ty) {
                    for (int k = 0; k < ty + 2; ++k) { // other colour's rows y0-1 .. y0+ty
                        const int y = y0 - 1 + k, r = mc::lband_row(y, Ly, periodic != 0);
                        bad += r < -1 || r >= Ly;
                        // a single wrap leaves the lattice
                        once += periodic && y >= 2 * Ly;
                    }
                    for (int y = y0; y < std::min(y0 + ty, Ly); ++y) { // the tile's sites
                        bad += mc::lband_row(y, Ly, periodic != 0) != y;
                        for (int d : {-1, 1}) {
                            const int n = y + d;
                            const int want = n >= 0 && n < Ly ? n : periodic ? (n + Ly) % Ly : -1;
                            bad += mc::lband_row(n, Ly, periodic != 0) != want;
                        }
                    }
                }
    std::printf("%ld wrong rows, %ld rows that a single wrap leaves outside\n", bad, once);
    return bad != 0 || once == 0;
}
