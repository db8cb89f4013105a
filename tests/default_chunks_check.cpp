// Planes per workgroup of default tiles, on the host: one round of workgroups
// only from 1.4 rounds of single planes on, FP32 fcc with two planes at most.
#include <cstdio>
#include <vector>

#include "abi_internal.h"

namespace mcabi {
Tile default_tile(const mc_replica_desc *reps, int n, size_t esz);
}
using namespace mcabi;

static int check(int kind, size_t esz, int n, int L, double radius, int zc)
{
    mc_replica_desc d = {};
    d.kind = kind;
    d.Lx = d.Ly = d.Lz = L;
    d.periodic_mask = radius > 0.0 ? 0 : 7;
    d.sphere_radius = radius;
    d.J = 1.0, d.T = 1.0, d.e[2] = 1.0;
    const std::vector<mc_replica_desc> reps((size_t)n, d);
    const Tile t = default_tile(reps.data(), n, esz);
    if (t.zc != zc)
        std::printf("kind %d, %zu bytes, %d x %d^3, R %g: kernel %d, %d planes, expected %d\n", kind,
                    esz, n, L, radius, t.kernel, t.zc, zc);
    return t.zc != zc;
}

int main()
{
    int bad = 0;
    // 0.84, 1.12, 1.25, 1.42, 2 and 7.8 rounds
    bad += check(MC_SC, 4, 1, 96, 0, 1) + check(MC_SC, 4, 1, 104, 0, 1);
    bad += check(MC_SC, 4, 16, 40, 0, 1) + check(MC_SC, 4, 1, 112, 0, 2);
    bad += check(MC_SC, 4, 1, 128, 0, 2) + check(MC_SC, 4, 1, 200, 0, 8);
    // FP64: 1.09, 1.69 and 4 rounds
    bad += check(MC_SC, 8, 1, 80, 0, 1) + check(MC_SC, 8, 1, 96, 0, 2);
    bad += check(MC_SC, 8, 1, 128, 0, 4);
    // fcc: 1.12, 2 and 3.9 rounds in FP32, 3.4 in FP64, a sphere
    bad += check(MC_FCC, 4, 1, 104, 0, 1) + check(MC_FCC, 4, 1, 128, 0, 2);
    bad += check(MC_FCC, 4, 1, 160, 0, 2) + check(MC_FCC, 8, 1, 96, 0, 4);
    bad += check(MC_FCC, 4, 1, 160, 75, 2);
    // beyond eight planes: about 6000 workgroups as before
    bad += check(MC_SC, 4, 1, 464, 0, 9) + check(MC_SC, 8, 1, 464, 0, 31);
    return bad ? 1 : 0;
}
