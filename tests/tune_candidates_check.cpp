// The autotuner's candidates, on the host: a handle with teams has every
// candidate of one without (the teams are timed besides them).
#include <algorithm>
#include <cstdio>
#include <vector>

#include "abi_internal.h"

namespace mcabi {
std::vector<Tile> tile_candidates(const mc_sim *h);
}
using namespace mcabi;

int main()
{
    int bad = 0;
    for (int L : {8, 16, 20, 24, 48})
        for (int kind : {MC_SC, MC_BCC, MC_FCC})
            for (mc_precision prec : {MC_F32, MC_F64}) {
                mc_sim h;
                h.n_reps = 1;
                h.kind = kind;
                h.prec = prec;
                h.lds_max = 158 * 1024;
                mc_replica_desc d = {};
                d.kind = kind;
                d.Lx = d.Ly = d.Lz = L;
                d.periodic_mask = 7;
                d.J = 1.0, d.T = 1.0, d.e[2] = 1.0;
                h.desc.push_back(d);
                mc_spin_buffers b = {};
                RepDev R;
                fill_repdev(d, b, R);
                h.reps.push_back(R);
                const std::vector<Tile> plain = tile_candidates(&h);
                char ws = 0;
                h.team_ws = &ws;
                const std::vector<Tile> teams = tile_candidates(&h);
                bool same = plain.size() == teams.size() && !plain.empty();
                for (size_t i = 0; same && i < plain.size(); ++i) same = same_tile(plain[i], teams[i]);
                int lds = 0;
                for (const Tile &t : teams) lds += t.kernel == KERNEL_LDS;
                if (!same || lds != (lds_fits(&h) ? 3 : 0)) {
                    std::printf("kind %d, L %d, precision %d: %zu candidates, %zu with teams, %d in LDS\n",
                                kind, L, (int)prec, plain.size(), teams.size(), lds);
                    ++bad;
                }
                h.team_ws = nullptr;
            }
    return bad ? 1 : 0;
}
