// Layout arithmetic of the team workspace, on the host: for handles whose
// sweeps run by teams, and every work list that their scratch can hold, the
// workspace is used only where it lies outside the layout in force.  Prints one
// line per case; exit code 1 on an overlap.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "abi_internal.h"

namespace mcabi {
Tile default_tile(const mc_replica_desc *reps, int n, size_t esz);
void make_work(const mc_replica_desc *reps, int n, const Tile &t, std::vector<WorkItem> &work,
               std::vector<uint32_t> &begin, std::vector<uint32_t> &end);
ScratchLayout scratch_layout(int n_reps, uint64_t n_items, int n_colours);
} // namespace mcabi
using namespace mcabi;

static int check(int n, int Lx, int Ly, int Lz, uint64_t need)
{
    mc_sim h;
    h.n_reps = n;
    h.kind = MC_SC;
    h.n_colours = 2;
    mc_replica_desc d = {};
    d.kind = MC_SC;
    d.Lx = Lx, d.Ly = Ly, d.Lz = Lz;
    d.periodic_mask = 7;
    d.J = 1.0, d.T = 1.0, d.e[2] = 1.0;
    h.desc.assign((size_t)n, d);
    auto layout = [&](const Tile &t) {
        std::vector<uint32_t> b, e;
        make_work(h.desc.data(), n, t, h.work, b, e);
        return scratch_layout(n, h.work.size(), h.n_colours);
    };
    uint64_t required = 0;
    if (mc_required_scratch(h.desc.data(), n, &required) != MC_OK) return 1;
    h.scratch = (char *)0x100000000000; // arithmetic only
    h.scratch_bytes = std::max<uint64_t>(required, 4u << 20);
    h.lay = layout(default_tile(h.desc.data(), n, sizeof(float)));
    const uint64_t beside = align_up(h.lay.total, 256); // right behind the default layout
    const uint64_t at = team_offset(h.scratch_bytes, h.lay.total, need);
    int bad = 0, inside = 0, moved = 0;
    if (at == kTeamNoRoom) bad += h.lay.total + need + 256 <= h.scratch_bytes;
    else bad += at < h.lay.total || at + need > h.scratch_bytes || at % 256 != 0;
    const ScratchLayout first = h.lay;
    for (int kernel : {KERNEL_TILE, KERNEL_STRIP, KERNEL_BAND})
        for (int tx : {8, 16, 64})
            for (int zc : {1, 2, 5, 16, 64}) {
                const int ty = kernel == KERNEL_TILE ? 256 / tx : 2;
                h.lay = layout(Tile{kernel, kernel == KERNEL_TILE ? tx : 64, ty, zc});
                if (h.lay.total > h.scratch_bytes) continue; // refused by mc_set_tile
                inside += beside < h.lay.total && h.lay.total > first.total;
                if (at == kTeamNoRoom) continue;
                h.team_ws = h.scratch + at;
                h.team_owned = false;
                h.team_on = false;
                const bool overlap = at < h.lay.total;
                bad += team_disjoint(&h) == overlap;
                if (!overlap) continue;
                // the state must not be put into the live layout again
                ++moved;
                (void)team_activate(&h);
                bad += h.team_on && !h.team_owned;
                team_release(&h);
            }
    std::printf("%d x %dx%dx%d, %llu bytes: workspace at %lld of %llu, layouts over the default's end "
                "%d, over the workspace %d, bad %d\n", n, Lx, Ly, Lz, (unsigned long long)need,
                at == kTeamNoRoom ? -1ll : (long long)at, (unsigned long long)h.scratch_bytes, inside,
                moved, bad);
    return bad;
}

int main()
{
    int bad = 0;
    for (uint64_t need : {100000ull, 1000001ull, 2500000ull, 3800000ull, 5000000ull}) {
        bad += check(12, 8, 8, 100, need);
        bad += check(8, 4, 4, 400, need);
        bad += check(22, 20, 20, 20, need);
        bad += check(24, 22, 22, 22, need);
        bad += check(5, 24, 24, 24, need);
    }
    // everything, nothing and one byte less than what is left
    bad += team_offset(4096, 4096, 0) != 4096;
    bad += team_offset(4096, 256, 3840) != 256;
    bad += team_offset(4096, 256, 3841) != kTeamNoRoom;
    bad += team_offset(4096, 0, 4097) != kTeamNoRoom;
    return bad ? 1 : 0;
}
