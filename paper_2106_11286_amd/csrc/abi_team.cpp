// abi_team.cpp -- team sweeps of small lattices (kernels_team.hip): which
// handles use them, how the planes are dealt to workgroups, and their launches.
#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "abi_internal.h"

using namespace mcabi;

namespace {

// Sweeps per measured launch (a launch keeps the sums of every sweep).
constexpr uint32_t kTeamChunk = 64;
// Sweeps per unmeasured launch (bounds one launch to some tens of ms).
constexpr uint32_t kTeamLong = 4096;
// Polls of a word before a workgroup gives up (about 0.5 us each, 30 ms in all;
// mc_set_watchdog can lower it) and one workgroup does the launch's sweeps again.
constexpr uint32_t kTeamSpins = 1u << 16;

// Plans whose colour phases look longer than this are not considered.
constexpr double kTeamPhaseUs = 4.5;
// Box sites of a handle: beyond, a pass launch is no longer mostly overhead.
constexpr uint64_t kTeamSites = 400000;

struct TeamPlan {
    std::vector<TeamWg> wgs;
    uint64_t words = 0;
    uint32_t lds = 0;
    int threads = 0;
    uint32_t most = 1, polls = 1, members = 1; // sites of a colour per workgroup, rounds
                                               // of polled words, largest team
    double phase_us = 0.0; // bound on the time of a colour phase
    bool teams = false;    // some replica has more than one workgroup
};

// What n sweeps cost, in us, by teams and without them: the figures behind
// team_from.  Fitted to 145 lattices and batches (sc, bcc, fcc, both precisions,
// 4 k to 260 k sites), 1 to 20 sweeps a call; where the two come close the plain
// kernels are taken.  Per call (launch, filling and writing back the planes) a
// team costs about 9 us and more with its workgroups, two or four pass launches
// 3; per colour a team's exchange and updates cost 1.8 us with a hundred sites
// per workgroup, 2.2 with 512 and 4 to 5 with twice that, a pass 3.4 to 5.
// Unmeasured, us per call, teams / plain: sc 40^3 one sweep 16.4 / 11.4, 20
// sweeps 158 / 180; fcc 32^3 20 sweeps 435 / 330; FP64 16^3 one sweep 13.3 / 17.
struct TeamCost {
    bool f64, fcc, bcc, tile, lds; // tile: the pass kernel is not a pair or band kernel
    bool ragged;                   // rows that are no multiple of 64 bytes
    uint32_t most, polls, threads, grid, members, lds_sites, items;
    int nc;
    double team(uint32_t n, bool measure) const
    {
        const double low = std::min(most, 512u), high = most - low;
        double phase = f64 ? (fcc ? 2.85 : bcc ? 2.6 : 2.15) + (bcc ? 0.0016 : 0.0018) * low
                           : (fcc ? 2.45 : bcc ? 2.2 : 1.75) + 0.0008 * low;
        phase += (f64 ? 0.004 : fcc || polls > 1 ? 0.0018 : bcc ? 0.002 : 0.0024) * high;
        phase += (f64 ? 2.0 : fcc ? 1.65 : bcc ? 1.3 : 0.9) * (polls - 1);
        if (tile && !fcc && !bcc) phase += f64 ? 0.3 : 0.15; // a sphere's test per site
        if (measure) phase += fcc ? 0.2 : 0.35;
        double t = 8.8 + 0.032 * grid + (fcc ? 2.0 : 0.0) + n * nc * phase;
        // the records: one workgroup adds its team's sums, 8 n of them at a time
        if (measure) t += 0.8 + 0.16 * members * ((8u * n + threads - 1) / threads);
        return t;
    }
    double plain(uint32_t n, bool measure) const
    {
        if (lds) { // per colour by its sites; a measured call's records are copied
            const double site = f64 ? (fcc ? 0.0033 : bcc ? 0.0026 : 0.0020)
                                    : (fcc ? 0.0022 : bcc ? 0.0018 : 0.0012);
            return 8.0 + (measure ? 8.0 : 0.0) + n * (nc * site * lds_sites + (measure ? 1.2 : 0.0));
        }
        const bool basis = fcc || bcc;
        double pass = f64 ? (fcc ? 4.8 : bcc ? 4.4 : 5.1)
                          : (fcc ? 4.1 : bcc ? 3.75 : ragged ? 4.5 : 4.3);
        if (tile) pass = basis ? 1.25 * pass : f64 ? 3.9 : 3.3;
        // the reduction's launch and a share per workgroup of the passes
        const double records = (fcc ? 5.6 : bcc ? 4.2 : 4.0) +
                               (tile ? 0.005 : 0.0025) * items;
        return 2.9 + n * (nc * pass + (measure ? records : 0.0));
    }
};

// Deal every replica's planes so that a workgroup holds about `q` sites of a colour.
TeamPlan plan_teams(const mc_sim *h, uint32_t q)
{
    TeamPlan P;
    const int esz = h->prec == MC_F64 ? 8 : 4, nc = h->n_colours, nw = h->prec == MC_F64 ? 6 : 3;
    uint32_t most = 1, plane_most = 1;
    for (int r = 0; r < h->n_reps; ++r) {
        const RepDev &R = h->reps[r];
        const uint32_t psites = (uint32_t)R.Lxh * (uint32_t)R.Ly;
        const int nz = (int)std::min<uint32_t>((uint32_t)R.Lz, std::max(1u, q / psites));
        const int members = (R.Lz + nz - 1) / nz;
        const bool per = (R.pmask & 4u) != 0;
        // slots: one per outer plane of a workgroup
        std::vector<int> lo_slot(members), hi_slot(members);
        int slots = 0;
        for (int m = 0; m < members; ++m) {
            const int n = std::min(nz, R.Lz - m * nz);
            lo_slot[m] = slots++;
            hi_slot[m] = n > 1 ? slots++ : lo_slot[m];
        }
        const uint32_t first = (uint32_t)P.wgs.size();
        for (int m = 0; m < members; ++m) {
            TeamWg w;
            std::memset(&w, 0, sizeof w);
            w.rep = (uint32_t)r;
            w.z0 = m * nz;
            w.nz = std::min(nz, R.Lz - w.z0);
            const int below = m > 0 ? m - 1 : (per ? members - 1 : -1);
            const int above = m < members - 1 ? m + 1 : (per ? 0 : -1);
            w.z_lo = w.z0 > 0 ? w.z0 - 1 : (per ? R.Lz - 1 : -1);
            w.z_hi = w.z0 + w.nz < R.Lz ? w.z0 + w.nz : (per ? 0 : -1);
            const bool team = members > 1;
            w.lo = team && below >= 0 ? hi_slot[below] : -1;
            w.hi = team && above >= 0 ? lo_slot[above] : -1;
            w.own_lo = team && below >= 0 ? lo_slot[m] : -1;
            w.own_hi = team && above >= 0 ? hi_slot[m] : -1;
            w.first = first;
            w.members = (uint32_t)members;
            w.words = P.words;
            P.wgs.push_back(w);
        }
        P.teams |= members > 1;
        P.members = std::max(P.members, (uint32_t)members);
        if (members > 1) P.words += (uint64_t)slots * nc * nw * psites;
        P.lds = std::max<uint32_t>(
            P.lds, (uint32_t)std::min<uint64_t>(0xFFFFFFFFu, team_lds_bytes(h->kind, psites, nz, esz)));
        most = std::max(most, psites * (uint32_t)nz);
        plane_most = std::max(plane_most, psites);
    }
    P.threads = (int)std::min<uint32_t>(TEAM_THREADS, (most + 63u) / 64u * 64u);
    // the exchange, then rounds of updates and of polled words
    const uint32_t rounds = (most + (uint32_t)P.threads - 1) / (uint32_t)P.threads;
    const uint32_t polls = (plane_most + (uint32_t)P.threads - 1) / (uint32_t)P.threads;
    P.most = most;
    P.polls = polls;
    P.phase_us = 1.0 + (h->prec == MC_F64 ? 1.5 : 0.65) * rounds +
                 (h->prec == MC_F64 ? 0.8 : 0.55) * polls;
    return P;
}

// Kernels of this process that the GPU can run beside one another: HIP's
// hardware queues, 4 unless the environment asks for more.
uint32_t hardware_queues()
{
    const char *v = std::getenv("GPU_MAX_HW_QUEUES");
    const long n = v ? std::strtol(v, nullptr, 10) : 0;
    return (uint32_t)std::max(4l, std::min(n, 32l));
}

void team_bind(mc_sim *h, char *ws, bool owned)
{
    h->team_ws = ws;
    h->team_owned = owned;
    h->team_state = (uint32_t *)ws;
    h->team_wgs = (TeamWg *)(ws + h->team_off_wgs);
    h->team_words = (uint64_t *)(ws + h->team_off_words);
    h->team_partials = (double *)(ws + h->team_off_part);
}

// A workspace of the library's own.
bool team_own(mc_sim *h)
{
    char *ws = nullptr;
    if (hipMalloc((void **)&ws, h->team_bytes) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    team_bind(h, ws, true);
    return true;
}

} // namespace

namespace mcabi {

void team_init(mc_sim *h)
{
    h->team_ws = nullptr;
    h->team_on = false;
    // The LDS kernel (one workgroup per replica) is the faster one while a
    // colour takes its workgroup one round: 864 sites 2.7 us per sweep against
    // 3.7, FP64 504 sites 4.4 against 5.8; beyond, sc 16^3 (2048) 5.2 against
    // 3.8, FP64 8.5 against 4.9.
    uint32_t most = 0;
    uint64_t sites = 0;
    for (const RepDev &R : h->reps) {
        most = std::max(most, R.plane);
        sites += R.n_box;
    }
    if (h->tile.kernel == KERNEL_LDS && most <= (h->prec == MC_F64 ? 640u : 1024u)) return;
    if (sites > kTeamSites) return;
    int dev = 0, cus = 0;
    if (h->lds_max == 0 || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    if (h->stream) { // a stream kept to part of the compute units
        uint32_t mask[32] = {0};
        if (hipExtStreamGetCUMask(h->stream, 32, mask) != hipSuccess) {
            (void)hipGetLastError();
            return;
        }
        int n = 0;
        for (uint32_t m : mask) n += __builtin_popcount(m);
        if (n > 0) cus = std::min(cus, n);
    }
    const bool f64 = h->prec == MC_F64;
    // the smallest share per workgroup whose launch fits the GPU `share` times
    // over: team launches on as many streams then seldom wait for each other's
    // workgroups to leave.  (Seldom, not never: other kernels and other
    // processes take their part, too, which costs time, see kernels_team.hip.)
    const uint32_t share = hardware_queues();
    TeamPlan P;
    bool found = false;
    for (uint32_t q = 64; q <= 8192 && !found; q += q / 8) {
        P = plan_teams(h, q);
        // more planes per workgroup need more LDS and more rounds
        if (!P.teams || P.lds > h->lds_max || P.phase_us > kTeamPhaseUs) return;
        if (P.wgs.size() > (size_t)cus) continue;
        int per_cu = 0;
        if (team_allow(h->kind, f64, P.lds) != hipSuccess ||
            team_slots(h->kind, f64, P.threads, P.lds, &per_cu) != hipSuccess) {
            (void)hipGetLastError();
            return;
        }
        found = P.wgs.size() * share <= (size_t)cus * (size_t)std::max(0, per_cu);
    }
    if (!found) return;
    {
        TeamCost c;
        c.f64 = f64;
        c.fcc = h->kind == MC_FCC;
        c.bcc = h->kind == MC_BCC;
        c.tile = h->pass_tile.kernel == KERNEL_TILE || h->pass_tile.kernel == KERNEL_BSTRIP;
        c.lds = h->default_tile.kernel == KERNEL_LDS;
        c.most = P.most;
        c.polls = P.polls;
        c.threads = (uint32_t)P.threads;
        c.grid = (uint32_t)P.wgs.size();
        c.members = P.members;
        c.lds_sites = most;
        c.ragged = false;
        for (const RepDev &R : h->reps) c.ragged |= R.Lxh % 16 != 0;
        c.items = (uint32_t)h->work.size();
        c.nc = h->n_colours;
        for (int m = 0; m < 2; ++m) {
            h->team_from[m] = kTeamNever;
            for (uint32_t n = kTeamChunk; n > 0 && c.team(n, m) < c.plain(n, m); --n)
                h->team_from[m] = n;
        }
        if (h->team_from[0] == kTeamNever && h->team_from[1] == kTeamNever) return;
    }
    uint64_t o = 0;
    const uint64_t n_state = 4 + 3 * (uint64_t)h->n_reps;
    h->team_off_wgs = (o = align_up(sizeof(uint32_t) * n_state, 256));
    h->team_off_words = (o = align_up(o + sizeof(TeamWg) * P.wgs.size(), 256));
    h->team_off_part = (o = align_up(o + sizeof(uint64_t) * P.words, 256));
    h->team_bytes = o + sizeof(double) * NQ * kTeamChunk * P.wgs.size();
    h->team_grid = (uint32_t)P.wgs.size();
    h->team_threads = P.threads;
    h->team_lds = P.lds;
    h->team_table.swap(P.wgs);
    const uint64_t at = team_offset(h->scratch_bytes, h->lay.total, h->team_bytes);
    if (at != kTeamNoRoom &&
        check_device_buffer(h->scratch, at + h->team_bytes, "scratch", -1) == MC_OK) {
        team_bind(h, h->scratch + at, false);
    } else {
        g_err.clear(); // the allocation ends before scratch_bytes: leave its end alone
        if (!team_own(h)) return;
    }
    if (team_activate(h) != hipSuccess) {
        (void)hipGetLastError();
        team_release(h);
    }
}

uint64_t team_offset(uint64_t scratch_bytes, uint64_t used, uint64_t need)
{
    if (need > scratch_bytes) return kTeamNoRoom;
    const uint64_t at = (scratch_bytes - need) / 256 * 256;
    return at >= used ? at : kTeamNoRoom;
}

bool team_disjoint(const mc_sim *h)
{
    return h->team_owned || h->lay.total <= (uint64_t)(h->team_ws - h->scratch);
}

hipError_t team_activate(mc_sim *h)
{
    // a tile chosen since may have taken the scratch up to its end, and the LDS
    // kernel keeps the layout of the tile before it
    if (!team_disjoint(h) && !team_own(h)) return hipSuccess; // the plain kernels go on
    // tags start above the zeroed words
    const hipError_t e =
        launch_zero_u32(h->team_state, (uint32_t)(h->team_off_part / sizeof(uint32_t)), h->stream);
    if (e != hipSuccess) return e;
    h->team_on = true;
    return hipMemcpyAsync(h->team_wgs, h->team_table.data(), sizeof(TeamWg) * h->team_table.size(),
                          hipMemcpyHostToDevice, h->stream);
}

mc_status team_resume(mc_sim *h)
{
    if (!h->team_ws || !same_tile(h->tile, h->default_tile)) return MC_OK;
    HIP_TRY(team_activate(h));
    HIP_TRY(hipStreamSynchronize(h->stream));
    return MC_OK;
}

void team_release(mc_sim *h)
{
    if (h->team_ws && h->team_owned) (void)hipFree(h->team_ws);
    h->team_ws = nullptr;
    h->team_on = false;
}

bool team_takes(const mc_sim *h, uint32_t n, bool measure)
{
    return h->team_on && n >= h->team_from[measure ? 1 : 0];
}

mc_status enqueue_team(mc_sim *h, uint32_t n, bool measure, uint32_t slot0, TeamHost host)
{
    TeamLaunch L;
    L.reps_dev = h->reps_dev;
    L.wgs = h->team_wgs;
    L.words = h->team_words;
    L.epoch = h->team_state;
    L.redone = h->team_state + 1;
    L.launch = h->team_state + 2;
    L.done = h->team_state + 3;
    L.ended = h->team_state + 4;
    L.left = L.ended + 2 * (size_t)h->n_reps;
    L.tctr_dev = h->tctr;
    L.partials = h->team_partials;
    L.records = h->records;
    L.n_reps = (uint32_t)h->n_reps;
    L.seed_lo = (uint32_t)h->seed;
    L.seed_hi = (uint32_t)(h->seed >> 32);
    L.ring = kRing;
    L.spin_limit = std::min(kTeamSpins, h->spin_limit);
    for (uint32_t done = 0; done < n;) {
        const uint32_t k = std::min(measure ? kTeamChunk : kTeamLong, n - done);
        L.n_sweeps = k;
        L.slot0 = (slot0 + done) % kRing;
        L.host_last = measure && host == TeamHost::last && done + k == n ? h->host_last : nullptr;
        L.host_ring = measure && host == TeamHost::all ? h->host_rec : nullptr;
        HIP_TRY(launch_team(h->kind, h->prec == MC_F64, measure, L, h->team_grid, h->team_threads,
                            h->team_lds, h->stream));
        done += k;
    }
    return MC_OK;
}

} // namespace mcabi

extern "C" mc_status mc_get_team(mc_sim *h, int32_t replica, int32_t *workgroups, int32_t *planes,
                                 int32_t *last_planes, uint32_t from_sweeps[2], uint64_t *redone)
{
    if (!alive(h)) return fail(MC_E_STATE, "invalid or destroyed handle");
    if (replica < 0 || replica >= h->n_reps)
        return fail(MC_E_ARG, "replica %d out of range [0, %d)", replica, h->n_reps);
    int32_t n = 0, first = 0, last = 0;
    if (h->team_on)
        for (const TeamWg &w : h->team_table)
            if (w.rep == (uint32_t)replica) {
                if (n++ == 0) first = w.nz;
                last = w.nz;
            }
    if (workgroups) *workgroups = n;
    if (planes) *planes = first;
    if (last_planes) *last_planes = last;
    if (from_sweeps)
        for (int m = 0; m < 2; ++m) from_sweeps[m] = h->team_on ? h->team_from[m] : kTeamNever;
    if (!redone) return MC_OK;
    *redone = 0;
    if (!h->team_on) return MC_OK;
    uint32_t v = 0;
    HIP_TRY(hipStreamSynchronize(h->stream));
    HIP_TRY(hipMemcpy(&v, h->team_state + 1, sizeof v, hipMemcpyDeviceToHost));
    *redone = v;
    return MC_OK;
}
