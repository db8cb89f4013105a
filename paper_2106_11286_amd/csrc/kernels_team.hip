// kernels_team.hip -- whole sweeps of small lattices by teams of workgroups:
// every replica's planes are dealt to the workgroups of its team, which hold
// them in LDS for the whole launch and exchange boundary planes through
// tagged words.
#include <mutex>
#include <type_traits>

#include "device_common.hpp"

namespace mc {

// ---------------------------------------------------------------------------
// Team sweeps.  A workgroup owns nz consecutive planes of one replica (all
// colours, in LDS, with a halo plane on either side) for n whole sweeps.
//
// Bound: a small lattice has a few microseconds of arithmetic per sweep, so a
// launch per colour pass pays mostly for launches (about 5 us each), and one
// workgroup per replica leaves most of the chip idle (sc 16^3 FP64: 14.9 us
// per sweep on one CU).  Here a colour phase costs one exchange between
// neighbouring workgroups, about 1 to 1.5 us wherever they run.
//
// Exchange.  After updating colour c a workgroup publishes the new spins of
// its boundary planes as 64-bit words, 32 bits of a component beside a 32-bit
// tag (launch epoch + phase), each one relaxed atomic store; its neighbours
// poll the words they need until the tag is the phase's.  A word carries its
// own arrival, so no fence, flag or cache operation is involved, and the two
// workgroups may sit on different XCDs.  A word of phase p is overwritten at
// phase p + NC: by then its owner has seen words of phase p or later from
// every reader, which published them after the workgroup barrier that ended
// its own reads of phase p.  Proposals do not depend on the spins and are
// drawn between the request for the words and their arrival (FP64: ahead of the
// request).
//
// The site updates are the other kernels' templates on the same values in the
// same order (a missing plane beyond an open face reads as zero, which adds
// exactly nothing), so the chain is bitwise theirs.
//
// Ending.  The workgroups of a team wait for each other, so all of them have to
// be running, and nothing reserves the GPU for them: other launches, of this
// process or another, may hold it.  So every wait is bounded and giving up costs
// time only.  Planes are written back when the whole team has finished; where a
// wait gives up before that, everybody leaves with the planes in memory as they
// were before the launch, and the last to leave does the launch's sweeps alone,
// in memory, waiting for nobody (TEAM_REDO).  The agreement is one more exchange
// per launch, about 1.4 us (17 x 24^3, 64 sweeps in two launches: 569 us without
// it, 576 with it).  A redone launch takes 4 to 11 times as long (24^3 x 17 26 us
// per sweep for 7.3, 50 x 38 x 23 91 for 8.0).
// ---------------------------------------------------------------------------
template <typename T> using lptr = __attribute__((address_space(3))) T *;

template <typename T> constexpr int team_words() { return sizeof(T) == 8 ? 6 : 3; }

__device__ __forceinline__ void publish(uint64_t *w, uint32_t stride, uint32_t tag, float x, float y,
                                        float z)
{
    const uint64_t t = (uint64_t)tag << 32;
    const float v[3] = {x, y, z};
#pragma unroll
    for (int a = 0; a < 3; ++a)
        __hip_atomic_store(w + (size_t)a * stride, t | __float_as_uint(v[a]), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish(uint64_t *w, uint32_t stride, uint32_t tag, double x,
                                        double y, double z)
{
    const uint64_t t = (uint64_t)tag << 32;
    const double v[3] = {x, y, z};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        __hip_atomic_store(w + (size_t)(2 * a) * stride, t | (uint32_t)__double2loint(v[a]),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(w + (size_t)(2 * a + 1) * stride, t | (uint32_t)__double2hiint(v[a]),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

template <typename T> struct Polled {
    uint64_t w[team_words<T>()];
};
template <typename T>
__device__ __forceinline__ void poll_issue(Polled<T> &q, const uint64_t *w, uint32_t stride)
{
#pragma unroll
    for (int a = 0; a < team_words<T>(); ++a)
        q.w[a] = __hip_atomic_load(w + (size_t)a * stride, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T> __device__ __forceinline__ bool poll_ready(const Polled<T> &q, uint32_t tag)
{
    bool ok = true;
#pragma unroll
    for (int a = 0; a < team_words<T>(); ++a) ok &= (uint32_t)(q.w[a] >> 32) == tag;
    return ok;
}
__device__ __forceinline__ Vec3<float> polled_spin(const Polled<float> &q)
{
    return {__uint_as_float((uint32_t)q.w[0]), __uint_as_float((uint32_t)q.w[1]),
            __uint_as_float((uint32_t)q.w[2])};
}
__device__ __forceinline__ Vec3<double> polled_spin(const Polled<double> &q)
{
    return {__hiloint2double((int)(uint32_t)q.w[1], (int)(uint32_t)q.w[0]),
            __hiloint2double((int)(uint32_t)q.w[3], (int)(uint32_t)q.w[2]),
            __hiloint2double((int)(uint32_t)q.w[5], (int)(uint32_t)q.w[4])};
}

// How a team's launch ends: a count of the workgroups that have finished, which
// commits when it reaches all of them, or with TEAM_REDO set before that, which
// nothing undoes.
constexpr uint32_t TEAM_REDO = 0x80000000u;
__device__ __forceinline__ uint32_t load_word(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool team_settled(uint32_t v, uint32_t members)
{
    return v == members || (v & TEAM_REDO) != 0u;
}
// Ask for a redo; returns what it has come to.
__device__ __forceinline__ uint32_t team_give_up(uint32_t *ended, uint32_t members)
{
    uint32_t v = load_word(ended);
    while (!team_settled(v, members))
        if (__hip_atomic_compare_exchange_strong(ended, &v, v | TEAM_REDO, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            v |= TEAM_REDO;
    return v;
}

// Field at a site of colour c (J not applied) and, for the basis lattices, its
// part of the shared bonds.  The planes begin at x, y, z, `plane` elements per
// colour.
template <typename T> struct SiteField {
    T hx = 0, hy = 0, hz = 0, sh_x = 0, sh_y = 0, sh_z = 0;
};
template <typename T, int KIND, typename P>
__device__ __forceinline__ SiteField<T> team_field(P x, P y, P z, uint32_t plane, int c, int Lx,
                                                   int Lxh, int Ly, int Lz, bool px, bool py,
                                                   bool pz, int xh, int yy, int zz, int p)
{
    constexpr int NB = basis_count(KIND);
    SiteField<T> f;
    if constexpr (KIND == SC) {
        sc_site_field<T>(x, y, z, c ? 0u : plane, Lxh, Ly, Lz, px, py, pz, xh, yy, zz, p, f.hx,
                         f.hy, f.hz);
        return f;
    } else {
        auto of = [&](auto basis) __attribute__((always_inline)) {
            constexpr int B = decltype(basis)::value < NB ? decltype(basis)::value : 0;
            SiteField<T> g;
            basis_site_field<KIND, B, T>(x, y, z, plane, Lx, Ly, Lz, px, py, pz, xh, yy, zz, g.hx,
                                         g.hy, g.hz, g.sh_x, g.sh_y, g.sh_z);
            return g;
        };
        switch (c) {
        case 0: return of(std::integral_constant<int, 0>());
        case 1: return of(std::integral_constant<int, 1>());
        case 2: return of(std::integral_constant<int, 2>());
        default: return of(std::integral_constant<int, 3>());
        }
    }
}

template <typename T, int KIND, bool MEASURE>
__global__ void __launch_bounds__(TEAM_THREADS, sizeof(T) == 8 ? 2 : 4) k_team_sweeps(TeamLaunch L)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    __shared__ double red[TEAM_THREADS / 64][NQ];
    __shared__ uint32_t s_abort[2], s_last, s_commit; // s_abort: a wait gave up, per phase parity
    constexpr int NB = basis_count(KIND);
    constexpr int NC = KIND == SC ? 2 : NB;
    constexpr int NW = team_words<T>();
    const TeamWg w = L.wgs[blockIdx.x];
    const RepDev &R = L.reps_dev[w.rep];
    const int Lx = R.Lx, Ly = R.Ly, Lz = R.Lz, Lxh = R.Lxh, nz = w.nz, nzl = nz + 2;
    const bool sphere = R.sphere;
    const double r2x4 = R.r2x4;
    const uint32_t plane = R.plane, rid = R.rid;
    const gptr<T> gx = as_global<T>(R.sx), gy = as_global<T>(R.sy), gz = as_global<T>(R.sz);
    const T J = (T)R.J, K = (T)R.K, ex = (T)R.e[0], ey = (T)R.e[1], ez = (T)R.e[2];
    const T beta = (T)R.beta;
    const double Jd = R.J, Kd = R.K;
    const bool greedy = R.greedy != 0;
    const bool px = R.pmask & 1u, py = R.pmask & 2u;
    const uint32_t t0 = *L.tctr_dev, epoch = *L.epoch, launch = *L.launch;
    const uint32_t row = (uint32_t)Lxh, psites = row * (uint32_t)Ly; // one colour of one plane
    const uint32_t own = psites * (uint32_t)nz, lplane = psites * (uint32_t)nzl;
    const FastDiv f_row = fast_div(row), f_y = fast_div((uint32_t)Ly);
    const lptr<T> lx = (lptr<T>)(lptr<unsigned char>)lds_raw;
    const lptr<T> ly = lx + NC * lplane, lz = ly + NC * lplane;
    const uint32_t tid = threadIdx.x, nt = blockDim.x;
    if (tid < 2) s_abort[tid] = 0;

    // the owned planes and the halo planes as they are before the launch
    // (a neighbour writes its planes back only after its last phase, which
    // needs words published after this load)
    // several elements' loads are in flight at a time
    auto fill = [&](uint32_t n, auto source) __attribute__((always_inline)) {
        constexpr int U = 4;
        for (uint32_t i0 = tid; i0 < n; i0 += U * nt) {
            Vec3<T> v[U];
            uint32_t dst[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t i = i0 + (uint32_t)u * nt;
                uint32_t g = 0;
                const bool there = i < n && source(i, g, dst[u]);
                v[u] = {T(0), T(0), T(0)};
                if (there) v[u] = {gx[g], gy[g], gz[g]};
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i0 + (uint32_t)u * nt < n) {
                    lx[dst[u]] = v[u].x;
                    ly[dst[u]] = v[u].y;
                    lz[dst[u]] = v[u].z;
                }
        }
    };
    for (int c = 0; c < NC; ++c) {
        const uint32_t gsrc = (uint32_t)c * plane, ldst = (uint32_t)c * lplane;
        fill(own, [&](uint32_t i, uint32_t &g, uint32_t &l) {
            g = gsrc + (uint32_t)w.z0 * psites + i;
            l = ldst + psites + i;
            return true;
        });
        if (c == 0) continue; // colour 0 is updated before its halo is first read
        fill(2 * psites, [&](uint32_t i, uint32_t &g, uint32_t &l) {
            const bool up = i >= psites;
            const uint32_t k = up ? i - psites : i;
            const int z = up ? w.z_hi : w.z_lo;
            l = ldst + (up ? (uint32_t)(nz + 1) * psites : 0u) + k;
            g = gsrc + (uint32_t)(z < 0 ? 0 : z) * psites + k;
            return z >= 0;
        });
    }
    // beyond an open face colour 0 reads as zero, too
    for (uint32_t i = tid; i < psites; i += nt) {
        if (w.z_lo < 0) lx[i] = ly[i] = lz[i] = T(0);
        const uint32_t l = (uint32_t)(nz + 1) * psites + i;
        if (w.z_hi < 0) lx[l] = ly[l] = lz[l] = T(0);
    }
    uint64_t *const words = L.words + w.words;
    // two words per team, used in turn
    uint32_t *const ended = L.ended + 2u * w.rep + (launch & 1u);
    const uint32_t slot_words = (uint32_t)(NC * NW) * psites;
    // halo sites polled per phase: the plane below, then the plane above
    const uint32_t n_lo = w.lo >= 0 ? psites : 0u, n_poll = n_lo + (w.hi >= 0 ? psites : 0u);
    const uint32_t n_phases = L.n_sweeps * (uint32_t)NC;

    // site k of colour c of planes z0, z0 + 1, ...
    struct Site {
        uint32_t s; // canonical index
        int xh, y, zl, p;
        bool occ;
    };
    auto locate = [&](int z0, int c, uint32_t k) -> Site {
        Site q;
        const uint32_t r = div_of(k, f_row);
        q.xh = (int)(k - r * row);
        const uint32_t zz = div_of(r, f_y);
        q.y = (int)(r - zz * (uint32_t)Ly);
        q.zl = (int)zz;
        const int z = z0 + q.zl;
        int x2 = 0, y2 = 2 * q.y - Ly, z2 = 2 * z - Lz; // half cells from the centre
        if constexpr (KIND == SC) {
            q.p = (c + q.y + z) & 1;
            q.s = ((uint32_t)z0 * (uint32_t)Ly + r) * (uint32_t)Lx + 2u * (uint32_t)q.xh +
                  (uint32_t)q.p;
            x2 = 2 * (2 * q.xh + q.p) - Lx;
        } else {
            q.p = 0;
            q.s = ((uint32_t)z0 * psites + k) * (uint32_t)NB + (uint32_t)c;
            x2 = 2 * q.xh + (KIND == FCC ? (int)(c == 1 || c == 2) : c) - Lx;
            y2 += KIND == FCC ? (int)(c == 1 || c == 3) : c;
            z2 += KIND == FCC ? (int)(c >= 2) : c;
        }
        q.occ = !sphere || (double)(x2 * x2 + y2 * y2 + z2 * z2) <= r2x4;
        return q;
    };
    // its decision and its part of the sums
    auto attempt = [&](const Proposal<T> &pr, int c, T &sx, T &sy, T &sz, const SiteField<T> &f,
                       double (&acc)[Q_N]) __attribute__((always_inline)) -> bool {
        const T hx = f.hx * J, hy = f.hy * J, hz = f.hz * J;
        T dH;
        const bool a = decide<T>(pr, sx, sy, sz, hx, hy, hz, K, ex, ey, ez, beta, greedy, dH);
        if (MEASURE) {
            if constexpr (KIND == SC)
                observe<T>(acc, sx, sy, sz, ex, ey, ez, c == 1, hx, hy, hz, 1.0);
            else
                observe<T>(acc, sx, sy, sz, ex, ey, ez, true, f.sh_x, f.sh_y, f.sh_z, Jd);
            acc[Q_NACC] += a ? 1.0 : 0.0;
        }
        return a;
    };
    // a sweep's sums over the workgroup (waves in order), into its partial slot
    auto store_sums = [&](const double (&acc)[Q_N], uint32_t sw, uint32_t wg) {
        store_wave_sums(acc, red[tid >> 6]);
        __syncthreads();
        if (tid < Q_N) {
            double v = 0.0;
            for (uint32_t i = 0; i < (nt + 63u) / 64u; ++i) v += red[i][tid];
            double *p = L.partials + ((size_t)sw * gridDim.x + wg) * NQ + tid;
            __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };

    bool alive = true;
    uint32_t phase = 0;
    for (uint32_t sw = 0; sw < L.n_sweeps && alive; ++sw) {
        const uint32_t t = t0 + sw;
        double acc[Q_N] = {0, 0, 0, 0, 0, 0};
        // one copy of the phase for every colour (the code stays small)
#pragma clang loop unroll(disable)
        for (int c = 0; c < NC && alive; ++c, ++phase) {
            const int cp = c == 0 ? NC - 1 : c - 1; // the colour updated last
            const bool mine = phase > 0 && tid < n_poll;
            // word 0 of halo site i (32-bit offsets from the team's words)
            const uint32_t off_lo = (uint32_t)w.lo * slot_words + (uint32_t)(cp * NW) * psites;
            const uint32_t off_hi =
                (uint32_t)w.hi * slot_words + (uint32_t)(cp * NW) * psites - n_lo;
            const uint32_t want = epoch + phase; // tag of phase - 1
            // two sites' words are in flight at a time
            Polled<T> q0, q1;
            auto request = [&](uint32_t i) __attribute__((always_inline)) {
                poll_issue<T>(q0, words + (i + (i >= n_lo ? off_hi : off_lo)), psites);
                // a thread without a second site reads its first one again
                const uint32_t j = i + nt < n_poll ? i + nt : i;
                poll_issue<T>(q1, words + (j + (j >= n_lo ? off_hi : off_lo)), psites);
            };
            auto keep = [&](const Polled<T> &q, uint32_t i) __attribute__((always_inline)) {
                const Vec3<T> v = polled_spin(q);
                const uint32_t l = (uint32_t)cp * lplane + (i >= n_lo ? own + psites - n_lo : 0u) + i;
                lx[l] = v.x;
                ly[l] = v.y;
                lz[l] = v.z;
            };
            // Request this thread's first halo words, draw its first site's
            // proposal meanwhile, then wait for the words.  An FP64 proposal
            // takes longer than the neighbours need: words asked for before it
            // come back old and are asked for again, so FP64 asks after it.
            // us per sweep, before / after: FP32 24^3 x 17 7.12 / 7.88,
            // 50x37x23 8.22 / 8.50; FP64 16^3 4.87 / 4.61, 20^3 x 3 5.34 / 4.97,
            // fcc 16^3 13.3 / 12.8.
            constexpr bool ask_first = sizeof(T) == 4;
            if constexpr (ask_first)
                if (mine) request(tid);
            uint32_t k = tid;
            bool first = true;
#pragma clang loop unroll(disable)
            do {
                Site st = {};
                Proposal<T> pr = {};
                if (k < own) {
                    st = locate(w.z0, c, k);
                    pr = propose<T>(philox10(st.s, rid, t, 0u, L.seed_lo, L.seed_hi));
                }
                if (first) {
                    first = false;
                    if (mine) {
                        if constexpr (!ask_first) request(tid);
#pragma clang loop unroll(disable)
                        for (uint32_t i = tid;;) {
                            bool here = true;
                            for (uint32_t spins = 1;
                                 !(poll_ready<T>(q0, want) && poll_ready<T>(q1, want)); ++spins) {
                                if (spins > L.spin_limit ||
                                    ((spins & 255u) == 0u &&
                                     (load_word(ended) & TEAM_REDO) != 0u)) {
                                    here = false;
                                    break;
                                }
                                request(i);
                            }
                            if (!here) {
                                s_abort[phase & 1u] = 1;
                                break;
                            }
                            keep(q0, i);
                            if (i + nt < n_poll) keep(q1, i + nt);
                            i += 2 * nt;
                            if (i >= n_poll) break;
                            request(i);
                        }
                    }
                    __syncthreads();
                    if (w.members == 1 && w.z_lo >= 0) {
                        // one workgroup holds the whole periodic lattice: its
                        // own outer planes are each other's halo
                        for (uint32_t i = tid; i < 2 * psites; i += nt) {
                            const bool up = i >= psites;
                            const uint32_t b = (uint32_t)cp * lplane + (up ? i - psites : i);
                            const uint32_t src = b + (up ? psites : own);
                            const uint32_t dst = b + (up ? own + psites : 0u);
                            lx[dst] = lx[src];
                            ly[dst] = ly[src];
                            lz[dst] = lz[src];
                        }
                        __syncthreads();
                    }
                    if (s_abort[phase & 1u]) { // the same for the whole workgroup
                        alive = false;
                        break;
                    }
                }
                if (k < own) {
                    const uint32_t at = (uint32_t)c * lplane + psites + k;
                    T sx = lx[at], sy = ly[at], sz = lz[at];
                    if (st.occ) {
                        // planes 1 .. nz of the held ones never wrap
                        const SiteField<T> f =
                            team_field<T, KIND>(lx, ly, lz, lplane, c, Lx, Lxh, Ly, nzl, px, py,
                                                true, st.xh, st.y, st.zl + 1, st.p);
                        if (attempt(pr, c, sx, sy, sz, f, acc)) {
                            lx[at] = sx;
                            ly[at] = sy;
                            lz[at] = sz;
                        }
                    }
                    // boundary planes for the neighbours (unoccupied sites
                    // too: a neighbour waits for every word of the plane)
                    const uint32_t tag = epoch + phase + 1u;
                    if (st.zl == 0 && w.own_lo >= 0)
                        publish(words + (size_t)(uint32_t)w.own_lo * slot_words +
                                    (size_t)(uint32_t)(c * NW) * psites + k,
                                psites, tag, sx, sy, sz);
                    if (st.zl == nz - 1 && w.own_hi >= 0 && w.own_hi != w.own_lo)
                        publish(words + (size_t)(uint32_t)w.own_hi * slot_words +
                                    (size_t)(uint32_t)(c * NW) * psites + (k - (own - psites)),
                                psites, tag, sx, sy, sz);
                }
                k += nt;
            } while (k < own);
        }
        if (MEASURE && alive) store_sums(acc, sw, blockIdx.x);
    }
    __syncthreads();
    // Commit or redo.  s_last: the last of the team to get here, which turns its
    // sums into records.  The sums were stored by agent-scope atomics by wave 0,
    // whose thread 0 waits for them before it counts.
    if (tid == 0) {
        bool last = true, commit = true;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0x0F70); // vmcnt 0
        if (w.members > 1u) {
            uint32_t v;
            if (alive && L.spin_limit > 0u) { // no budget: nobody waits, not even briefly
                v = __hip_atomic_fetch_add(ended, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) +
                    1u;
                last = v == w.members;
                for (uint32_t spins = 1; !team_settled(v, w.members); ++spins)
                    v = spins > L.spin_limit ? team_give_up(ended, w.members) : load_word(ended);
            } else {
                v = team_give_up(ended, w.members);
            }
            commit = v == w.members;
            if (!commit) {
                uint32_t *const left = L.left + w.rep;
                last = __hip_atomic_fetch_add(left, 1u, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT) + 1u == w.members;
                if (last) {
                    __hip_atomic_store(left, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_fetch_add(L.redone, 1u, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            // the next launch's word, which nobody reads yet
            if (last)
                __hip_atomic_store(L.ended + 2u * w.rep + ((launch & 1u) ^ 1u), 0u,
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        s_last = last;
        s_commit = commit;
    }
    __syncthreads();
    if (s_commit) {
        for (int c = 0; c < NC; ++c)
            for (uint32_t i = tid; i < own; i += nt) {
                const uint32_t g = (uint32_t)c * plane + (uint32_t)w.z0 * psites + i;
                const uint32_t l = (uint32_t)c * lplane + psites + i;
                gx[g] = lx[l];
                gy[g] = ly[l];
                gz[g] = lz[l];
            }
    } else if (s_last) {
        // the whole replica, colour by colour, in memory; its sums as those of
        // the team's first workgroup, the others' zero
        const bool pz = R.pmask & 4u;
        for (uint32_t sw = 0; sw < L.n_sweeps; ++sw) {
            double acc[Q_N] = {0, 0, 0, 0, 0, 0};
#pragma clang loop unroll(disable)
            for (int c = 0; c < NC; ++c) {
#pragma clang loop unroll(disable)
                for (uint32_t k = tid; k < plane; k += nt) {
                    const Site st = locate(0, c, k);
                    if (!st.occ) continue;
                    const Proposal<T> pr =
                        propose<T>(philox10(st.s, rid, t0 + sw, 0u, L.seed_lo, L.seed_hi));
                    const uint32_t at = (uint32_t)c * plane + k;
                    T sx = gx[at], sy = gy[at], sz = gz[at];
                    const SiteField<T> f =
                        team_field<T, KIND>(gx, gy, gz, plane, c, Lx, Lxh, Ly, Lz, px, py, pz, st.xh,
                                            st.y, st.zl, st.p);
                    if (attempt(pr, c, sx, sy, sz, f, acc)) {
                        gx[at] = sx;
                        gy[at] = sy;
                        gz[at] = sz;
                    }
                }
                __syncthreads();
            }
            if (MEASURE) {
                store_sums(acc, sw, w.first);
                if (tid < Q_N)
                    for (uint32_t m = 1; m < w.members; ++m)
                        __hip_atomic_store(L.partials + ((size_t)sw * gridDim.x + w.first + m) * NQ +
                                               tid,
                                           0.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (MEASURE && tid < 64u) { // wave 0 stored the sums
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_s_waitcnt(0x0F70); // vmcnt 0
        }
    }
    __syncthreads();
    if (MEASURE && s_last) {
        for (uint32_t j = tid; j < L.n_sweeps * 8u; j += nt) {
            const uint32_t sw = j >> 3, i = j & 7u;
            const uint32_t src = i == R_MX   ? (uint32_t)Q_MX
                                 : i == R_MY ? (uint32_t)Q_MY
                                 : i == R_MZ ? (uint32_t)Q_MZ
                                 : i == R_EEX ? (uint32_t)Q_SH
                                 : i == R_EAN ? (uint32_t)Q_PE2
                                              : (uint32_t)Q_NACC;
            double v = 0.0;
            if (i <= (uint32_t)R_NACC) {
                const double *p = L.partials + ((size_t)sw * gridDim.x + w.first) * NQ + src;
                for (uint32_t m = 0; m < w.members; ++m)
                    v += __hip_atomic_load(p + (size_t)m * NQ, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
            }
            if (i == (uint32_t)R_EEX) v = -v;
            if (i == (uint32_t)R_EAN) v = -Kd * v;
            if (i == (uint32_t)R_SWEEP) v = (double)(t0 + sw) + 1.0;
            if (i == 7u) v = 0.0;
            const size_t at = ((size_t)((L.slot0 + sw) % L.ring) * L.n_reps + w.rep) * NR + i;
            L.records[at] = v;
            if (L.host_ring) L.host_ring[at] = v;
            if (L.host_last && sw + 1u == L.n_sweeps) L.host_last[(size_t)w.rep * NR + i] = v;
        }
    }
    if (tid == 0) {
        const uint32_t old = __hip_atomic_fetch_add(L.done, 1u, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
        if (old + 1u == gridDim.x) {
            __hip_atomic_store(L.done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *L.tctr_dev = t0 + L.n_sweeps;
            *L.epoch = epoch + n_phases;
            *L.launch = launch + 1u;
        }
    }
}

template <typename T, int KIND> static const void *team_fn(bool measure)
{
    return measure ? (const void *)&k_team_sweeps<T, KIND, true>
                   : (const void *)&k_team_sweeps<T, KIND, false>;
}
static const void *team_kernel(int kind, bool f64, bool measure)
{
    switch (kind) {
    case SC: return f64 ? team_fn<double, SC>(measure) : team_fn<float, SC>(measure);
    case BCC: return f64 ? team_fn<double, BCC>(measure) : team_fn<float, BCC>(measure);
    default: return f64 ? team_fn<double, FCC>(measure) : team_fn<float, FCC>(measure);
    }
}

hipError_t launch_team(int kind, bool f64, bool measure, const TeamLaunch &L, uint32_t grid,
                       int threads, uint32_t lds_bytes, hipStream_t st)
{
    if (grid == 0 || L.n_sweeps == 0) return hipSuccess;
    if (kind < 0 || kind > 2 || threads < 64 || threads > TEAM_THREADS || threads % 64)
        return hipErrorInvalidValue;
    TeamLaunch a = L;
    void *args[] = {&a};
    return hipLaunchKernel(team_kernel(kind, f64, measure), dim3(grid), dim3(threads), args,
                           lds_bytes, st);
}

// Dynamic LDS beyond the default limit has to be allowed per kernel (and
// device); the allowance is shared by every handle and only ever raised.
hipError_t team_allow(int kind, bool f64, uint32_t bytes)
{
    static std::mutex mu;
    static uint32_t allowed[64][3][2];
    if (kind < 0 || kind > 2) return hipErrorInvalidValue;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    uint32_t &a = allowed[dev][kind][f64 ? 1 : 0];
    if (bytes <= a) return hipSuccess;
    for (bool measure : {false, true}) {
        e = hipFuncSetAttribute(team_kernel(kind, f64, measure),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) return e;
    }
    a = bytes;
    return hipSuccess;
}

hipError_t team_slots(int kind, bool f64, int threads, uint32_t lds_bytes, int *per_cu)
{
    *per_cu = 1 << 30;
    for (bool measure : {false, true}) {
        int n = 0;
        const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &n, team_kernel(kind, f64, measure), threads, lds_bytes);
        if (e != hipSuccess) return e;
        if (n < *per_cu) *per_cu = n;
    }
    return hipSuccess;
}

} // namespace mc
