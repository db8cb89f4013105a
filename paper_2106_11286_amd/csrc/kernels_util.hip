// kernels_util.hip -- initial state, layout conversion, the observable
// finalise, counters, fills and the memory-pattern probe.
#include "device_common.hpp"

namespace mc {

// ---------------------------------------------------------------------------
// Initial state and layout conversion (one replica per launch).
// ---------------------------------------------------------------------------
struct SiteCoord {
    int x, y, z, b;
    uint32_t s; // canonical index
};

__device__ __forceinline__ SiteCoord decode(const RepDev &R, int kind, uint32_t i)
{
    SiteCoord c;
    const uint32_t colour = i / R.plane, j = i - colour * R.plane;
    if (kind == SC) {
        const uint32_t xh = j % (uint32_t)R.Lxh, r = j / (uint32_t)R.Lxh;
        c.y = (int)(r % (uint32_t)R.Ly);
        c.z = (int)(r / (uint32_t)R.Ly);
        c.x = 2 * (int)xh + (int)((colour + c.y + c.z) & 1u);
        c.b = 0;
        c.s = (uint32_t)(c.z * R.Ly + c.y) * (uint32_t)R.Lx + c.x;
    } else {
        c.x = (int)(j % (uint32_t)R.Lx);
        const uint32_t r = j / (uint32_t)R.Lx;
        c.y = (int)(r % (uint32_t)R.Ly);
        c.z = (int)(r / (uint32_t)R.Ly);
        c.b = (int)colour;
        c.s = j * (uint32_t)basis_count(kind) + colour;
    }
    return c;
}

__device__ __forceinline__ bool occupied_site(const RepDev &R, int kind, const SiteCoord &c)
{
    int bx = 0, by = 0, bz = 0;
    if (kind == BCC) bx = by = bz = c.b;
    if (kind == FCC) {
        bx = c.b == 1 || c.b == 2;
        by = c.b == 1 || c.b == 3;
        bz = c.b == 2 || c.b == 3;
    }
    return occupied(R, c.x, c.y, c.z, bx, by, bz);
}

template <typename T>
__global__ void __launch_bounds__(256)
k_init(RepDev R, int kind, int mode, uint32_t k0, uint32_t k1)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < R.n_box;
         i += gridDim.x * blockDim.x) {
        const SiteCoord c = decode(R, kind, i);
        T vx = 0, vy = 0, vz = 0;
        if (occupied_site(R, kind, c)) {
            if (mode == 1) {
                vx = (T)R.e[0];
                vy = (T)R.e[1];
                vz = (T)R.e[2];
            } else {
                const Words w = philox10(c.s, R.rid, 0u, 1u, k0, k1);
                sphere_point(uniform23<T>(w.w0), uniform23<T>(w.w1), vx, vy, vz);
            }
        }
        ((T *)R.sx)[i] = vx;
        ((T *)R.sy)[i] = vy;
        ((T *)R.sz)[i] = vz;
    }
}

// Layout conversion, bound by its streams (every spin read once and written
// once).  Simple cubic: packed column j of either colour is the pair of
// natural sites 2j, 2j+1, whose order the row's parity gives, so a thread
// converts V consecutive columns with 16-byte accesses on both sides (V = 1
// where a colour plane is no multiple of V columns).  One element per thread
// with stride-2 natural accesses and four integer divisions took 114 us on a
// 16 M-site film, FP32; this takes 64 with V = 1 (6.0 TB/s).
template <typename T, int V> struct alignas(sizeof(T) * V) Pack {
    T v[V];
};
template <typename T, int V>
__global__ void __launch_bounds__(256)
k_layout_sc(RepDev R, Div31 d_lxh, Div31 d_ly, int to_natural, T *nx, T *ny, T *nz)
{
    const uint32_t n = R.plane / V, stride = gridDim.x * blockDim.x;
    T *const packed[3] = {(T *)R.sx, (T *)R.sy, (T *)R.sz};
    T *const natural[3] = {nx, ny, nz};
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint32_t j = i * V;
        bool odd[V]; // the even column holds colour 1
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const uint32_t row = div31(j + k, d_lxh), z = div31(row, d_ly);
            odd[k] = ((row - z * (uint32_t)R.Ly + z) & 1u) != 0;
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            T *const c0 = packed[a] + j, *const c1 = c0 + R.plane, *const nat = natural[a] + 2 * (size_t)j;
            Pack<T, V> p0, p1, q0, q1; // q0, q1: the natural run of 2 V sites
            if (to_natural) {
                p0 = *(const Pack<T, V> *)c0;
                p1 = *(const Pack<T, V> *)c1;
#pragma unroll
                for (int k = 0; k < V; ++k) {
                    const T even = odd[k] ? p1.v[k] : p0.v[k], other = odd[k] ? p0.v[k] : p1.v[k];
                    (2 * k < V ? q0 : q1).v[2 * k % V] = even;
                    (2 * k + 1 < V ? q0 : q1).v[(2 * k + 1) % V] = other;
                }
                *(Pack<T, V> *)nat = q0;
                *(Pack<T, V> *)(nat + V) = q1;
            } else {
                q0 = *(const Pack<T, V> *)nat;
                q1 = *(const Pack<T, V> *)(nat + V);
#pragma unroll
                for (int k = 0; k < V; ++k) {
                    const T even = (2 * k < V ? q0 : q1).v[2 * k % V];
                    const T other = (2 * k + 1 < V ? q0 : q1).v[(2 * k + 1) % V];
                    p0.v[k] = odd[k] ? other : even;
                    p1.v[k] = odd[k] ? even : other;
                }
                *(Pack<T, V> *)c0 = p0;
                *(Pack<T, V> *)c1 = p1;
            }
        }
    }
}
// bcc / fcc: a cell's NB sites are consecutive in natural order (one vector
// access) and one element of each basis plane (coalesced over the cells).
template <typename T, int NB>
__global__ void __launch_bounds__(256)
k_layout_basis(RepDev R, int to_natural, T *nx, T *ny, T *nz)
{
    const uint32_t stride = gridDim.x * blockDim.x;
    T *const packed[3] = {(T *)R.sx, (T *)R.sy, (T *)R.sz};
    T *const natural[3] = {nx, ny, nz};
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < R.plane; i += stride)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            Pack<T, NB> *const nat = (Pack<T, NB> *)natural[a] + i;
            Pack<T, NB> q;
            if (to_natural) {
#pragma unroll
                for (int b = 0; b < NB; ++b) q.v[b] = packed[a][(size_t)b * R.plane + i];
                *nat = q;
            } else {
                q = *nat;
#pragma unroll
                for (int b = 0; b < NB; ++b) packed[a][(size_t)b * R.plane + i] = q.v[b];
            }
        }
}

// ---------------------------------------------------------------------------
// Finalise: `blocks` workgroups per replica each sum a contiguous share of the
// replica's partial slots (all passes); with more than one, the last of them to
// finish sums their shares in index order.  The result depends only on the
// work list and the number of workgroups.
//
// One launch (4.5 us) where a second one for the last step cost as much again.
// The shares travel as agent-scope atomic stores that their wave waits for
// before it counts itself (at most 32 counts per replica): no fence, whose
// write-back of the L2 in every workgroup once made a single launch 159 us on
// 64 replicas.  The count is kept beside the replica's first share.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
k_finalize(const RepDev *__restrict__ reps, int n_colours, uint32_t blocks,
           const double *__restrict__ partials, uint32_t n_items,
           const uint32_t *__restrict__ tctr, uint32_t t_add, double *stage,
           double *__restrict__ records, double *host_last)
{
    __shared__ double red[4][Q_N], out[Q_N];
    __shared__ uint32_t s_last;
    const uint32_t r = blockIdx.x / blocks, j = blockIdx.x % blocks, q = threadIdx.x;
    const RepDev &R = reps[r];
    const uint32_t n = R.item_end - R.item_begin;
    const uint32_t b0 = R.item_begin + (uint32_t)(((uint64_t)n * j) / blocks);
    const uint32_t b1 = R.item_begin + (uint32_t)(((uint64_t)n * (j + 1)) / blocks);
    double a[Q_N] = {0, 0, 0, 0, 0, 0};
    for (int c = 0; c < n_colours; ++c)
        for (uint32_t it = b0 + threadIdx.x; it < b1; it += blockDim.x) {
            const double *p = partials + ((size_t)c * n_items + it) * NQ;
#pragma unroll
            for (int i = 0; i < Q_N; ++i) a[i] += p[i];
        }
    store_wave_sums(a, red[threadIdx.x >> 6]);
    __syncthreads();
    double *const share = stage + (size_t)r * FIN_BLOCKS * NQ;
    if (q < (uint32_t)Q_N) {
        double v = 0.0;
        for (int w = 0; w < 4; ++w) v += red[w][q];
        if (blocks == 1u) out[q] = v;
        else
            __hip_atomic_store(share + (size_t)j * NQ + q, v, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
    if (blocks > 1u) {
        if (q == 0) {
            // the shares were stored by this wave
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_s_waitcnt(0x0F70); // vmcnt 0
            uint32_t *const count = (uint32_t *)(share + NQ - 1);
            const uint32_t old = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT);
            s_last = old + 1u == blocks;
            if (s_last)
                __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (!s_last) return;
        if (q < (uint32_t)Q_N) {
            // every load is issued before the first add
            double v[FIN_BLOCKS];
#pragma unroll
            for (uint32_t b = 0; b < FIN_BLOCKS; ++b)
                v[b] = b < blocks ? __hip_atomic_load(share + b * NQ + q, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT)
                                  : 0.0;
            double sum = 0.0;
#pragma unroll
            for (uint32_t b = 0; b < FIN_BLOCKS; ++b) sum += v[b];
            out[q] = sum;
        }
    }
    __syncthreads();
    if (q >= (uint32_t)NR) return;
    const double v = q == R_MX     ? out[Q_MX]
                     : q == R_MY   ? out[Q_MY]
                     : q == R_MZ   ? out[Q_MZ]
                     : q == R_EEX  ? -out[Q_SH]
                     : q == R_EAN  ? -R.K * out[Q_PE2]
                     : q == R_NACC ? out[Q_NACC]
                     : q == R_SWEEP ? (double)(*tctr + t_add)
                                    : 0.0;
    records[(size_t)r * NR + q] = v;
    if (host_last) host_last[(size_t)r * NR + q] = v;
}

__global__ void k_advance(uint32_t *tctr, uint32_t n)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *tctr += n;
}

__global__ void k_set_counter(uint32_t *tctr, uint32_t v)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *tctr = v;
}

__global__ void k_fill_zero(double *p, uint64_t n)
{
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = 0.0;
}

// ---------------------------------------------------------------------------
// Memory-pattern probe: the HBM streams of one colour pass without its
// arithmetic.  Three component arrays of 2 P elements; the first half is read
// and written in place, the second half read (24 B read and 12 B written per
// FP32 element of the first half), two elements per lane per access.
// ---------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256) k_stream_probe(T *x, T *y, T *z, uint64_t P)
{
    const uint64_t n2 = P / 2; // element pairs per half
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n2;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t a = 2 * i, b = P + 2 * i;
        const T x0 = x[a] + x[b], x1 = x[a + 1] + x[b + 1];
        const T y0 = y[a] + y[b], y1 = y[a + 1] + y[b + 1];
        const T z0 = z[a] + z[b], z1 = z[a + 1] + z[b + 1];
        x[a] = x0;
        x[a + 1] = x1;
        y[a] = y0;
        y[a + 1] = y1;
        z[a] = z0;
        z[a + 1] = z1;
    }
}

static unsigned grid_for(uint32_t n)
{
    uint32_t g = (n + 255) / 256;
    return g < 8192 ? (g ? g : 1) : 8192;
}

hipError_t launch_init(bool f64, int kind, const RepDev *rep_host, int mode, uint32_t seed_lo,
                       uint32_t seed_hi, hipStream_t st)
{
    const unsigned g = grid_for(rep_host->n_box);
    if (f64)
        hipLaunchKernelGGL((k_init<double>), dim3(g), dim3(256), 0, st, *rep_host, kind, mode,
                           seed_lo, seed_hi);
    else
        hipLaunchKernelGGL((k_init<float>), dim3(g), dim3(256), 0, st, *rep_host, kind, mode,
                           seed_lo, seed_hi);
    return hipGetLastError();
}

template <typename T>
static hipError_t layout_dispatch(int kind, const RepDev &R, bool to_natural, T *nx, T *ny, T *nz,
                                  hipStream_t st)
{
    constexpr int V = 16 / (int)sizeof(T);
    const int nat = (int)to_natural;
    if (kind == SC) {
        const Div31 dx = make_div31((uint32_t)R.Lxh), dy = make_div31((uint32_t)R.Ly);
        if (R.plane % V == 0)
            hipLaunchKernelGGL((k_layout_sc<T, V>), dim3(grid_for(R.plane / V)), dim3(256), 0, st, R,
                               dx, dy, nat, nx, ny, nz);
        else
            hipLaunchKernelGGL((k_layout_sc<T, 1>), dim3(grid_for(R.plane)), dim3(256), 0, st, R, dx,
                               dy, nat, nx, ny, nz);
    } else if (kind == BCC) {
        hipLaunchKernelGGL((k_layout_basis<T, 2>), dim3(grid_for(R.plane)), dim3(256), 0, st, R, nat,
                           nx, ny, nz);
    } else {
        hipLaunchKernelGGL((k_layout_basis<T, 4>), dim3(grid_for(R.plane)), dim3(256), 0, st, R, nat,
                           nx, ny, nz);
    }
    return hipGetLastError();
}

hipError_t launch_layout(bool f64, int kind, const RepDev *rep_host, bool to_natural, void *nx,
                         void *ny, void *nz, hipStream_t st)
{
    return f64 ? layout_dispatch<double>(kind, *rep_host, to_natural, (double *)nx, (double *)ny,
                                         (double *)nz, st)
               : layout_dispatch<float>(kind, *rep_host, to_natural, (float *)nx, (float *)ny,
                                        (float *)nz, st);
}

hipError_t launch_finalize(const RepDev *reps_dev, int n_reps, int n_colours, uint32_t blocks,
                           const double *partials_dev, uint32_t n_items,
                           const uint32_t *tctr_dev, uint32_t t_add, double *records_dev,
                           double *stage_dev, double *host_last, hipStream_t st)
{
    if (blocks < 1u || blocks > FIN_BLOCKS) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_finalize, dim3((uint32_t)n_reps * blocks), dim3(256), 0, st, reps_dev,
                       n_colours, blocks, partials_dev, n_items, tctr_dev, t_add, stage_dev,
                       records_dev, host_last);
    return hipGetLastError();
}

__global__ void k_zero_u32(uint32_t *p, uint32_t n)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        p[i] = 0u;
}

hipError_t launch_zero_u32(uint32_t *p, uint32_t n, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero_u32, dim3((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024), dim3(256),
                       0, st, p, n);
    return hipGetLastError();
}

// Replica exchange (one workgroup; the pairs of a round are disjoint, so
// each thread owns the slots it writes).  Counter (k, 0, t, 2) keys the
// uniform of pair k after t sweeps.
__global__ void __launch_bounds__(256) k_exchange(ExchangeLaunch L)
{
    const uint32_t rnd = *L.round, t = *L.tctr_dev;
    __syncthreads();
    for (uint32_t k = 2u * threadIdx.x + (rnd & 1u); k + 1u < L.n; k += 2u * blockDim.x) {
        const uint32_t i = L.rep_at[k], j = L.rep_at[k + 1u];
        const double *ri = L.records + (size_t)i * NR, *rj = L.records + (size_t)j * NR;
        const double Ei = ri[R_EEX] + ri[R_EAN], Ej = rj[R_EEX] + rj[R_EAN];
        const double delta = (L.beta[k] - L.beta[k + 1u]) * (Ei - Ej);
        bool acc = delta >= 0.0;
        if (!acc) {
            const Words w = philox10(k, 0u, t, 2u, L.seed_lo, L.seed_hi);
            acc = uniform23<double>(w.w0) < exp(delta);
        }
        L.attempted[k] += 1u;
        if (acc) {
            L.accepted[k] += 1u;
            L.rep_at[k] = j;
            L.rep_at[k + 1u] = i;
            L.reps_dev[i].beta = L.beta[k + 1u];
            L.reps_dev[j].beta = L.beta[k];
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) *L.round = rnd + 1u;
}

hipError_t launch_exchange(const ExchangeLaunch &L, hipStream_t st)
{
    hipLaunchKernelGGL(k_exchange, dim3(1), dim3(256), 0, st, L);
    return hipGetLastError();
}

__global__ void k_xcd_probe(uint32_t *out, uint32_t n)
{
    if (threadIdx.x == 0 && blockIdx.x < n) out[blockIdx.x] = xcd_id();
}

hipError_t launch_xcd_probe(uint32_t *out, uint32_t n, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_xcd_probe, dim3(n), dim3(64), 0, st, out, n);
    return hipGetLastError();
}

hipError_t launch_advance(uint32_t *tctr_dev, uint32_t n, hipStream_t st)
{
    hipLaunchKernelGGL(k_advance, dim3(1), dim3(64), 0, st, tctr_dev, n);
    return hipGetLastError();
}

hipError_t launch_set_counter(uint32_t *tctr_dev, uint32_t v, hipStream_t st)
{
    hipLaunchKernelGGL(k_set_counter, dim3(1), dim3(64), 0, st, tctr_dev, v);
    return hipGetLastError();
}

hipError_t launch_fill_zero(double *p, uint64_t n, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    const unsigned g = grid_for((uint32_t)(n < 0xFFFFFFFFull ? n : 0xFFFFFFFFull));
    hipLaunchKernelGGL(k_fill_zero, dim3(g), dim3(256), 0, st, p, n);
    return hipGetLastError();
}

hipError_t launch_stream_probe(bool f64, void *x, void *y, void *z, uint64_t P, uint32_t grid,
                               hipStream_t st)
{
    if (grid == 0 || P < 2) return hipErrorInvalidValue;
    if (f64)
        hipLaunchKernelGGL(k_stream_probe<double>, dim3(grid), dim3(256), 0, st, (double *)x,
                           (double *)y, (double *)z, P);
    else
        hipLaunchKernelGGL(k_stream_probe<float>, dim3(grid), dim3(256), 0, st, (float *)x,
                           (float *)y, (float *)z, P);
    return hipGetLastError();
}

} // namespace mc
