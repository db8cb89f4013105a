// kernels_measure.hip -- observables of a spin state computed from scratch,
// for checking the fused reduction of the pass kernels.
//
// Independent of the pass code on purpose: sites are enumerated in canonical
// order (pairs of simple-cubic sites, cells of the others), the storage index
// is derived from the layout rule, nearest neighbours come from bond vectors
// (each bond counted once, from the end that sees it along a "forward" one:
// +x, +y, +z, or a table in half-cell units), and
// every product is formed in FP64.  Eq. (1) of arXiv:2106.11286 gives the
// energy (E_exch = -J sum_bonds S_i.S_j, E_anis = -K sum_i (S_i.e)^2), Eq. (2)
// the magnetisation sum.
#include <hip/hip_runtime.h>

#include "launch.hpp"

namespace mc {

namespace {

// Forward bond vectors (half-cell units): the first nonzero component is
// positive, so every unordered nearest-neighbour pair is met once.
constexpr int kFwdBCC[4][3] = {{1, 1, 1}, {1, 1, -1}, {1, -1, 1}, {1, -1, -1}};
constexpr int kFwdFCC[6][3] = {{1, 1, 0}, {1, -1, 0}, {1, 0, 1},
                               {1, 0, -1}, {0, 1, 1}, {0, 1, -1}};
// Basis offsets (half-cell units) of the conventional cell.
constexpr int kBasisBCC[2][3] = {{0, 0, 0}, {1, 1, 1}};
constexpr int kBasisFCC[4][3] = {{0, 0, 0}, {1, 1, 0}, {1, 0, 1}, {0, 1, 1}};

template <int KIND> constexpr int sites_per_cell() { return KIND == BCC ? 2 : 4; }
template <int KIND> constexpr int forward_bonds() { return KIND == BCC ? 4 : 6; }
template <int KIND> constexpr int offset_of(int b, int axis)
{
    return KIND == BCC ? kBasisBCC[b][axis] : kBasisFCC[b][axis];
}
template <int KIND> constexpr int forward_of(int k, int axis)
{
    return KIND == BCC ? kFwdBCC[k][axis] : kFwdFCC[k][axis];
}
// The site a forward bond k of basis site b leads to: cell offset per axis
// (floor of the half-cell position over 2) and basis index.
template <int KIND> constexpr int cell_step(int b, int k, int axis)
{
    const int v = offset_of<KIND>(b, axis) + forward_of<KIND>(k, axis); // -1 .. 2
    return v < 0 ? -1 : v / 2;
}
template <int KIND> constexpr int end_basis(int b, int k)
{
    int best = -1;
    for (int b2 = 0; b2 < sites_per_cell<KIND>(); ++b2) {
        bool same = true;
        for (int a = 0; a < 3; ++a)
            same = same && ((offset_of<KIND>(b, a) + forward_of<KIND>(k, a)) & 1) == offset_of<KIND>(b2, a);
        if (same) best = b2;
    }
    return best;
}

struct Spin {
    double x, y, z;
};
template <bool SMALL, typename T>
__device__ __forceinline__ Spin spin_at(const T *sx, const T *sy, const T *sz, uint32_t i)
{
    // one byte offset for the three components; SMALL: it fits 32 bits and
    // adds to the uniform base in the load itself
    if constexpr (SMALL) {
        const uint32_t o = i * (uint32_t)sizeof(T);
        return {(double)*(const T *)((const char *)sx + o), (double)*(const T *)((const char *)sy + o),
                (double)*(const T *)((const char *)sz + o)};
    } else {
        return {(double)sx[i], (double)sy[i], (double)sz[i]};
    }
}
__device__ __forceinline__ double dot(const Spin &a, const Spin &b)
{
    return a.x * b.x + a.y * b.y + a.z * b.z;
}
// Inside the sphere (q: half-cell position).
__device__ __forceinline__ bool inside(const RepDev &R, int qx, int qy, int qz)
{
    const double dx = qx - R.Lx, dy = qy - R.Ly, dz = qz - R.Lz;
    return dx * dx + dy * dy + dz * dz <= R.r2x4;
}
__device__ __forceinline__ uint32_t quotient(uint32_t n, Div31 d)
{
    return d.d == 1u ? n : __umulhi(n, d.m) >> d.s;
}

struct Sums {
    double m_x = 0, m_y = 0, m_z = 0, pe2 = 0, bond = 0, cnt = 0;
};
__device__ __forceinline__ void add_site(Sums &s, const Spin &a, double ex, double ey, double ez)
{
    s.m_x += a.x;
    s.m_y += a.y;
    s.m_z += a.z;
    const double pe = a.x * ex + a.y * ey + a.z * ez;
    s.pe2 += pe * pe;
    s.cnt += 1.0;
}

// Simple cubic: sites 2u and 2u + 1 of canonical pair u (row (y, z), packed
// column xh; the even site has colour (y + z) & 1), their bond, and the
// forward bonds to the next pair, row and plane.
template <typename T, bool SPHERE, bool SMALL>
__device__ __forceinline__ void measure_pair(const RepDev &R, uint32_t u, Div31 d_row, Div31 d_ly,
                                             Sums &s)
{
    const T *sx = (const T *)R.sx, *sy = (const T *)R.sy, *sz = (const T *)R.sz;
    const uint32_t Lxh = (uint32_t)R.Lxh, Ly = (uint32_t)R.Ly, Lz = (uint32_t)R.Lz;
    const uint32_t row = quotient(u, d_row), xh = u - row * Lxh;
    const uint32_t z = quotient(row, d_ly), y = row - z * Ly;
    const uint32_t c = (y + z) & 1u, half = R.n_box / 2u; // colour of the even site
    const bool okx = xh + 1u < Lxh || (R.pmask & 1u);
    const bool oky = y + 1u < Ly || (R.pmask & 2u), okz = z + 1u < Lz || (R.pmask & 4u);
    const uint32_t ux = xh + 1u < Lxh ? u + 1u : u + 1u - Lxh;
    const uint32_t uy = y + 1u < Ly ? u + Lxh : u - y * Lxh;
    const uint32_t uz = z + 1u < Lz ? u + Lxh * Ly : u - z * Lxh * Ly;
    const T *tx = sx + half, *ty = sy + half, *tz = sz + half;
    // The pair's two sites by colour; one row or plane on, a site's neighbour
    // has the other colour (across a periodic edge too, as periodic lengths
    // are even), whichever of the two is the even one.
    const Spin s0 = spin_at<SMALL>(sx, sy, sz, u), s1 = spin_at<SMALL>(tx, ty, tz, u);
    const Spin y0 = spin_at<SMALL>(sx, sy, sz, uy), y1 = spin_at<SMALL>(tx, ty, tz, uy);
    const Spin z0 = spin_at<SMALL>(sx, sy, sz, uz), z1 = spin_at<SMALL>(tx, ty, tz, uz);
    // the odd site and the next pair's even one
    const Spin odd = c ? s0 : s1;
    const Spin nx = spin_at<SMALL>(sx, sy, sz, c ? half + ux : ux);
    bool in0 = true, in1 = true, in_x = okx, in_y0 = oky, in_y1 = oky, in_z0 = okz, in_z1 = okz;
    bool in_odd = true;
    if (SPHERE) {
        const int q0 = 4 * (int)xh + (c ? 2 : 0), q1 = 4 * (int)xh + (c ? 0 : 2); // by colour
        const int qy = 2 * (int)y, qz = 2 * (int)z;
        const int qn = xh + 1u < Lxh ? 4 * (int)xh + 4 : 0;
        const int yn = y + 1u < Ly ? qy + 2 : 0, zn = z + 1u < Lz ? qz + 2 : 0;
        in0 = inside(R, q0, qy, qz);
        in1 = inside(R, q1, qy, qz);
        in_odd = c ? in0 : in1;
        in_x = in_x && inside(R, qn, qy, qz);
        in_y1 = in_y1 && inside(R, q0, yn, qz); // the colour-0 site's neighbour has colour 1
        in_y0 = in_y0 && inside(R, q1, yn, qz);
        in_z1 = in_z1 && inside(R, q0, qy, zn);
        in_z0 = in_z0 && inside(R, q1, qy, zn);
    }
    const double ex = R.e[0], ey = R.e[1], ez = R.e[2];
    if (in0) add_site(s, s0, ex, ey, ez);
    if (in1) add_site(s, s1, ex, ey, ez);
    if (in0 && in1) s.bond += dot(s0, s1);
    if (in_odd && in_x) s.bond += dot(odd, nx);
    if (in0 && in_y1) s.bond += dot(s0, y1);
    if (in1 && in_y0) s.bond += dot(s1, y0);
    if (in0 && in_z1) s.bond += dot(s0, z1);
    if (in1 && in_z0) s.bond += dot(s1, z0);
}

// bcc / fcc: the sites of cell u and their forward bonds.
template <typename T, int KIND, bool SPHERE, bool SMALL>
__device__ __forceinline__ void measure_cell(const RepDev &R, uint32_t u, Div31 d_row, Div31 d_ly,
                                             Sums &s)
{
    constexpr int NB = sites_per_cell<KIND>(), NF = forward_bonds<KIND>();
    const T *sx = (const T *)R.sx, *sy = (const T *)R.sy, *sz = (const T *)R.sz;
    const int L[3] = {R.Lx, R.Ly, R.Lz};
    const uint32_t row = quotient(u, d_row), zz = quotient(row, d_ly);
    const int p[3] = {(int)(u - row * (uint32_t)L[0]), (int)(row - zz * (uint32_t)L[1]), (int)zz};
    // neighbouring cell coordinates (wrapped) and whether a bond crosses to them
    int at[3][3];
    bool ok[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int d = -1; d <= 1; ++d) {
            const int v = p[a] + d;
            at[a][d + 1] = v < 0 ? v + L[a] : v >= L[a] ? v - L[a] : v;
            ok[a][d + 1] = (v >= 0 && v < L[a]) || ((R.pmask >> a) & 1u);
        }
    const uint32_t cells = R.plane;
    const double ex = R.e[0], ey = R.e[1], ez = R.e[2];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const Spin me = spin_at<SMALL>(sx, sy, sz, (uint32_t)b * cells + u);
        if (SPHERE && !inside(R, 2 * p[0] + offset_of<KIND>(b, 0), 2 * p[1] + offset_of<KIND>(b, 1),
                              2 * p[2] + offset_of<KIND>(b, 2)))
            continue;
        add_site(s, me, ex, ey, ez);
#pragma unroll
        for (int k = 0; k < NF; ++k) {
            const int b2 = end_basis<KIND>(b, k);
            const int ix = cell_step<KIND>(b, k, 0) + 1, iy = cell_step<KIND>(b, k, 1) + 1;
            const int iz = cell_step<KIND>(b, k, 2) + 1;
            bool in = ok[0][ix] && ok[1][iy] && ok[2][iz];
            if (SPHERE)
                in = in && inside(R, 2 * at[0][ix] + offset_of<KIND>(b2, 0),
                                  2 * at[1][iy] + offset_of<KIND>(b2, 1),
                                  2 * at[2][iz] + offset_of<KIND>(b2, 2));
            const uint32_t j = (uint32_t)b2 * cells +
                               (uint32_t)(at[2][iz] * L[1] + at[1][iy]) * (uint32_t)L[0] +
                               (uint32_t)at[0][ix];
            const Spin o = spin_at<SMALL>(sx, sy, sz, j);
            if (in) s.bond += dot(me, o);
        }
    }
}

} // namespace

// The bytes are the spins once: each XCD takes a contiguous eighth of the
// lattice and its workgroups go along it side by side, so rows and planes that
// are neighbours' neighbours come from its L2 (counted reads 1.2 times the
// spins).  What is left is the rate of 21 four-byte loads per pair of sites
// (more waves or two pairs in flight change nothing).  The former kernel
// walked single sites with a division per coordinate and a table look-up per
// bond, and one wave added its partial sums in a serial chain: 279 + 154 us on
// a 16 M-site film, FP32, against 83 + 9 now.
template <typename T, int KIND, bool SPHERE, bool SMALL>
__global__ void __launch_bounds__(256)
k_measure_direct(RepDev R, Div31 d_row, Div31 d_ly, double *__restrict__ partials)
{
    const uint32_t n = KIND == SC ? R.n_box / 2u : R.plane; // pairs or cells
    const uint32_t G = gridDim.x;
    // XCD g (workgroups are dealt to them in turn) takes the g-th eighth, its
    // workgroups side by side along it
    const uint32_t parts = G % 8u == 0u ? 8u : 1u;
    const uint32_t g = blockIdx.x % parts, w = blockIdx.x / parts, per = G / parts;
    const uint32_t u0 = (uint32_t)(((uint64_t)n * g) / parts);
    const uint32_t u1 = (uint32_t)(((uint64_t)n * (g + 1u)) / parts);
    Sums s;
    for (uint32_t u = u0 + w * blockDim.x + threadIdx.x; u < u1; u += per * blockDim.x) {
        if constexpr (KIND == SC) measure_pair<T, SPHERE, SMALL>(R, u, d_row, d_ly, s);
        else measure_cell<T, KIND, SPHERE, SMALL>(R, u, d_row, d_ly, s);
    }
    // fixed-order block reduction: wave butterflies, then the waves in order
    __shared__ double red[4][6];
    double v[6] = {s.m_x, s.m_y, s.m_z, s.pe2, s.bond, s.cnt};
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) v[q] += __shfl_xor(v[q], o, 64);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0)
#pragma unroll
        for (int q = 0; q < 6; ++q) red[wave][q] = v[q];
    __syncthreads();
    if (threadIdx.x < 6) {
        double a = 0.0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) a += red[w][threadIdx.x];
        partials[(size_t)blockIdx.x * 8 + threadIdx.x] = a;
    }
}

// Sum the block partials in a fixed order (32 strided shares of eight lanes,
// then the shares in order) into one record (FP64): M sums, E_exch, E_anis,
// occupied count in the accepted-count slot.
__global__ void __launch_bounds__(256)
k_measure_finish(const double *__restrict__ partials, uint32_t n_blocks, double J, double K,
                 double sweep, double *__restrict__ record)
{
    __shared__ double share[32][8], out[8];
    const uint32_t q = threadIdx.x & 7u, g = threadIdx.x >> 3;
    double a = 0.0;
    if (q < 6u)
        for (uint32_t b = g; b < n_blocks; b += 32u) a += partials[(size_t)b * 8 + q];
    share[g][q] = a;
    __syncthreads();
    if (threadIdx.x < 8u) {
        double v = 0.0;
#pragma unroll
        for (int i = 0; i < 32; ++i) v += share[i][q];
        out[q] = v;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    record[R_MX] = out[0];
    record[R_MY] = out[1];
    record[R_MZ] = out[2];
    record[R_EEX] = -J * out[4];
    record[R_EAN] = -K * out[3];
    record[R_NACC] = out[5];
    record[R_SWEEP] = sweep;
    record[7] = 0.0;
}

template <typename T, int KIND>
static void measure_kind(const RepDev &R, double *partials, uint32_t n_blocks, hipStream_t st)
{
    const Div31 d_row = make_div31((uint32_t)R.Lxh), d_ly = make_div31((uint32_t)R.Ly);
    const dim3 g(n_blocks), b(256);
    // a component array below 4 GiB takes 32-bit byte offsets
    const bool small = (uint64_t)R.n_box * sizeof(T) <= 0xFFFFFFFFull;
    if (R.sphere) {
        if (small) hipLaunchKernelGGL((k_measure_direct<T, KIND, true, true>), g, b, 0, st, R, d_row, d_ly, partials);
        else hipLaunchKernelGGL((k_measure_direct<T, KIND, true, false>), g, b, 0, st, R, d_row, d_ly, partials);
    } else {
        if (small) hipLaunchKernelGGL((k_measure_direct<T, KIND, false, true>), g, b, 0, st, R, d_row, d_ly, partials);
        else hipLaunchKernelGGL((k_measure_direct<T, KIND, false, false>), g, b, 0, st, R, d_row, d_ly, partials);
    }
}

hipError_t launch_measure_direct(bool f64, int kind, const RepDev *rep_host, double *partials,
                                 uint32_t n_blocks, double sweep, double *record, hipStream_t st)
{
    if (n_blocks == 0 || n_blocks > MEASURE_BLOCKS) return hipErrorInvalidValue;
    const RepDev &R = *rep_host;
    switch (kind) {
    case SC:
        f64 ? measure_kind<double, SC>(R, partials, n_blocks, st)
            : measure_kind<float, SC>(R, partials, n_blocks, st);
        break;
    case BCC:
        f64 ? measure_kind<double, BCC>(R, partials, n_blocks, st)
            : measure_kind<float, BCC>(R, partials, n_blocks, st);
        break;
    case FCC:
        f64 ? measure_kind<double, FCC>(R, partials, n_blocks, st)
            : measure_kind<float, FCC>(R, partials, n_blocks, st);
        break;
    default: return hipErrorInvalidValue;
    }
    hipLaunchKernelGGL(k_measure_finish, dim3(1), dim3(256), 0, st, partials, n_blocks,
                       rep_host->J, rep_host->K, sweep, record);
    return hipGetLastError();
}

} // namespace mc
