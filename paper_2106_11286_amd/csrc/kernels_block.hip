// kernels_block.hip -- the paper's block scheme in synchronous form, for
// comparison with the colour sweep (simple cubic).  A step is two launches:
// every block of n consecutive canonical sites picks one site and computes its
// attempt from the state before the step, staging the accepted spin; then the
// staged moves are written and the step's counts added up.
//
// Bound: the gather of seven scattered spins per attempt, about the whole
// lattice through the L2 per step.  Each XCD takes a contiguous eighth of the
// blocks, so its part of the lattice stays in its L2; the counts go to one
// slot per workgroup and are summed by one workgroup of the second launch
// (three same-address atomics per wave, 12.6 ns each in turn, made a step of
// 128^3, n = 8, 163 us; it takes 22 now); the divisions by the
// lattice edges and by n are multiplications by host-made constants.
#include "device_common.hpp"

namespace mc {

__device__ __forceinline__ uint32_t block_pick(uint32_t k, uint32_t n, uint32_t n_box,
                                               uint32_t rid, uint32_t step, uint32_t k0,
                                               uint32_t k1, Words &w)
{
    const uint32_t m = min(n, n_box - k * n);
    w = philox10(k, rid, step, 3u, k0, k1);
    return k * n + (uint32_t)(((uint64_t)w.w3 * m) >> 32);
}

// Colour-packed storage index of canonical sc site (x, y, z).
__device__ __forceinline__ uint32_t sc_store(int x, int y, int z, int Lx, int Ly, uint32_t plane)
{
    const uint32_t c = (uint32_t)(x + y + z) & 1u;
    return c * plane + (((uint32_t)(z * Ly + y) * (uint32_t)Lx + (uint32_t)x) >> 1);
}

template <typename T>
__global__ void __launch_bounds__(256) k_block_propose(BlockLaunch B)
{
    const RepDev &R = B.rep;
    __shared__ uint32_t s_cnt[4][3];
    // workgroups are dealt to the XCDs in turn: XCD g takes the g-th eighth of
    // the chunks (a multiple of 8 workgroups)
    const uint32_t per = gridDim.x >> 3;
    const uint32_t chunk = (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
    const uint32_t k_begin = chunk * B.chunk;
    const uint32_t k_end = min(B.n_blocks, k_begin + B.chunk);
    uint32_t att = 0, acc = 0, conf = 0;
    for (uint32_t k = k_begin + threadIdx.x; k < k_end; k += blockDim.x) {
        const int Lx = R.Lx, Ly = R.Ly, Lz = R.Lz;
        Words w;
        const uint32_t s = block_pick(k, B.n, R.n_box, R.rid, B.step, B.seed_lo, B.seed_hi, w);
        const uint32_t row = div31(s, B.d_lx), zz = div31(row, B.d_ly);
        const int x = (int)(s - row * (uint32_t)Lx), y = (int)(row - zz * (uint32_t)Ly);
        const int z = (int)zz;
        uint32_t out = 0xFFFFFFFFu;
        if (occupied(R, x, y, z, 0, 0, 0)) {
            ++att;
            bool hit = false;
            const T *gx = (const T *)R.sx, *gy = (const T *)R.sy, *gz = (const T *)R.sz;
            const bool px = R.pmask & 1u, py = R.pmask & 2u, pz = R.pmask & 4u;
            // neighbours -x, +x, -y, +y, -z, +z (missing across open faces)
            int q[6][3] = {{x - 1, y, z}, {x + 1, y, z}, {x, y - 1, z},
                           {x, y + 1, z}, {x, y, z - 1}, {x, y, z + 1}};
            T hx = 0, hy = 0, hz = 0;
#pragma unroll
            for (int j = 0; j < 6; ++j) {
                int &a = q[j][0], &b = q[j][1], &c = q[j][2];
                bool ok = true;
                if (a < 0) { a += Lx; ok &= px; }
                if (a >= Lx) { a -= Lx; ok &= px; }
                if (b < 0) { b += Ly; ok &= py; }
                if (b >= Ly) { b -= Ly; ok &= py; }
                if (c < 0) { c += Lz; ok &= pz; }
                if (c >= Lz) { c -= Lz; ok &= pz; }
                if (!ok || !occupied(R, a, b, c, 0, 0, 0)) {
                    a = -1;
                    continue;
                }
                const uint32_t i = sc_store(a, b, c, Lx, Ly, R.plane);
                hx += gx[i];
                hy += gy[i];
                hz += gz[i];
                if (B.count_conflicts && !hit) {
                    // a neighbour in this block is not its choice
                    const uint32_t qs = ((uint32_t)(c * Ly + b) * (uint32_t)Lx) + (uint32_t)a;
                    const uint32_t kq = div31(qs, B.d_n);
                    Words w2;
                    if (kq != k && block_pick(kq, B.n, R.n_box, R.rid, B.step, B.seed_lo,
                                              B.seed_hi, w2) == qs)
                        hit = true;
                }
            }
            conf += hit ? 1u : 0u;
            const T J = (T)R.J;
            hx *= J;
            hy *= J;
            hz *= J;
            const uint32_t i = sc_store(x, y, z, Lx, Ly, R.plane);
            T sx = gx[i], sy = gy[i], sz = gz[i];
            T dH;
            if (metropolis_words<T>(w, sx, sy, sz, hx, hy, hz, (T)R.K, (T)R.e[0], (T)R.e[1],
                                    (T)R.e[2], (T)R.beta, R.greedy != 0, dH)) {
                ++acc;
                out = i;
                T *st = (T *)B.stage_spin + 3 * (size_t)k;
                st[0] = sx;
                st[1] = sy;
                st[2] = sz;
            }
        }
        B.stage_idx[k] = out;
    }
    // counts: wave sums, then the workgroup's slot
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        att += __shfl_xor(att, o, 64);
        acc += __shfl_xor(acc, o, 64);
        conf += __shfl_xor(conf, o, 64);
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        s_cnt[wave][0] = att;
        s_cnt[wave][1] = acc;
        s_cnt[wave][2] = conf;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        uint32_t v = 0;
        for (int i = 0; i < 4; ++i) v += s_cnt[i][threadIdx.x];
        B.slots[blockIdx.x * 4u + threadIdx.x] = v;
    }
}

template <typename T>
__global__ void __launch_bounds__(256) k_block_apply(BlockLaunch B)
{
    if (blockIdx.x + 1u == gridDim.x) {
        // the last workgroup adds the step's counts to the totals: every
        // thread takes its slots' three counts, all loads in flight at once
        __shared__ uint32_t s_sum[4][3];
        constexpr uint32_t PER = BLOCK_SLOTS / 256u;
        uint4 c[PER];
#pragma unroll
        for (uint32_t u = 0; u < PER; ++u) {
            const uint32_t j = threadIdx.x + u * 256u;
            c[u] = j < B.n_slots ? ((const uint4 *)B.slots)[j] : make_uint4(0, 0, 0, 0);
        }
        uint32_t v[3] = {0, 0, 0};
#pragma unroll
        for (uint32_t u = 0; u < PER; ++u) {
            v[0] += c[u].x;
            v[1] += c[u].y;
            v[2] += c[u].z;
        }
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) v[q] += __shfl_xor(v[q], o, 64);
        if ((threadIdx.x & 63u) == 0)
            for (int q = 0; q < 3; ++q) s_sum[threadIdx.x >> 6][q] = v[q];
        __syncthreads();
        if (threadIdx.x < 3u) {
            unsigned long long n = 0;
            for (int w = 0; w < 4; ++w) n += s_sum[w][threadIdx.x];
            B.counts[threadIdx.x] += n;
        }
        return;
    }
    const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= B.n_blocks) return;
    const uint32_t i = B.stage_idx[k];
    if (i == 0xFFFFFFFFu) return;
    const T *st = (const T *)B.stage_spin + 3 * (size_t)k;
    ((T *)B.rep.sx)[i] = st[0];
    ((T *)B.rep.sy)[i] = st[1];
    ((T *)B.rep.sz)[i] = st[2];
}

hipError_t launch_block_step(bool f64, const BlockLaunch &L, hipStream_t st)
{
    if (L.n_blocks == 0) return hipSuccess;
    BlockLaunch B = L;
    // a multiple of 8 workgroups, at most one slot each
    uint32_t grid = (B.n_blocks + 255u) / 256u;
    grid = (grid + 7u) / 8u * 8u;
    if (grid > BLOCK_SLOTS) grid = BLOCK_SLOTS;
    B.n_slots = grid;
    B.chunk = (uint32_t)(((uint64_t)B.n_blocks + grid - 1u) / grid);
    B.d_n = make_div31(B.n);
    B.d_lx = make_div31((uint32_t)B.rep.Lx);
    B.d_ly = make_div31((uint32_t)B.rep.Ly);
    const dim3 g(grid), ga((B.n_blocks + 255u) / 256u + 1u), b(256);
    if (f64) {
        hipLaunchKernelGGL(k_block_propose<double>, g, b, 0, st, B);
        hipLaunchKernelGGL(k_block_apply<double>, ga, b, 0, st, B);
    } else {
        hipLaunchKernelGGL(k_block_propose<float>, g, b, 0, st, B);
        hipLaunchKernelGGL(k_block_apply<float>, ga, b, 0, st, B);
    }
    return hipGetLastError();
}

} // namespace mc
