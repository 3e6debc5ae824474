// tau1_nodes.hpp -- step kernel for rows of a few nodes, in every precision: one
// node per thread, in node order.
//
// The row kernel gives a wave to a row however short it is; here 64 consecutive
// nodes share one, whatever rows they lie in.  The node reads the pre-step
// (drho, v) of each source x - c_k (periodic wrap, then the solid test), forms
// the equilibrium of Eq. (3) minus its weight and accumulates density and
// momentum in direction order; a solid source is replaced by the node's own
// state with the opposite direction (halfway bounce-back, Eq. (11)).  One
// reciprocal per node (division-saving algorithm).  Every operation is rounded
// by itself, as in the row kernel: the bits are the same, so which of the two
// runs is a matter of time only.
//
// What bounds it: the 76 values and addresses that each node forms for itself
// (FP64 D3Q19 0.073 ns a node, FP32 0.042).
#pragma once

#include "tau1_kernels.hpp"
#include "tau1_lines.hpp"

namespace tau1 {

constexpr int kNodeThreads = 256;

template <int Q, int P>
__global__ __launch_bounds__(kNodeThreads) void k_nodes(StepArgs a) {
#pragma clang fp contract(off)
    using St = Storage<P>;
    using S = typename St::S;
    using T = typename St::T;
    using L = Lattice<Q>;
    const int s = sample_of_block(a.samples, a.nsamples, blockIdx.x);
    const SampleDev& sd = a.samples[s];
    const int64_t i = (int64_t)(blockIdx.x - sd.block0) * kNodeThreads + threadIdx.x;
    if (i >= sd.n) return;
    const int nx = sd.nx, ny = sd.ny, nz = sd.nz;
    const int x = (int)(i % nx);
    const int y = (int)((i / nx) % ny);
    const int z = (int)(i / ((int64_t)nx * ny));
    const uint32_t* mask = reinterpret_cast<const uint32_t*>(a.base + sd.mask);
    if (solid_bit(mask, sd.words, ny, x, y, z)) return;

    const S* pre = reinterpret_cast<const S*>(a.base + sd.state[a.parity]);
    S* post = reinterpret_cast<S*>(a.base + sd.state[a.parity ^ 1]);
    const int64_t st = sd.stride;
    const T isr = inv_scale_rho<P>(a), isu = inv_scale_u<P>(a);
    const T d0 = St::load(pre, i, isr);
    const T v0x = St::load(pre + st, i, isu);
    const T v0y = St::load(pre + 2 * st, i, isu);
    const T v0z = St::load(pre + 3 * st, i, isu);

    T d = 0, jx = 0, jy = 0, jz = 0;
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        const int cx = L::c[k].x, cy = L::c[k].y, cz = L::c[k].z;
        int sx = x - cx, sy = y - cy, sz = z - cz;
        sx += sx < 0 ? nx : 0; sx -= sx >= nx ? nx : 0;
        sy += sy < 0 ? ny : 0; sy -= sy >= ny ? ny : 0;
        sz += sz < 0 ? nz : 0; sz -= sz >= nz ? nz : 0;
        T ds, vx, vy, vz, ex, ey, ez;
        if (!solid_bit(mask, sd.words, ny, sx, sy, sz)) {
            const int64_t j = sx + (int64_t)nx * (sy + (int64_t)ny * sz);
            ds = St::load(pre, j, isr);
            vx = St::load(pre + st, j, isu);
            vy = St::load(pre + 2 * st, j, isu);
            vz = St::load(pre + 3 * st, j, isu);
            ex = (T)cx; ey = (T)cy; ez = (T)cz;
        } else {
            ds = d0; vx = v0x; vy = v0y; vz = v0z;
            ex = (T)-cx; ey = (T)-cy; ez = (T)-cz;
        }
        const T rho = (T)1 + ds;
        const T cu = (ex * vx + ey * vy) + ez * vz;
        const T vv = (vx * vx + vy * vy) + vz * vz;
        const T p = ((T)3 * cu + ((T)4.5 * cu) * cu) - (T)1.5 * vv;
        const T f = (T)weight<Q>(k) * (ds + rho * p);
        d += f;
        jx += (T)cx * f;
        jy += (T)cy * f;
        jz += (T)cz * f;
    }
    const T r = (T)1 / ((T)1 + d);
    const T ghx = gh_of<T>(a, 0), ghy = gh_of<T>(a, 1), ghz = gh_of<T>(a, 2);
    const T ux = jx * r + ghx, uy = jy * r + ghy, uz = jz * r + ghz;
    const T sr = scale_rho<P>(a), su = scale_u<P>(a);
    St::store(post, i, d, sr);
    St::store(post + st, i, ux + ghx, su);
    St::store(post + 2 * st, i, uy + ghy, su);
    St::store(post + 3 * st, i, uz + ghz, su);
}

#define TAU1_ND_TABLE_DECL(PP) void* nd_kernel_##PP(int q);
TAU1_ND_TABLE_DECL(0) TAU1_ND_TABLE_DECL(1) TAU1_ND_TABLE_DECL(2) TAU1_ND_TABLE_DECL(3)
#undef TAU1_ND_TABLE_DECL

inline void* pick_nodes(int q, int p) {
    switch (p) {
        case kF64: return nd_kernel_0(q);
        case kF32: return nd_kernel_1(q);
        case kF16: return nd_kernel_2(q);
        case kBF16: return nd_kernel_3(q);
    }
    return nullptr;
}

// Whether one node per thread is the faster for a context's samples: a wave's
// plane in the row kernel takes the time of `per_wave` nodes here, and a launch
// here ends later by that of `more` nodes.  Measured us a step, one node per
// thread / row kernel, D3Q19 of 2^20 nodes: FP64 rows of 1 node 76 / 738, 4 nodes
// 76 / 220, 12 nodes 79 / 88, 16 nodes 79 / 72, FP32 40 / 424, 40 / 132, 45 / 52,
// 46 / 45; of 2^15 nodes: FP64 rows of 4 nodes 8.7 / 13.3, 8 nodes 8.8 / 8.4.  Of 675 cases timed both ways (three lattices
// and precisions, rows of 1-32 nodes, 2^12 to 2^22 nodes) 653 go to the faster
// kernel or lose at most 5 %, and 5 lose more by the row kernel (at most 10.6
// against 13.2, half storage, rows of 16 nodes).
template <typename SH>
inline bool nodes_faster(const SH* s, int n, int lattice, int precision) {
    const int64_t per_wave =
        precision == kF64 ? (lattice < 27 ? 16 : 12) : lattice < 27 ? 18 : 16;
    constexpr int64_t more = 32768;
    int64_t nodes = 0, waves = 0;
    for (int i = 0; i < n; ++i) {
        const SampleDev& sd = s[i].dev;
        nodes += sd.n;
        waves += (int64_t)sd.ln_windows * sd.ny * sd.nz;
    }
    return nodes + more < per_wave * waves;
}

// First workgroup of each sample (block0); returns the number of workgroups.
template <typename SH>
inline int64_t nodes_tiling(SH* s, int n) {
    int64_t blocks = 0;
    for (int i = 0; i < n; ++i) {
        s[i].dev.block0 = blocks;
        blocks += (s[i].dev.n + kNodeThreads - 1) / kNodeThreads;
    }
    return blocks;
}

}  // namespace tau1
