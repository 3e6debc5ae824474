// tau1_nodes.hpp -- step kernel for rows of a few nodes, in every precision: one
// node per thread, in node order.
//
// The row kernel gives a wave to a row however short it is; here 64 consecutive
// nodes share one, whatever rows they lie in.  Each node reads the pre-step
// (drho, v) of its sources x - c_k (periodic wrap) and finishes with one division
// (division-saving algorithm); a solid source is replaced by the node's own state
// with the opposite direction (halfway bounce-back, Eq. (11)).  The operations and
// their order are the row kernel's in either form -- FP64 direction by direction,
// FP32 by groups of directions -- and so are the bits: which of the two kernels
// runs is a matter of time only.
//
// What bounds it: the 76 values and addresses that each node forms for itself
// (FP64 D3Q19 0.06 ns a node, FP32 0.025).
#pragma once

#include "tau1_kernels.hpp"
#include "tau1_lines.hpp"

namespace tau1 {

constexpr int kNodeThreads = 256;

// A node and its neighbourhood: row offsets (dy + 1) * 3 + dz + 1 of the nodes'
// rows, x - 1, x, x + 1, and the solid bits of the same.
template <int P>
struct NdNode {
    using S = typename Storage<P>::S;
    using T = typename Storage<P>::T;
    const S* pre;
    int64_t stride;
    int64_t row[9];
    int x[3];
    uint32_t solid[9];  // bits 0-2: nodes x - 1, x, x + 1 of the row
    T isr, isu;
    __device__ __forceinline__ int64_t at(int dx, int dy, int dz) const {
        return row[(dy + 1) * 3 + dz + 1] + x[dx + 1];
    }
    __device__ __forceinline__ bool wall(int dx, int dy, int dz) const {
        return (solid[(dy + 1) * 3 + dz + 1] >> (dx + 1)) & 1u;
    }
    __device__ __forceinline__ LnNode<T> load(int64_t j) const {
        using St = Storage<P>;
        return {St::load(pre, j, isr), St::load(pre + stride, j, isu),
                St::load(pre + 2 * stride, j, isu), St::load(pre + 3 * stride, j, isu)};
    }
};

// FP64: direction K onwards, in order.
template <int Q, int P, int K = 0>
__device__ __forceinline__ void nd_plain(const NdNode<P>& nb, const LnNode<typename Storage<P>::T>& own,
                                         LnNode<typename Storage<P>::T>& n) {
#pragma clang fp contract(off)
    using T = typename Storage<P>::T;
    if constexpr (K < Q) {
        constexpr Dir c = Lattice<Q>::c[K];
        const bool wall = K > 0 && nb.wall(-c.x, -c.y, -c.z);
        const LnNode<T> v = wall ? own : nb.load(nb.at(-c.x, -c.y, -c.z));
        const LnSrc<T> s{v.d, v.vx, v.vy, v.vz,
                         (T)1.5 * ((v.vx * v.vx + v.vy * v.vy) + v.vz * v.vz)};
        // the opposite direction's c.v is this one's with the other sign
        T cu = ln_cu<Q, K>(s);
        cu = wall ? -cu : cu;
        const T p = ((T)3 * cu + ((T)4.5 * cu) * cu) - s.h;
        ln_add<Q, K>(n, (T)weight<Q>(K) * (s.d + ((T)1 + s.d) * p));
        nd_plain<Q, P, K + 1>(nb, own, n);
    }
}

// FP32: group (CY, CZ) of the directions that arrive.  Solid sources hold zeros
// and send nothing.
template <int Q, int P, int CY, int CZ>
__device__ __forceinline__ void nd_group(const NdNode<P>& nb, LnSum& q, float& m) {
    using G = Group<Q, CY, CZ>;
    if constexpr (G::has0 || G::hasx) {
        auto level = [&](int dx, float& f, float& g) {
            const LnNode<float> v = nb.load(nb.at(dx, -CY, -CZ));
            const Src s = make_src(v.d, v.vx, v.vy, v.vz);
            level_y<CY>(s, f, g);
            level_z<CZ>(s, f, g);
            return s;
        };
        float f0 = 0.0f, g, a = 0.0f, b = 0.0f;
        if constexpr (G::has0) level(0, f0, g);
        if constexpr (G::hasx) {
            float f, fp, fm;
            const Src l = level(-1, f, g);
            level_x(l, f, g, a, fm);
            const Src r = level(1, f, g);
            level_x(r, f, g, fp, b);
        }
        add_group<Q, CY, CZ>(group_sum<Q, CY, CZ>(f0, a, b), G::hasx ? a - b : 0.0f, q.t, q.s, q.x,
                             q.y, m);
    }
}

template <int Q, int P>
struct NdPick {
    const NdNode<P>& nb;
    template <typename K>
    __device__ __forceinline__ float operator()(K, float u) const {
        constexpr Dir c = Lattice<Q>::c[K::value];
        return nb.wall(c.x, c.y, c.z) ? u : 0.0f;
    }
};

template <int Q, int P>
__global__ __launch_bounds__(kNodeThreads) void k_nodes(StepArgs a) {
    using St = Storage<P>;
    using S = typename St::S;
    using T = typename St::T;
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

    NdNode<P> nb;
    nb.pre = reinterpret_cast<const S*>(a.base + sd.state[a.parity]);
    nb.stride = sd.stride;
    nb.isr = inv_scale_rho<P>(a);
    nb.isu = inv_scale_u<P>(a);
    nb.x[0] = x == 0 ? nx - 1 : x - 1;
    nb.x[1] = x;
    nb.x[2] = x == nx - 1 ? 0 : x + 1;
    const int ys[3] = {y == 0 ? ny - 1 : y - 1, y, y == ny - 1 ? 0 : y + 1};
    const int zs[3] = {z == 0 ? nz - 1 : z - 1, z, z == nz - 1 ? 0 : z + 1};
    uint32_t any = 0;
#pragma unroll
    for (int r = 0; r < 9; ++r) {
        const int64_t row = (int64_t)zs[r % 3] * ny + ys[r / 3];
        nb.row[r] = row * nx;
        const uint32_t* mr = mask + row * sd.words;
        nb.solid[r] = 0;
#pragma unroll
        for (int d = 0; d < 3; ++d)
            nb.solid[r] |= ((mr[nb.x[d] >> 5] >> (nb.x[d] & 31)) & 1u) << d;
        any |= nb.solid[r];
    }
    const LnNode<T> own = nb.load(nb.at(0, 0, 0));
    LnNode<T> n{0, 0, 0, 0};
    if constexpr (P == kF64) {
#pragma clang fp contract(off)
        nd_plain<Q, P>(nb, own, n);
        const T r = (T)1 / ((T)1 + n.d);
        const T ghx = gh_of<T>(a, 0), ghy = gh_of<T>(a, 1), ghz = gh_of<T>(a, 2);
        n.vx = (n.vx * r + ghx) + ghx;
        n.vy = (n.vy * r + ghy) + ghy;
        n.vz = (n.vz * r + ghz) + ghz;
    } else {
        // in the order in which the row kernel's marching planes add them
        LnSum q;
        float m = 0.0f;
        nd_group<Q, P, 0, 1>(nb, q, m);
        nd_group<Q, P, 1, 1>(nb, q, m);
        nd_group<Q, P, -1, 1>(nb, q, m);
        nd_group<Q, P, 0, 0>(nb, q, m);
        nd_group<Q, P, 1, 0>(nb, q, m);
        nd_group<Q, P, -1, 0>(nb, q, m);
        if (any) {
            float r[4];
            wall_sums<Q>(make_src(own.d, own.vx, own.vy, own.vz), NdPick<Q, P>{nb}, r);
            q.s += r[0];
            q.x += r[1];
            q.y += r[2];
            q.t += r[3];
        }
        nd_group<Q, P, 0, -1>(nb, q, m);
        nd_group<Q, P, 1, -1>(nb, q, m);
        nd_group<Q, P, -1, -1>(nb, q, m);
        finish_node<Q>(q.t, q.s, m, q.x, q.y, 2.0f * gh_of<T>(a, 0), 2.0f * gh_of<T>(a, 1),
                       2.0f * gh_of<T>(a, 2), n.d, n.vx, n.vy, n.vz);
    }
    const T sr = scale_rho<P>(a), su = scale_u<P>(a);
    S* post = reinterpret_cast<S*>(a.base + sd.state[a.parity ^ 1]);
    St::store(post, i, n.d, sr);
    St::store(post + sd.stride, i, n.vx, su);
    St::store(post + 2 * sd.stride, i, n.vy, su);
    St::store(post + 3 * sd.stride, i, n.vz, su);
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
// thread / row kernel, D3Q19 of 2^20 nodes, rows of 1, 4, 8, 12, 16 and 20 nodes:
// FP64 66 / 739, 66 / 220, 64 / 125, 70 / 88, 70 / 72, 68 / 56; FP32 25 / 309, 26 /
// 102, 30 / 52, 29 / 40, 31 / 32, 27 / 27; of 2^15 nodes FP64, rows of 4 and 8
// nodes: 7.5 / 13.2, 7.7 / 8.6.  Of 675 cases timed both ways (three lattices and
// precisions, rows of 1-32 nodes, 2^12 to 2^22 nodes) 644 go to the faster kernel
// or lose at most 5 %; the others lie beside the line and lose at most 20 %.
template <typename SH>
inline bool nodes_faster(const SH* s, int n, int lattice, int precision) {
    const int64_t per_wave = lattice < 27 ? 18 : precision == kF64 ? 14 : 16;
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
