// tau1_kernels.hpp -- D2Q9 step kernel and the service kernels
// (geometry encode, state upload/readback, FP64 reductions, copy probe).
#pragma once

#include <algorithm>

#include "tau1_args.hpp"

namespace tau1 {

// Sample owning a block of a per-node launch (samples sorted by block0).
__device__ __forceinline__ int sample_of_block(const SampleDev* s, int n, int64_t b) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s[mid].block0 <= b) lo = mid; else hi = mid - 1;
    }
    return lo;
}


// ---------------------------------------------------------------------------
// D2Q9 steps of the validation workloads (nz = 1): up to kD2MaxSteps time steps
// per launch.  A workgroup holds a square of kD2Side x kD2Side nodes, one per
// thread, advances it T steps between barriers and stores the inner kD2Side -
// 2 T: a node T away from the square's edge does not see what lies beyond.
// The squares overlap, so a launch needs nothing from another's; the nodes
// computed twice come out the same.
//
// Per step each node forms what it sends in its eight directions (the
// equilibria of Eq. (3) minus their weights), passes them through LDS and adds
// what it receives, in direction order.  With node types: a wall source (type
// 1) returns the node's own value in the opposite direction (halfway
// bounce-back, Eq. (11)), read from the node's own place; a moving wall (type
// 2) adds the wall's momentum to it,
//   f_k(x) = f_opp(k)(x) + 6 w_k rho(x) (c_k . u_wall).
// With a.xbc the fluid nodes of columns x = 0 and nx - 1 are constant-pressure
// nodes (Zou-He): the populations that would come from outside are unknown,
// the known ones fix rho u_x through
//   inlet:  rho_in u_x  = drho_in  - [f0 + f3 + f4 + 2 (f2 + f6 + f8)]
//   outlet: rho_out u_x = [f0 + f3 + f4 + 2 (f1 + f5 + f7)] - drho_out
// (values minus their weights), and the node's new state is (rho_b, u_x, 0).
// FP64 reproduces the oracle's roundings (contraction off).
//
// What bounds it: with one step per launch and one thread per node that read its
// nine sources from memory, a launch and its chain of dependent reads (FP64,
// 6.6 us a step on 160^2 nodes, 8.4 us on 1000 x 100); now vector issue of the
// equilibria and the division, about 1.1 us a step and workgroup (1.5 and 2.3
// us a step).  More steps per launch save launches and repeat more nodes, so
// their number is chosen per lattice (d2q9_steps).
// ---------------------------------------------------------------------------
constexpr int kD2Side = 32;
constexpr int kD2Threads = kD2Side * kD2Side;
constexpr int kD2MaxSteps = 10;

// Square of a core of `core` nodes a side.
constexpr int d2q9_core(int steps) { return kD2Side - 2 * steps; }

template <int P>
__global__ __launch_bounds__(kD2Threads) void k_d2q9(StepArgs a) {
#pragma clang fp contract(off)
    using St = Storage<P>;
    using S = typename St::S;
    using T = typename St::T;
    using L = Lattice<9>;
    __shared__ T sent[8][kD2Threads];
    const int s = sample_of_block(a.samples, a.nsamples, blockIdx.x);
    const SampleDev& sd = a.samples[s];
    const int nx = sd.nx, ny = sd.ny;
    const int core = d2q9_core(a.d2_span);
    const int b = (int)(blockIdx.x - sd.block0);
    const int lx = threadIdx.x % kD2Side, ly = threadIdx.x / kD2Side;
    const int gx = (b % sd.ln_windows) * core - a.d2_span + lx;
    const int gy = (b / sd.ln_windows) * core - a.d2_span + ly;
    auto wrap = [](int g, int n) {  // few turns at most: g is within a square of [0, n)
        while (g < 0) g += n;
        while (g >= n) g -= n;
        return g;
    };
    const int x = wrap(gx, nx), y = wrap(gy, ny);
    // beyond a pressure column there is nothing (never used by the nodes inside)
    const bool outside = a.xbc && (gx < 0 || gx >= nx);
    const int64_t i = x + (int64_t)nx * y;
    const uint8_t* type = a.base + sd.types;
    const uint8_t own = outside ? 0 : type[i];
    const bool fluid = !outside && own == 0;
    __shared__ uint8_t kind[kD2Threads];
    kind[threadIdx.x] = own;
    __syncthreads();

    const S* pre = reinterpret_cast<const S*>(a.base + sd.state[a.parity]);
    S* post = reinterpret_cast<S*>(a.base + sd.state[a.parity ^ 1]);
    const int64_t st = sd.stride;
    T d = St::load(pre, i, (T)1);
    T vx = St::load(pre + st, i, (T)1);
    T vy = St::load(pre + 2 * st, i, (T)1);
    const T uwx = (T)a.uw[0], uwy = (T)a.uw[1];
    const bool pressure = a.xbc && (x == 0 || x == nx - 1);

    // where each direction's value comes from: the node x - c_k's slot of
    // direction k, or at a wall the node's own slot of the opposite direction;
    // nodes at the square's edge read their own (their results are not used)
    int from[9];
    uint32_t moving = 0;
#pragma unroll
    for (int k = 1; k < 9; ++k) {
        const int cx = L::c[k].x, cy = L::c[k].y;
        const int opp = (k & 1) ? k + 1 : k - 1;
        const int sx = lx - cx, sy = ly - cy;
        const bool in = sx >= 0 && sx < kD2Side && sy >= 0 && sy < kD2Side;
        const int src = in ? sy * kD2Side + sx : (int)threadIdx.x;
        const int tj = kind[src];
        from[k] = tj != 0 ? (opp - 1) * kD2Threads + (int)threadIdx.x : (k - 1) * kD2Threads + src;
        moving |= (uint32_t)(tj == 2) << k;
    }
    const T ghx = gh_of<T>(a, 0), ghy = gh_of<T>(a, 1);
    T* slots = &sent[0][0];
    for (int step = 0; step < a.d2_steps; ++step) {
        // rows this far from the square's edge still matter (a wave holds two)
        const bool rows = ly + 1 >= step && ly - 1 <= kD2Side - 1 - step;
        T f[9];
        if (rows) {
            const T rho = (T)1 + d;
            const T h = (T)1.5 * (vx * vx + vy * vy);
            f[0] = (T)weight<9>(0) * (d + rho * -h);
            // opposite directions share 3 cu and (4.5 cu) cu (exact: cu only
            // changes its sign)
#pragma unroll
            for (int k = 1; k < 9; k += 2) {
                const int cx = L::c[k].x, cy = L::c[k].y;
                const T cu = cx == 0 ? (cy > 0 ? vy : -vy)
                             : cy == 0 ? (cx > 0 ? vx : -vx)
                                       : (cx > 0 ? vx : -vx) + (cy > 0 ? vy : -vy);
                const T t1 = (T)3 * cu, t2 = ((T)4.5 * cu) * cu;
                sent[k - 1][threadIdx.x] = (T)weight<9>(k) * (d + rho * ((t1 + t2) - h));
                sent[k][threadIdx.x] = (T)weight<9>(k) * (d + rho * ((t2 - t1) - h));
            }
        }
        __syncthreads();
        if (rows) {
#pragma unroll
            for (int k = 1; k < 9; ++k) f[k] = slots[from[k]];
        }
        __syncthreads();
        if (rows && fluid) {
            if (moving) {
#pragma unroll
                for (int k = 1; k < 9; ++k) {
                    const T cw = (T)L::c[k].x * uwx + (T)L::c[k].y * uwy;
                    const T fw = f[k] + (T)6 * (T)weight<9>(k) * ((T)1 + d) * cw;
                    f[k] = ((moving >> k) & 1u) ? fw : f[k];
                }
            }
            T ux, uy;
            if (pressure) {
                const bool inlet = x == 0;
                const T db = (T)(inlet ? a.din : a.dout);
                if (inlet) {
                    const T sk = (f[0] + f[3] + f[4]) + (T)2 * ((f[2] + f[6]) + f[8]);
                    ux = (db - sk) / ((T)1 + db) + ghx;
                } else {
                    const T sk = (f[0] + f[3] + f[4]) + (T)2 * ((f[1] + f[5]) + f[7]);
                    ux = (sk - db) / ((T)1 + db) + ghx;
                }
                d = db;
                uy = ghy;
            } else {
                T jx = 0, jy = 0;
                d = 0;
#pragma unroll
                for (int k = 0; k < 9; ++k) {
                    d += f[k];
                    if (L::c[k].x != 0) jx += (T)L::c[k].x * f[k];
                    if (L::c[k].y != 0) jy += (T)L::c[k].y * f[k];
                }
                const T r = (T)1 / ((T)1 + d);
                ux = jx * r + ghx;
                uy = jy * r + ghy;
            }
            vx = ux + ghx;
            vy = uy + ghy;
        }
    }
    // the core's nodes inside the lattice (the z component stays zero)
    const bool mine = lx >= a.d2_span && lx < kD2Side - a.d2_span && ly >= a.d2_span &&
                      ly < kD2Side - a.d2_span && gx < nx && gy < ny;
    if (mine && fluid) {
        St::store(post, i, d, (T)1);
        St::store(post + st, i, vx, (T)1);
        St::store(post + 2 * st, i, vy, (T)1);
    }
}

// Squares of the samples at `steps` steps per launch: sets each sample's squares
// per row and first workgroup; returns the number of workgroups.
template <typename SH>
inline int64_t d2q9_blocks(SH* s, int n, int steps) {
    const int core = d2q9_core(steps);
    int64_t blocks = 0;
    for (int i = 0; i < n; ++i) {
        SampleDev& sd = s[i].dev;
        sd.ln_windows = (sd.nx + core - 1) / core;
        sd.block0 = blocks;
        blocks += (int64_t)sd.ln_windows * ((sd.ny + core - 1) / core);
    }
    return blocks;
}

// Steps per launch for a context's samples: the number with the shortest
// modelled time a step.  A launch takes 3.4 us alone and 5 us with a workgroup
// on every CU, and 1.1-1.4 us a step for each round of them (fitted in FP64 to
// 1-10 steps per launch; measured us a step at the choice and at one step per
// launch: 40^2 nodes 1.4 / 4.6, 160^2 1.7 / 4.9, 400^2 3.1 / 6.4, 1000 x 100
// 2.1 / 5.8, 1600 x 200 5.1 / 10.5).  FP32 steps are shorter and larger lattices
// run two workgroups on a CU, which the model leaves out; against one thread per
// node and one step per launch the choice still gives, FP64 / FP32, 1000^2 nodes
// 25.7 -> 12.6 / 18.6 -> 7.2, 3000 x 1000 66 -> 50 / 48 -> 32, 6000^2 967 -> 638 /
// 660 -> 362 us a step.
template <typename SH>
inline int d2q9_steps(SH* s, int n) {
    int best = 1;
    double best_t = 0;
    for (int t = 1; t <= kD2MaxSteps; ++t) {
        const int64_t blocks = d2q9_blocks(s, n, t), rounds = (blocks + 255) / 256;
        const double f = std::min(1.0, blocks / 256.0);
        const double us = (3.4 + 1.6 * f) / t + rounds * (1.1 + 0.3 * f);
        if (t == 1 || us < best_t) {
            best = t;
            best_t = us;
        }
    }
    return best;
}

// State upload: staging FP64 (drho0, u0) for nodes [i0, i0 + len) of one
// sample into both buffers; v = u + g/2; solid nodes get exact zeros.
template <int P>
__global__ void k_upload(StepArgs a, int s, const uint8_t* __restrict__ solid,
                         const double* __restrict__ drho0, const double* __restrict__ u0,
                         int64_t i0, int64_t len) {
    using St = Storage<P>;
    using S = typename St::S;
    using T = typename St::T;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= len) return;
    const SampleDev& sd = a.samples[s];
    const int64_t i = i0 + t;
    T d = 0, vx = 0, vy = 0, vz = 0;
    if (!solid[t]) {
        // widen/narrow from FP64 in the compute type, then add g/2 there
        d = drho0 ? (T)drho0[t] : (T)0;
        vx = (u0 ? (T)u0[t] : (T)0) + gh_of<T>(a, 0);
        vy = (u0 ? (T)u0[len + t] : (T)0) + gh_of<T>(a, 1);
        vz = (u0 ? (T)u0[2 * len + t] : (T)0) + gh_of<T>(a, 2);
    }
    const T sr = scale_rho<P>(a), su = scale_u<P>(a);
    const int x = (int)(i % sd.nx);
    const int y = (int)((i / sd.nx) % sd.ny);
    const int z = (int)(i / ((int64_t)sd.nx * sd.ny));
    const int64_t e = state_slot(a.base, sd, x, y, z, i);
    if (e < 0) return;  // all-solid chunk of the packed layout: no storage
    for (int b = 0; b < 2; ++b) {
        S* p = reinterpret_cast<S*>(a.base + sd.state[b]);
        St::store(p, e, d, sr);
        St::store(p + sd.stride, e, vx, su);
        St::store(p + 2 * sd.stride, e, vy, su);
        St::store(p + 3 * sd.stride, e, vz, su);
    }
}

// State readback: nodes [i0, i0 + len) of one sample, current buffer, as FP64
// (out_d: drho; out_u: ux | uy | uz, each len values; either may be null; both
// may lie in pinned host memory); u = v - g/2 in FP64; solid nodes read 0.
// With phys_rho out_d holds rho = 1 + drho (formed in FP64; 1 at solid nodes)
// instead.  *bad is set where a fluid value is not finite.
template <int P>
__global__ void k_export(StepArgs a, int s, double* __restrict__ out_d, double* __restrict__ out_u,
                         int64_t i0, int64_t len, double* bad, int phys_rho) {
    using St = Storage<P>;
    using S = typename St::S;
    using T = typename St::T;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= len) return;
    const SampleDev& sd = a.samples[s];
    const int64_t i = i0 + t;
    const int x = (int)(i % sd.nx);
    const int y = (int)((i / sd.nx) % sd.ny);
    const int z = (int)(i / ((int64_t)sd.nx * sd.ny));
    const uint32_t* mask = reinterpret_cast<const uint32_t*>(a.base + sd.mask);
    double d = 0, ux = 0, uy = 0, uz = 0;
    if (!solid_bit(mask, sd.words, sd.ny, x, y, z)) {
        const S* p = reinterpret_cast<const S*>(a.base + sd.state[a.parity]);
        const int64_t e = state_slot(a.base, sd, x, y, z, i);  // a fluid node has a slot
        d = (double)St::load(p, e, inv_scale_rho<P>(a));
        ux = (double)St::load(p + sd.stride, e, inv_scale_u<P>(a)) - a.gh[0];
        uy = (double)St::load(p + 2 * sd.stride, e, inv_scale_u<P>(a)) - a.gh[1];
        uz = (double)St::load(p + 3 * sd.stride, e, inv_scale_u<P>(a)) - a.gh[2];
        if (!isfinite(d) || !isfinite(ux) || !isfinite(uy) || !isfinite(uz)) *bad = 1.0;
    }
    if (out_d) out_d[t] = phys_rho ? 1.0 + d : d;
    if (out_u) {
        out_u[t] = ux;
        out_u[len + t] = uy;
        out_u[2 * len + t] = uz;
    }
}

// ---------------------------------------------------------------------------
// FP64 reductions (mass and permeability), deterministic: block b owns the
// contiguous node range [b*chunk, (b+1)*chunk); each thread sums its strided
// sub-sequence in order, each wave combines its lanes with a fixed butterfly
// of lane shuffles, and the block's first wave adds the four wave totals in
// wave order.  Partials: (sum drho, sum u_axis, fluid count, non-finite
// count) per block.  The same order on every run gives the same bits.
// ---------------------------------------------------------------------------
constexpr int kReduceBlocks = 1024;
constexpr int kReduceThreads = 256;
constexpr int kReduceWaves = kReduceThreads / 64;

// Sum over the 64 lanes of a wave by an xor butterfly: lane i adds lane
// i ^ m for m = 32, 16, ..., 1.  Both partners form the same sum (addition
// commutes exactly), so every lane ends with the same total.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

// The four sums of a block in wave order; valid in thread 0.
__device__ __forceinline__ void block_sum4(double (&acc)[4]) {
    __shared__ double sh[kReduceWaves][4];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = wave_sum(acc[c]);
    if (lane == 0)
#pragma unroll
        for (int c = 0; c < 4; ++c) sh[wave][c] = acc[c];
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            double t = sh[0][c];
            for (int w = 1; w < kReduceWaves; ++w) t += sh[w][c];
            acc[c] = t;
        }
}

template <int P>
__global__ __launch_bounds__(kReduceThreads) void k_reduce_partial(StepArgs a, int s, int axis,
                                                                   double* __restrict__ partial) {
    using St = Storage<P>;
    using S = typename St::S;
    const SampleDev& sd = a.samples[s];
    const int64_t chunk = (sd.n + kReduceBlocks - 1) / kReduceBlocks;
    const int64_t beg = (int64_t)blockIdx.x * chunk;
    const int64_t end = min(beg + chunk, sd.n);
    const uint32_t* mask = reinterpret_cast<const uint32_t*>(a.base + sd.mask);
    const S* p = reinterpret_cast<const S*>(a.base + sd.state[a.parity]);
    const S* pu = p + (int64_t)(1 + axis) * sd.stride;
    double acc[4] = {0, 0, 0, 0};  // sum drho, sum u, fluid nodes, non-finite nodes
    for (int64_t i = beg + threadIdx.x; i < end; i += kReduceThreads) {
        const int x = (int)(i % sd.nx);
        const int y = (int)((i / sd.nx) % sd.ny);
        const int z = (int)(i / ((int64_t)sd.nx * sd.ny));
        if (solid_bit(mask, sd.words, sd.ny, x, y, z)) continue;
        const int64_t e = state_slot(a.base, sd, x, y, z, i);
        const double d = (double)St::load(p, e, inv_scale_rho<P>(a));
        const double u = (double)St::load(pu, e, inv_scale_u<P>(a)) - a.gh[axis];
        if (!isfinite(d) || !isfinite(u)) { acc[3] += 1; continue; }
        acc[0] += d;
        acc[1] += u;
        acc[2] += 1;
    }
    block_sum4(acc);
    if (threadIdx.x == 0)
#pragma unroll
        for (int c = 0; c < 4; ++c) partial[blockIdx.x * 4 + c] = acc[c];
}

}  // namespace tau1
