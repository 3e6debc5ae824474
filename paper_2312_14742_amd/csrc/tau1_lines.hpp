// tau1_lines.hpp -- step kernel for rows of any length, in every precision: one
// node per lane (rows of a few nodes: tau1_nodes.hpp).
//
// A wave owns a window of at most 62 consecutive x-nodes of one row (plus the
// node on either side in the first and last lane, periodic in x; rows of 64
// nodes need no such lanes) and marches along z over a segment of planes.  It
// reads the window of rows y - 1, y, y + 1 with one coalesced load per row and
// array, requested ahead of its use; what goes to x +- 1 moves one lane by DPP.
//
// Two forms of the arithmetic:
//
// FP64 is the reference of the other modes: each node adds what arrives
// direction by direction, in the lattice's order, every operation rounded by
// itself and one division a node.  This is the plain evaluation of Eqs. (3) and
// (9)-(11); with g = 0 its bits are the oracle's.  The wave holds the sources of
// nine rows (planes z - 1, z, z + 1) and finishes one plane at a time, each
// direction formed in the source's lane.
//
// FP32, and 16-bit storage, sum by groups of directions (tau1_sums.hpp): a third
// of the instructions, and the smaller error.  The wave holds the three rows of
// one source plane at a time and sends each group to the planes z - 1, z, z + 1.
//
// Solid links need no vector work to be found: with one node per lane, the
// solid bits of a row window are a lane mask.  They are read with scalar loads
// from the extended mask, rotated on the scalar unit, and select each
// bounced-back value with one v_cndmask; a window (FP64: a pair of opposite
// directions) without a link skips its own values.
//
// What bounds it: vector issue (D3Q19, a node and plane, wall returns included:
// about 500 instructions in FP64, 220 in FP32) at the share of lanes that a row
// fills, and on small lattices the planes in a row that a segment takes, so
// segments are cut until the waves fill the card (lines_tiling).  Measured per
// step against one thread per node, which read 76 values and formed 64-bit
// addresses and zero-component products for each: 32^3 FP64 8.4 -> 4.5 us, porous
// 128^3 FP64 135 -> 53 us, porous 150 x 110 x 90 FP32 56 -> 18 us.
#pragma once

#include <algorithm>

#include "tau1_sums.hpp"

namespace tau1 {

constexpr int kLnWaves = 4;
constexpr int kLnThreads = 64 * kLnWaves;
constexpr int kLnWindow = 62;  // nodes per window when the neighbours take two lanes

// Value of lane l - 1 / l + 1 (the wave's ends wrap).
__device__ __forceinline__ float ln_prev(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(
        __builtin_bit_cast(int, v), 0x13C, 0xf, 0xf, true));  // wave_ror:1
}
__device__ __forceinline__ float ln_next(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(
        __builtin_bit_cast(int, v), 0x134, 0xf, 0xf, true));  // wave_rol:1
}
template <int CTRL>
__device__ __forceinline__ double ln_move64(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double ln_prev(double v) { return ln_move64<0x13C>(v); }
__device__ __forceinline__ double ln_next(double v) { return ln_move64<0x134>(v); }

// The stored state of one node, and what its equilibria are formed from
// (h = 1.5 v.v).
template <typename T>
struct LnNode {
    T d, vx, vy, vz;
};
template <typename T>
struct LnSrc {
    T d, vx, vy, vz, h;
};

// The words of the extended mask that hold a row window's solid bits.
struct LnWords {
    uint32_t w[3];
};

// Constants of one work item (one wave); uniform but for xb and lane masks.
// Rows y - 1, y, y + 1 are addressed by byte offsets from row 0 of the plane.
template <int P>
struct LnItem {
    using S = typename Storage<P>::S;
    using T = typename Storage<P>::T;
    int64_t row[3], mrow[3];    // byte offsets of the rows in a plane: state, mask
    int64_t plane, mplane;      // bytes of a plane
    int64_t stride;             // bytes between the state arrays
    int nz, z0, z1, xs;
    uint32_t xb;                // byte offset of the lane's node in its row
    uint64_t lanes;             // lanes whose node belongs to the window
    T isr, isu, sr, su;
    T gx, gy, gz;               // g / 2 (FP64), g (FP32)
};

// The march's position: plane to be requested next.
struct LnAt {
    const char* pre;   // its state
    const char* mask;  // its extended mask, at the window's first word
    int z;
};

template <int P>
__device__ __forceinline__ void ln_next_plane(const LnItem<P>& it, LnAt& at) {
    const bool wrap = ++at.z == it.nz;
    at.pre += wrap ? it.plane - it.nz * it.plane : it.plane;
    at.mask += wrap ? it.mplane - it.nz * it.mplane : it.mplane;
    at.z = wrap ? 0 : at.z;
}

// One lane's state in one row: uniform row pointers and a 32-bit lane offset
// (the offset is fixed in this block, so that the loads take it as it is
// instead of 64-bit lane addresses).
template <int P>
__device__ __forceinline__ void ln_load(const LnItem<P>& it, const char* row,
                                        LnNode<typename Storage<P>::S>& r) {
    using S = typename Storage<P>::S;
    uint32_t x = it.xb;
    asm volatile("" : "+v"(x));
    r.d = *reinterpret_cast<const S*>(row + x);
    r.vx = *reinterpret_cast<const S*>(row + it.stride + x);
    r.vy = *reinterpret_cast<const S*>(row + 2 * it.stride + x);
    r.vz = *reinterpret_cast<const S*>(row + 3 * it.stride + x);
}

template <int P>
__device__ __forceinline__ LnSrc<typename Storage<P>::T> ln_src(const LnItem<P>& it,
                                                               const LnNode<typename Storage<P>::S>& r) {
#pragma clang fp contract(off)
    using St = Storage<P>;
    using T = typename St::T;
    LnSrc<T> s;
    s.d = St::load(&r.d, 0, it.isr);
    s.vx = St::load(&r.vx, 0, it.isu);
    s.vy = St::load(&r.vy, 0, it.isu);
    s.vz = St::load(&r.vz, 0, it.isu);
    s.h = (T)1.5 * ((s.vx * s.vx + s.vy * s.vy) + s.vz * s.vz);
    return s;
}

// Scalar loads: the mask is constant while a step runs and the row uniform.
__device__ __forceinline__ void ln_words(const char* row, LnWords& o) {
    typedef const __attribute__((address_space(4))) uint32_t word_t;
    word_t* w = (word_t*)row;
#pragma unroll
    for (int i = 0; i < 3; ++i) o.w[i] = w[i];
}

// Solid lanes of a row window whose first bit is bit xs of the words.
__device__ __forceinline__ uint64_t ln_mask(const LnWords& w, int xs) {
    const uint64_t a = ((uint64_t)w.w[1] << 32) | w.w[0];
    return (a >> xs) | (((uint64_t)w.w[2] << (63 - xs)) << 1);
}

// c.v of direction K at a source.
template <int Q, int K, typename T>
__device__ __forceinline__ T ln_cu(const LnSrc<T>& s) {
#pragma clang fp contract(off)
    constexpr Dir c = Lattice<Q>::c[K];
    T cu = 0;
    if constexpr (c.x != 0) cu = c.x > 0 ? s.vx : -s.vx;
    if constexpr (c.y != 0) {
        const T v = c.y > 0 ? s.vy : -s.vy;
        cu = c.x != 0 ? cu + v : v;
    }
    if constexpr (c.z != 0) {
        const T v = c.z > 0 ? s.vz : -s.vz;
        cu = c.x != 0 || c.y != 0 ? cu + v : v;
    }
    return cu;
}

// What a source sends in direction K: Eq. (3) minus its weight.
template <int Q, int K, typename T>
__device__ __forceinline__ T ln_feq(const LnSrc<T>& s) {
#pragma clang fp contract(off)
    const T cu = ln_cu<Q, K>(s);
    const T p = ((T)3 * cu + ((T)4.5 * cu) * cu) - s.h;
    return (T)weight<Q>(K) * (s.d + ((T)1 + s.d) * p);
}

// Source rows y - 1, y, y + 1 of one plane.
template <typename T>
struct LnPlane {
    LnSrc<T> row[3];
};

// What arrives in direction K from the planes z - 1, z, z + 1.
template <int Q, int K, typename T>
__device__ __forceinline__ T ln_arrive(const LnPlane<T>& pm, const LnPlane<T>& pc,
                                       const LnPlane<T>& pp) {
    constexpr Dir c = Lattice<Q>::c[K];
    const LnPlane<T>& p = c.z > 0 ? pm : c.z < 0 ? pp : pc;
    const T f = ln_feq<Q, K>(p.row[1 - c.y]);
    if constexpr (c.x > 0) return ln_prev(f);
    else if constexpr (c.x < 0) return ln_next(f);
    else return f;
}

// Adds direction K's value to a node's density and momentum.
template <int Q, int K, typename T>
__device__ __forceinline__ void ln_add(LnNode<T>& n, T f) {
#pragma clang fp contract(off)
    constexpr Dir c = Lattice<Q>::c[K];
    n.d += f;
    if constexpr (c.x != 0) n.vx += c.x > 0 ? f : -f;
    if constexpr (c.y != 0) n.vy += c.y > 0 ? f : -f;
    if constexpr (c.z != 0) n.vz += c.z > 0 ? f : -f;
}

// Solid lanes of rows y - 1, y, y + 1 of one plane.
struct LnSolid {
    uint64_t row[3];
};

// Lanes whose neighbour x + c_K is solid (sm, sc, sp: planes z - 1, z, z + 1):
// the row's solid lanes, rotated by one for c_x, as the values move.
template <int Q, int K>
__device__ __forceinline__ uint64_t ln_links(const LnSolid& sm, const LnSolid& sc, const LnSolid& sp) {
    constexpr Dir c = Lattice<Q>::c[K];
    const LnSolid& s = c.z < 0 ? sm : c.z > 0 ? sp : sc;
    const uint64_t m = s.row[c.y + 1];
    return c.x < 0 ? (m << 1) | (m >> 63) : c.x > 0 ? (m >> 1) | (m << 63) : m;
}

// Directions K and K + 1 (opposite) of one node onwards, in order.  A source
// x - c_K that is solid returns the node's own value in the opposite direction
// (halfway bounce-back, Eq. (11)); the two own values share their terms, and are
// formed only where some lane of the window needs one.
template <int Q, int K = 1, typename T>
__device__ __forceinline__ void ln_gather(const LnPlane<T>& pm, const LnPlane<T>& pc,
                                          const LnPlane<T>& pp, const LnSolid& sm,
                                          const LnSolid& sc, const LnSolid& sp, uint64_t fluid,
                                          LnNode<T>& n) {
#pragma clang fp contract(off)
    if constexpr (K < Q) {
        T a = ln_arrive<Q, K>(pm, pc, pp), b = ln_arrive<Q, K + 1>(pm, pc, pp);
        const uint64_t la = ln_links<Q, K + 1>(sm, sc, sp) & fluid;  // x - c_K is x + c_(K + 1)
        const uint64_t lb = ln_links<Q, K>(sm, sc, sp) & fluid;
        if (la | lb) {
            const LnSrc<T>& o = pc.row[1];
            const T cu = ln_cu<Q, K>(o), rho = (T)1 + o.d;
            const T t1 = (T)3 * cu, t2 = ((T)4.5 * cu) * cu;
            const T fk = (T)weight<Q>(K) * (o.d + rho * ((t1 + t2) - o.h));
            const T fo = (T)weight<Q>(K) * (o.d + rho * ((t2 - t1) - o.h));
            a = __builtin_amdgcn_inverse_ballot_w64(la) ? fo : a;
            b = __builtin_amdgcn_inverse_ballot_w64(lb) ? fk : b;
        }
        ln_add<Q, K>(n, a);
        ln_add<Q, K + 1>(n, b);
        ln_gather<Q, K + 2>(pm, pc, pp, sm, sc, sp, fluid, n);
    }
}

// The three rows of a plane as requested: raw state and mask words.
template <int P>
struct LnRows {
    LnNode<typename Storage<P>::S> row[3];
    LnWords words[3];
};

template <int P>
__device__ __forceinline__ void ln_request(const LnItem<P>& it, const LnAt& at, LnRows<P>& r) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        ln_load(it, at.pre + it.row[i], r.row[i]);
        ln_words(at.mask + it.mrow[i], r.words[i]);
    }
}

// Solid bits of a requested plane's rows, landed.
template <int P>
__device__ __forceinline__ void ln_solid(const LnItem<P>& it, LnRows<P>& r, LnSolid& s) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
#pragma unroll
        for (int k = 0; k < 3; ++k) asm volatile("" : "+s"(r.words[i].w[k]));
        s.row[i] = ln_mask(r.words[i], it.xs);
    }
}

// FP64: the rows of a requested plane, landed: sources and solid bits.
template <int P>
__device__ __forceinline__ void ln_take(const LnItem<P>& it, LnRows<P>& r,
                                        LnPlane<typename Storage<P>::T>& p, LnSolid& s) {
#pragma unroll
    for (int i = 0; i < 3; ++i) p.row[i] = ln_src(it, r.row[i]);
    ln_solid(it, r, s);
}

// Stores a window of finished nodes, solid ones as zeros.
template <int P>
__device__ __forceinline__ void ln_store(const LnItem<P>& it, char* out,
                                         const LnNode<typename Storage<P>::T>& n, uint64_t solid) {
    using St = Storage<P>;
    using T = typename St::T;
    using S = typename St::S;
    const bool f = !__builtin_amdgcn_inverse_ballot_w64(solid);
    if (__builtin_amdgcn_inverse_ballot_w64(it.lanes)) {
        uint32_t x = it.xb;
        asm volatile("" : "+v"(x));
        St::store(reinterpret_cast<S*>(out + x), 0, f ? n.d : (T)0, it.sr);
        St::store(reinterpret_cast<S*>(out + it.stride + x), 0, f ? n.vx : (T)0, it.su);
        St::store(reinterpret_cast<S*>(out + 2 * it.stride + x), 0, f ? n.vy : (T)0, it.su);
        St::store(reinterpret_cast<S*>(out + 3 * it.stride + x), 0, f ? n.vz : (T)0, it.su);
    }
}

// FP64: one plane z, with the planes z - 1 and z at hand and the rows of z + 1 in
// `ahead`; requests plane z + 2's unless z is the segment's last.
template <int Q, int P>
__device__ __forceinline__ void ln_step(const LnItem<P>& it, int z,
                                        const LnPlane<typename Storage<P>::T>& pm,
                                        const LnPlane<typename Storage<P>::T>& pc,
                                        LnPlane<typename Storage<P>::T>& pp, const LnSolid& sm,
                                        const LnSolid& sc, LnSolid& sp, LnRows<P>& ahead, LnAt& at,
                                        char*& out) {
#pragma clang fp contract(off)
    using T = typename Storage<P>::T;
    ln_take(it, ahead, pp, sp);
    if (z + 1 < it.z1) {
        ln_next_plane(it, at);
        ln_request(it, at, ahead);
    }
    LnNode<T> n{0, 0, 0, 0};
    {
        const LnSrc<T>& o = pc.row[1];
        n.d += (T)weight<Q>(0) * (o.d + ((T)1 + o.d) * ((T)0 - o.h));
    }
    const uint64_t solid = sc.row[1];
    ln_gather<Q>(pm, pc, pp, sm, sc, sp, it.lanes & ~solid, n);
    const T r = (T)1 / ((T)1 + n.d);
    n.vx = (n.vx * r + it.gx) + it.gx;
    n.vy = (n.vy * r + it.gy) + it.gy;
    n.vz = (n.vz * r + it.gz) + it.gz;
    ln_store(it, out, n, solid);
    out += it.plane;
}

// FP32: the sums of one node in one destination plane.
struct LnSum {
    float t, s, x, y;
};

template <int Q, int CY, int CZ>
__device__ __forceinline__ void ln_group(const Src& s, float f, float g, LnSum& q, float& m) {
    using G = Group<Q, CY, CZ>;
    if constexpr (G::has0 || G::hasx) {
        level_z<CZ>(s, f, g);
        float a = 0.0f, b = 0.0f;
        if constexpr (G::hasx) {
            float fp, fm;
            level_x(s, f, g, fp, fm);
            a = ln_prev(fp);
            b = ln_next(fm);
        }
        add_group<Q, CY, CZ>(group_sum<Q, CY, CZ>(f, a, b), G::hasx ? a - b : 0.0f, q.t, q.s, q.x,
                             q.y, m);
    }
}

// A source row's directions c_y = CY; ZS as in the z-march's step: 0 = a plane
// of the segment, +1 / -1 = the plane before / after it (to one plane only).
template <int Q, int CY, int ZS>
__device__ __forceinline__ void ln_push(const Src& s, LnSum& pm, LnSum& pc, LnSum& pp, float& m) {
    float f, g;
    level_y<CY>(s, f, g);
    if constexpr (ZS == 0) ln_group<Q, CY, 0>(s, f, g, pc, m);
    if constexpr (ZS >= 0) ln_group<Q, CY, 1>(s, f, g, pp, m);
    if constexpr (ZS <= 0) ln_group<Q, CY, -1>(s, f, g, pm, m);
}

// The selection of wall_sums: direction k's value in the lanes whose neighbour
// x + c_k is solid (fluid: the window's fluid nodes).
template <int Q>
struct LnPick {
    const LnSolid &sm, &sc, &sp;
    uint64_t fluid;
    template <typename K>
    __device__ __forceinline__ uint64_t links(K) const {
        return ln_links<Q, K::value>(sm, sc, sp) & fluid;
    }
    template <typename K>
    __device__ __forceinline__ float operator()(K k, float u) const {
        return __builtin_amdgcn_inverse_ballot_w64(links(k)) ? u : 0.0f;
    }
};

template <int Q, int K = 1>
__device__ __forceinline__ uint64_t ln_any_link(const LnPick<Q>& p) {
    if constexpr (K >= Q) return 0;
    else return p.links(std::integral_constant<int, K>{}) | ln_any_link<Q, K + 1>(p);
}

template <int P>
__device__ __forceinline__ Src ln_src32(const LnItem<P>& it, const LnNode<typename Storage<P>::S>& r) {
    using St = Storage<P>;
    return make_src(St::load(&r.d, 0, it.isr), St::load(&r.vx, 0, it.isu), St::load(&r.vy, 0, it.isu),
                    St::load(&r.vz, 0, it.isu));
}

// FP32: one source plane zs, whose rows are in `ahead`; requests plane zs + 1's
// rows unless it is the last.  sm, sc: solid bits of planes zs - 1 and zs; sp
// receives those of zs + 1.
template <int Q, int P, int ZS>
__device__ __forceinline__ void ln_sstep(const LnItem<P>& it, int zs, LnSum& pm, LnSum& pc, LnSum& pp,
                                         const LnSolid& sm, const LnSolid& sc, LnSolid& sp,
                                         LnRows<P>& ahead, LnAt& at, char*& out) {
    using St = Storage<P>;
    using S = typename St::S;
    const Src m1 = ln_src32(it, ahead.row[0]), o = ln_src32(it, ahead.row[1]),
              p1 = ln_src32(it, ahead.row[2]);
    if constexpr (ZS >= 0) {
        ln_next_plane(it, at);
        ln_request(it, at, ahead);
    }
    float m = 0.0f;
    ln_push<Q, 0, ZS>(o, pm, pc, pp, m);
    ln_push<Q, 1, ZS>(m1, pm, pc, pp, m);
    ln_push<Q, -1, ZS>(p1, pm, pc, pp, m);
    if constexpr (ZS >= 0) ln_solid(it, ahead, sp);  // the mask words have landed meanwhile
    if constexpr (ZS == 0) {
        const LnPick<Q> pick{sm, sc, sp, it.lanes & ~sc.row[1]};
        if (ln_any_link(pick)) {
            float r[4];
            wall_sums<Q>(o, pick, r);
            pc.s += r[0];
            pc.x += r[1];
            pc.y += r[2];
            pc.t += r[3];
        }
    }
    // plane zs - 1 is complete: finalise and store the window
    if (ZS < 0 || (ZS == 0 && zs > it.z0)) {
        LnNode<float> n;
        finish_node<Q>(pm.t, pm.s, m, pm.x, pm.y, it.gx, it.gy, it.gz, n.d, n.vx, n.vy, n.vz);
        ln_store(it, out, n, sm.row[1]);
        out += it.plane;
    }
}

// Waves per SIMD: in FP64 as many as the sources of nine rows leave without
// spilling in the loop (one more: D3Q19 128^3 52 -> 144 us); FP32 takes 51-60
// registers, which is all eight.
constexpr int ln_waves(int q, int p) { return p == kF64 ? (q == 27 ? 2 : 3) : 8; }

template <int Q, int P>
__global__ __launch_bounds__(kLnThreads)
__attribute__((amdgpu_waves_per_eu(ln_waves(Q, P)))) void k_lines(StepArgs a) {
    using St = Storage<P>;
    using T = typename St::T;
    using S = typename St::S;
    // XCD-aware order: dispatch is round-robin over 8 XCDs, and each XCD takes
    // a contiguous range of the work, so that the rows next to a wave's are
    // mostly read through the same L2
    const uint32_t per = gridDim.x / 8;
    const uint32_t b = (blockIdx.x % 8) * per + blockIdx.x / 8;
    if (b >= (uint32_t)a.lblocks) return;
    int si = 0;
    if (a.nsamples > 1) {
        int lo = 0, hi = a.nsamples - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (a.samples[mid].block0 <= (int64_t)b) lo = mid; else hi = mid - 1;
        }
        si = __builtin_amdgcn_readfirstlane(lo);
    }
    const SampleDev* sd = a.samples + si;
    const int nx = sd->nx, ny = sd->ny, halo = sd->ln_halo;
    LnItem<P> it;
    it.nz = sd->nz;
    // work item: row fastest, then window, then z-segment
    const uint32_t w = __builtin_amdgcn_readfirstlane(
        (b - (uint32_t)sd->block0) * kLnWaves + (threadIdx.x >> 6));
    const uint32_t col = w / (uint32_t)ny, y = w % (uint32_t)ny;
    const uint32_t seg = col / (uint32_t)sd->ln_windows, win = col % (uint32_t)sd->ln_windows;
    it.z0 = (int)seg * sd->ln_lz;
    if (it.z0 >= it.nz) return;
    it.z1 = min(it.z0 + sd->ln_lz, it.nz);
    const int yr[3] = {y == 0 ? ny - 1 : (int)y - 1, (int)y, (int)y == ny - 1 ? 0 : (int)y + 1};
    const int64_t rowb = (int64_t)nx * sizeof(S), mrowb = (int64_t)sd->xwords * 4;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        it.row[i] = yr[i] * rowb;
        it.mrow[i] = yr[i] * mrowb;
    }
    it.plane = ny * rowb;
    it.mplane = ny * mrowb;
    it.stride = sd->stride * (int64_t)sizeof(S);
    const int x0 = (int)win * sd->ln_nodes;
    const int count = min(sd->ln_nodes, nx - x0);
    it.lanes = (count == 64 ? ~uint64_t(0) : ((uint64_t(1) << count) - 1)) << halo;
    // lanes past the window's right neighbour repeat in-range nodes
    const int lane = __lane_id();
    int x = x0 + min(lane, count + 2 * halo - 1) - halo;
    x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
    it.xb = (uint32_t)x * (uint32_t)sizeof(S);
    it.isr = inv_scale_rho<P>(a);
    it.isu = inv_scale_u<P>(a);
    it.sr = scale_rho<P>(a);
    it.su = scale_u<P>(a);
    constexpr T gs = P == kF64 ? 1 : 2;
    it.gx = gs * gh_of<T>(a, 0);
    it.gy = gs * gh_of<T>(a, 1);
    it.gz = gs * gh_of<T>(a, 2);

    // bit e of an extended mask row is node e - 1, and lane 0 holds node x0 - halo
    // (the words past a row's end reach lanes that hold no node; past the last
    // row lie two words more)
    const int bit0 = x0 - halo + 1;
    it.xs = bit0 & 31;
    LnAt at;
    at.z = (it.z0 == 0 ? it.nz : it.z0) - 1;
    at.pre = reinterpret_cast<const char*>(a.base + sd->state[a.parity]) + at.z * it.plane;
    at.mask = reinterpret_cast<const char*>(a.base + sd->xmask) + (bit0 >> 5) * 4 + at.z * it.mplane;
    char* out = reinterpret_cast<char*>(a.base + sd->state[a.parity ^ 1]) + it.z0 * it.plane + it.row[1];

    if constexpr (P == kF64) {
        // planes z0 - 1, z0 and z0 + 1 are requested together
        LnRows<P> first, second, ahead;
        ln_request(it, at, first);
        ln_next_plane(it, at);
        ln_request(it, at, second);
        ln_next_plane(it, at);
        ln_request(it, at, ahead);
        LnPlane<T> A, B, C;
        LnSolid sa, sb, sc;
        ln_take(it, first, A, sa);
        ln_take(it, second, B, sb);
        // the three planes' roles rotate statically (unrolled by three)
        for (int z = it.z0;;) {
            ln_step<Q, P>(it, z, A, B, C, sa, sb, sc, ahead, at, out);
            if (++z >= it.z1) break;
            ln_step<Q, P>(it, z, B, C, A, sb, sc, sa, ahead, at, out);
            if (++z >= it.z1) break;
            ln_step<Q, P>(it, z, C, A, B, sc, sa, sb, ahead, at, out);
            if (++z >= it.z1) break;
        }
    } else {
        LnRows<P> ahead;
        ln_request(it, at, ahead);
        LnSolid sa, sb, sc;
        ln_solid(it, ahead, sa);
        LnSum A, B, C;
        ln_sstep<Q, P, 1>(it, it.z0 - 1, B, C, A, sc, sa, sb, ahead, at, out);
        int zs = it.z0;
        while (true) {
            ln_sstep<Q, P, 0>(it, zs, C, A, B, sa, sb, sc, ahead, at, out);
            if (++zs >= it.z1) {
                sa = sb;
                break;
            }
            ln_sstep<Q, P, 0>(it, zs, A, B, C, sb, sc, sa, ahead, at, out);
            if (++zs >= it.z1) {
                A = B;
                sa = sc;
                break;
            }
            ln_sstep<Q, P, 0>(it, zs, B, C, A, sc, sa, sb, ahead, at, out);
            if (++zs >= it.z1) {
                A = C;
                break;
            }
        }
        ln_sstep<Q, P, -1>(it, it.z1, A, B, C, sa, sb, sc, ahead, at, out);
    }
}

#define TAU1_LN_TABLE_DECL(PP) void* ln_kernel_##PP(int q);
TAU1_LN_TABLE_DECL(0) TAU1_LN_TABLE_DECL(1) TAU1_LN_TABLE_DECL(2) TAU1_LN_TABLE_DECL(3)
#undef TAU1_LN_TABLE_DECL

inline void* pick_lines(int q, int p) {
    switch (p) {
        case kF64: return ln_kernel_0(q);
        case kF32: return ln_kernel_1(q);
        case kF16: return ln_kernel_2(q);
        case kBF16: return ln_kernel_3(q);
    }
    return nullptr;
}

// Windows of a sample's rows: as few as hold the row, of equal length.
inline void lines_windows(SampleDev& sd) {
    sd.ln_halo = sd.nx == 64 ? 0 : 1;
    sd.ln_windows = sd.ln_halo ? (sd.nx + kLnWindow - 1) / kLnWindow : 1;
    sd.ln_nodes = (sd.nx + sd.ln_windows - 1) / sd.ln_windows;
}

// Modelled time of a step at segments of lz planes, `waves` of them resident per
// SIMD at a time: a segment marches through lz planes after a start of about one
// plane's time, each plane takes a SIMD a time that grows with its waves w like
// 0.5 + w, and a launch runs in rounds of the resident waves.  Over ten lattices
// (FP64 32^3 to 256 x 256 x 128, FP32 and half storage 50^3 to 300 x 200 x 150)
// timed at three to ten lengths each, the length chosen is the fastest or within
// 3 % of it; a count of waves alone is not enough (128^3 FP64, 3 resident: 3072
// waves 52 us, 4224 59 us, 6144 53 us, 8448 56 us).
template <typename SH>
inline double lines_cost(const SH* s, int n, int resident, int lz) {
    int64_t waves = 0;
    int longest = 0;
    for (int i = 0; i < n; ++i) {
        const SampleDev& sd = s[i].dev;
        waves += (int64_t)sd.ln_windows * sd.ny * ((sd.nz + lz - 1) / lz);
        longest = std::max(longest, std::min(lz, sd.nz));
    }
    const int64_t per_simd = (waves + 1023) / 1024;
    const int64_t full = per_simd / resident, rest = per_simd % resident;
    return (longest + 1) * (full * (1.5 + resident) + (rest ? 1.5 + rest : 0.0));
}

// Work of a context's samples for the row kernel: the z-segments of the
// shortest modelled step, and each sample's first workgroup (block0).  Returns
// the number of workgroups.
constexpr int kLnMaxLz = 64;
template <typename SH>
inline int64_t lines_tiling(SH* s, int n, int lattice, int precision) {
    for (int i = 0; i < n; ++i) lines_windows(s[i].dev);
    const int resident = ln_waves(lattice, precision);
    int lz = 1;
    double best = lines_cost(s, n, resident, 1);
    for (int c = 2; c <= kLnMaxLz; ++c) {
        const double t = lines_cost(s, n, resident, c);
        if (t < best) {
            best = t;
            lz = c;
        }
    }
    int64_t blocks = 0;
    for (int i = 0; i < n; ++i) {
        SampleDev& sd = s[i].dev;
        const int segs = (sd.nz + lz - 1) / lz;
        sd.ln_lz = (sd.nz + segs - 1) / segs;
        sd.block0 = blocks;
        const int64_t waves = (int64_t)sd.ln_windows * sd.ny * ((sd.nz + sd.ln_lz - 1) / sd.ln_lz);
        blocks += (waves + kLnWaves - 1) / kLnWaves;
    }
    return blocks;
}

}  // namespace tau1
