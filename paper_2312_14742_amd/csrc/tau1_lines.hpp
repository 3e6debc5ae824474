// tau1_lines.hpp -- step kernel for rows of any length, in every precision: one
// node per lane.
//
// A wave owns a window of at most 62 consecutive x-nodes of one row (plus the
// node on either side in the first and last lane, periodic in x; rows of 64
// nodes need no such lanes) and marches along z over a segment of planes.  Per
// source plane it reads the window of rows y - 1, y, y + 1 with one coalesced
// load per row and array, requested one plane ahead, forms the sources and
// sends each group of directions (tau1_sums.hpp) to the planes z - 1, z, z + 1;
// values for x +- 1 move one lane by DPP.
//
// Solid links need no vector work: with one node per lane, the solid bits of a
// row window are a lane mask.  They are read with scalar loads from the
// extended mask, shifted on the scalar unit, and select each bounced-back
// value with one v_cndmask; a window without a wall node skips them all.
//
// What bounds it: vector issue (about 210 instructions a node and plane in
// FP32 D3Q19, wall returns included, beside 140 scalar ones) at the share of
// lanes that a row fills, and on small lattices the chain of planes of one
// segment, so segments are cut until the waves fill the card (lines_tiling).
// Measured per step against a pull kernel with one thread per node, which
// read 76 values and formed 64-bit addresses and zero-component products for
// each: 32^3 FP64 8.4 -> 3.9 us, porous 128^3 FP64 135 -> 36 us, porous 150 x
// 110 x 90 FP32 56 -> 17.5 us.
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

// The sums of one node in one destination plane, and the stored state of one
// node.
template <typename T>
struct LnSum {
    T t, s, x, y;
};
template <typename T>
struct LnNode {
    T d, vx, vy, vz;
};

// Solid bits of a row window for c_x = -1, 0, +1: bit l of m[c_x + 1] is set
// when the node at c_x from lane l's node is solid.
struct LnMask {
    uint64_t m[3];
};

// The four words of the extended mask that hold a row window's bits.
struct LnWords {
    uint32_t w[4];
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
    T isr, isu, sr, su, gx, gy, gz;
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
__device__ __forceinline__ SrcT<typename Storage<P>::T> ln_src(const LnItem<P>& it,
                                                              const LnNode<typename Storage<P>::S>& r) {
    using St = Storage<P>;
    return make_src(St::load(&r.d, 0, it.isr), St::load(&r.vx, 0, it.isu), St::load(&r.vy, 0, it.isu),
                    St::load(&r.vz, 0, it.isu));
}

// Scalar loads: the mask is constant while a step runs and the row uniform.
__device__ __forceinline__ void ln_words(const char* row, LnWords& o) {
    typedef const __attribute__((address_space(4))) uint32_t word_t;
    word_t* w = (word_t*)row;
#pragma unroll
    for (int i = 0; i < 4; ++i) o.w[i] = w[i];
}

// The lane masks of a row window whose first bit is bit xs of the words.
__device__ __forceinline__ LnMask ln_mask(const LnWords& w, int xs) {
    const uint64_t a = ((uint64_t)w.w[1] << 32) | w.w[0];
    const uint64_t b = ((uint64_t)w.w[3] << 32) | w.w[2];
    const uint64_t lo = (a >> xs) | ((b << (63 - xs)) << 1);
    const uint64_t hi = b >> xs;
    return {{lo, (lo >> 1) | (hi << 63), (lo >> 2) | (hi << 62)}};
}

template <int Q, int CY, int CZ, typename T>
__device__ __forceinline__ void ln_group(const SrcT<T>& s, T f, T g, LnSum<T>& q, T& m) {
    using G = Group<Q, CY, CZ>;
    if constexpr (G::has0 || G::hasx) {
        level_z<CZ>(s, f, g);
        T a = 0, b = 0;
        if constexpr (G::hasx) {
            T fp, fm;
            level_x(s, f, g, fp, fm);
            a = ln_prev(fp);
            b = ln_next(fm);
        }
        add_group<Q, CY, CZ>(group_sum<Q, CY, CZ>(f, a, b), G::hasx ? a - b : (T)0, q.t, q.s, q.x,
                             q.y, m);
    }
}

// A source row's directions c_y = CY; ZS as in the z-march's step: 0 = a plane
// of the segment, +1 / -1 = the plane before / after it (to one plane only).
template <int Q, int CY, int ZS, typename T>
__device__ __forceinline__ void ln_push(const SrcT<T>& s, LnSum<T>& pm, LnSum<T>& pc, LnSum<T>& pp,
                                        T& m) {
    T f, g;
    level_y<CY>(s, f, g);
    if constexpr (ZS == 0) ln_group<Q, CY, 0>(s, f, g, pc, m);
    if constexpr (ZS >= 0) ln_group<Q, CY, 1>(s, f, g, pp, m);
    if constexpr (ZS <= 0) ln_group<Q, CY, -1>(s, f, g, pm, m);
}

// Solid bits of rows y - 1, y, y + 1 of one plane.
struct LnSolid {
    LnMask row[3];
};

// The selection of wall_sums: direction k's value in the lanes whose neighbour
// x + c_k is solid (sm, sc, sp: planes z - 1, z, z + 1; fluid: the window's
// fluid nodes).
template <int Q>
struct LnPick {
    const LnSolid &sm, &sc, &sp;
    uint64_t fluid;
    template <typename K>
    __device__ __forceinline__ uint64_t links(K) const {
        constexpr Dir c = Lattice<Q>::c[K::value];
        const LnSolid& s = c.z < 0 ? sm : c.z > 0 ? sp : sc;
        return s.row[c.y + 1].m[c.x + 1] & fluid;
    }
    template <typename K, typename T>
    __device__ __forceinline__ T operator()(K k, T u) const {
        return __builtin_amdgcn_inverse_ballot_w64(links(k)) ? u : (T)0;
    }
};

template <int Q, int K = 1>
__device__ __forceinline__ uint64_t ln_any_link(const LnPick<Q>& p) {
    if constexpr (K >= Q) return 0;
    else return p.links(std::integral_constant<int, K>{}) | ln_any_link<Q, K + 1>(p);
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

// One source plane zs, whose rows are in `ahead`; requests plane zs + 1's rows
// unless it is the last.  sm, sc: solid bits of planes zs - 1 and zs; sp
// receives those of zs + 1.
template <int Q, int P, int ZS>
__device__ __forceinline__ void ln_step(const LnItem<P>& it, int zs, LnSum<typename Storage<P>::T>& pm,
                                        LnSum<typename Storage<P>::T>& pc,
                                        LnSum<typename Storage<P>::T>& pp, const LnSolid& sm,
                                        const LnSolid& sc, LnSolid& sp, LnRows<P>& ahead, LnAt& at,
                                        char*& out) {
    using St = Storage<P>;
    using T = typename St::T;
    using S = typename St::S;
    const SrcT<T> m1 = ln_src(it, ahead.row[0]), o = ln_src(it, ahead.row[1]),
                  p1 = ln_src(it, ahead.row[2]);
    if constexpr (ZS >= 0) {
        ln_next_plane(it, at);
        ln_request(it, at, ahead);
    }
    T m = 0;
    ln_push<Q, 0, ZS>(o, pm, pc, pp, m);
    ln_push<Q, 1, ZS>(m1, pm, pc, pp, m);
    ln_push<Q, -1, ZS>(p1, pm, pc, pp, m);
    if constexpr (ZS >= 0) {
        // the mask words have landed meanwhile
#pragma unroll
        for (int i = 0; i < 3; ++i) {
#pragma unroll
            for (int k = 0; k < 4; ++k) asm volatile("" : "+s"(ahead.words[i].w[k]));
            sp.row[i] = ln_mask(ahead.words[i], it.xs);
        }
    }
    if constexpr (ZS == 0) {
        const LnPick<Q> pick{sm, sc, sp, it.lanes & ~sc.row[1].m[1]};
        if (ln_any_link(pick)) {
            T r[4];
            wall_sums<Q>(o, pick, r);
            pc.s += r[0];
            pc.x += r[1];
            pc.y += r[2];
            pc.t += r[3];
        }
    }
    // plane zs - 1 is complete: finalise and store the window, solid nodes as zeros
    if (ZS < 0 || (ZS == 0 && zs > it.z0)) {
        T d, vx, vy, vz;
        finish_node<Q>(pm.t, pm.s, m, pm.x, pm.y, it.gx, it.gy, it.gz, d, vx, vy, vz);
        const bool f = !__builtin_amdgcn_inverse_ballot_w64(sm.row[1].m[1]);
        if (__builtin_amdgcn_inverse_ballot_w64(it.lanes)) {
            uint32_t x = it.xb;
            asm volatile("" : "+v"(x));
            St::store(reinterpret_cast<S*>(out + x), 0, f ? d : (T)0, it.sr);
            St::store(reinterpret_cast<S*>(out + it.stride + x), 0, f ? vx : (T)0, it.su);
            St::store(reinterpret_cast<S*>(out + 2 * it.stride + x), 0, f ? vy : (T)0, it.su);
            St::store(reinterpret_cast<S*>(out + 3 * it.stride + x), 0, f ? vz : (T)0, it.su);
        }
        out += it.plane;
    }
}

template <int Q, int P>
__global__ __launch_bounds__(kLnThreads)
__attribute__((amdgpu_waves_per_eu(P == kF64 ? 3 : 6))) void k_lines(StepArgs a) {
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
    it.gx = (T)2 * gh_of<T>(a, 0);
    it.gy = (T)2 * gh_of<T>(a, 1);
    it.gz = (T)2 * gh_of<T>(a, 2);

    // bit e of an extended mask row is node e - 1, and lane l's left neighbour
    // is node x0 - halo + l - 1: bit 0 of the window is bit x0 - halo of the row
    // (the word before the first row of the mask, for x0 = 0, lies inside the
    // workspace, and its bit reaches only lane 0's unused left neighbour)
    const int bit0 = x0 - halo;
    it.xs = bit0 & 31;
    LnAt at;
    at.z = (it.z0 == 0 ? it.nz : it.z0) - 1;
    at.pre = reinterpret_cast<const char*>(a.base + sd->state[a.parity]) + at.z * it.plane;
    at.mask = reinterpret_cast<const char*>(a.base + sd->xmask) + (bit0 >> 5) * 4 + at.z * it.mplane;
    char* out = reinterpret_cast<char*>(a.base + sd->state[a.parity ^ 1]) + it.z0 * it.plane + it.row[1];

    LnRows<P> ahead;
    ln_request(it, at, ahead);
    LnSolid sa, sb, sc;
#pragma unroll
    for (int i = 0; i < 3; ++i) sa.row[i] = ln_mask(ahead.words[i], it.xs);
    LnSum<T> A, B, C;
    // the three planes' roles rotate statically (unrolled by three)
    ln_step<Q, P, 1>(it, it.z0 - 1, B, C, A, sc, sa, sb, ahead, at, out);
    int zs = it.z0;
    while (true) {
        ln_step<Q, P, 0>(it, zs, C, A, B, sa, sb, sc, ahead, at, out);
        if (++zs >= it.z1) {
            sa = sb;
            break;
        }
        ln_step<Q, P, 0>(it, zs, A, B, C, sb, sc, sa, ahead, at, out);
        if (++zs >= it.z1) {
            A = B;
            sa = sc;
            break;
        }
        ln_step<Q, P, 0>(it, zs, B, C, A, sc, sa, sb, ahead, at, out);
        if (++zs >= it.z1) {
            A = C;
            break;
        }
    }
    ln_step<Q, P, -1>(it, it.z1, A, B, C, sa, sb, sc, ahead, at, out);
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

// Work of a context's samples for the row kernel: z-segments cut so that the
// waves come to about kLnTarget, and each sample's first workgroup (block0).
// Returns the number of workgroups.  Long segments repeat less work (a segment
// of n planes reads n + 2), short ones fill the card: measured per step on
// 128^3 FP64, 2048 waves 47 us, 3072 36 us, 4600 40 us, 6144 36 us; on 150 x
// 110 x 90 FP32, 2048 22 us, 3072 20 us, 4950 17.5 us, 7590 18.4 us.  FP64 runs
// at four waves per SIMD, the others at seven.
constexpr int64_t kLnTarget = 5000, kLnTarget64 = 3072;
constexpr int kLnMaxLz = 64;
template <typename SH>
inline int64_t lines_tiling(SH* s, int n, int precision) {
    int64_t planes = 0;
    for (int i = 0; i < n; ++i) {
        SampleDev& sd = s[i].dev;
        lines_windows(sd);
        planes += (int64_t)sd.ln_windows * sd.ny * sd.nz;
    }
    const int64_t target = precision == kF64 ? kLnTarget64 : kLnTarget;
    const int64_t lz = std::clamp<int64_t>(planes / target, 1, kLnMaxLz);
    int64_t blocks = 0;
    for (int i = 0; i < n; ++i) {
        SampleDev& sd = s[i].dev;
        const int64_t segs = (sd.nz + lz - 1) / lz;
        sd.ln_lz = (int32_t)((sd.nz + segs - 1) / segs);
        sd.block0 = blocks;
        const int64_t waves = (int64_t)sd.ln_windows * sd.ny * ((sd.nz + sd.ln_lz - 1) / sd.ln_lz);
        blocks += (waves + kLnWaves - 1) / kLnWaves;
    }
    return blocks;
}

}  // namespace tau1
