// tau1_sums.hpp -- sources, and equilibria and moment sums by groups of
// directions in FP32 (the form of the row and node kernels' FP32 modes; the
// z-march and chunk kernels take the sources from here and sum direction by
// direction).
//
// The directions of a lattice fall into nine groups by (c_y, c_z); a group
// holds at most the directions c_x = 0, +1, -1.  What a group sends to a node
// is needed in two forms only: its density sum
//   t = f_0(x) * W0 + WX * (f_+(x - 1) + f_-(x + 1)),
// which is also its momentum along y (times c_y) and z (times c_z), and the
// difference e = WX * (f_+(x - 1) - f_-(x + 1)), its momentum along x.  All
// weights are multiples of one unit (1/72, 1/36, 1/216 for D3Q15, D3Q19,
// D3Q27), so sums run over small integers and the unit is applied once per
// node.  Per node and step this takes 34 additions on D3Q19 and 53 on D3Q27
// where a sum per direction and component takes 49 and 81.
//
// It is also the more precise form: weights such as 1/18 rounded to FP32 lean
// the same way in every step, which a plain sum collects, while the one unit's
// rounding is known and taken back (finish_node).  Against FP64, over 36 cases
// (20-300 x 20-100 x 20-100 nodes, 50-400 steps), the error is a tenth of the
// plain sum's (geometric mean: density 0.10, velocity 0.09), and smaller in every
// one; without the density's correction and with a reciprocal of 1 ulp it was
// seven and five times as large.
//
// A plane's sums are kept by the source plane they came from:
//   T  from plane z - 1 (c_z = +1), C from plane z, M from plane z + 1:
//   rho - 1 = unit * (T + M) + unit * C,   j_z = T - M,
// so j_z costs one subtraction and a fresh plane needs no clearing.  Wall
// returns with z-momentum r_z go into T, and r_z is taken off C again.
//
// The equilibria of a source are evaluated level by level: f along (c_x, c_y,
// c_z) is a quadratic in each velocity component, so the value and slope at
// (c_y, 0) give those at (c_y, c_z), and those give the two directions c_x =
// +-1 with one shared term (38 operations for the 18 directions of D3Q19
// against 46 one by one).
#pragma once

#include "tau1_args.hpp"

// Multiply-adds fuse only where one expression writes a * b + c (and at the
// explicit fma calls), never across statements: every tile and load schedule
// of a kernel then forms each sum with the same roundings, so results do not
// depend on the tile the autotuner picks.
#pragma clang fp contract(on)

namespace tau1 {

// Per-source quantities: the equilibrium of Eq. (3) minus its weight in a
// direction with cu = c.v is w * (A + cu * (R3 + R45 * cu)) with
// A = drho - 1.5 rho v.v, R3 = 3 rho, R45 = 1.5 R3 (= 4.5 rho), rho = 1 + drho.
// R45 is always formed from R3, so a source shared as (A, R3, v) gives the
// same bits wherever it is evaluated.
struct Src {
    float a, r3, r45, vx, vy, vz;
};

__device__ __forceinline__ Src make_src(float d, float vx, float vy, float vz) {
    Src s;
    const float rho = 1.0f + d;
    const float vv = vx * vx + vy * vy + vz * vz;
    s.a = __builtin_fmaf(-1.5f * rho, vv, d);
    s.r3 = 3.0f * rho;
    s.r45 = 1.5f * s.r3;
    s.vx = vx;
    s.vy = vy;
    s.vz = vz;
    return s;
}

// Weight of a direction with n nonzero components, in units (0: the lattice
// has no such direction), and the unit.
template <int Q>
constexpr int weight_units(int n) {
    using L = Lattice<Q>;
    const double w = n == 0 ? L::w_rest : n == 1 ? L::w_face : n == 2 ? L::w_edge : L::w_corner;
    return (int)(w * L::units + 0.5);
}
template <int Q>
constexpr float weight_unit() { return (float)(1.0 / Lattice<Q>::units); }

// One group of directions (c_y, c_z): whether it holds c_x = 0 and c_x = +-1,
// and their weights.  t is formed as R f_0 + (f_+ + f_-) and added with
// weight WG.
template <int Q, int CY, int CZ>
struct Group {
    static constexpr int n = (CY != 0) + (CZ != 0);
    static constexpr int w0 = weight_units<Q>(n), wx = weight_units<Q>(n + 1);
    static constexpr bool has0 = w0 > 0, hasx = wx > 0;
    static constexpr int r = hasx ? w0 / wx : 1;
    static constexpr int wg = hasx ? wx : w0;
    static_assert(!(has0 && hasx) || w0 % wx == 0, "whole weight ratio");
};

// acc + W * v.
template <int W>
__device__ __forceinline__ float add_w(float acc, float v) {
    if constexpr (W == 1) return acc + v;
    else if constexpr (W == -1) return acc - v;
    else return __builtin_fmaf((float)W, v, acc);
}
// W * v.
template <int W>
__device__ __forceinline__ float mul_w(float v) {
    if constexpr (W == 1) return v;
    else return (float)W * v;
}

// f and slope of a source along (0, CY, 0): f = a + cu (r3 + r45 cu) at cu =
// CY vy, slope g = r3 + 2 r45 cu.
template <int CY>
__device__ __forceinline__ void level_y(const Src& s, float& f, float& g) {
    if constexpr (CY == 0) {
        f = s.a;
        g = s.r3;
    } else {
        const float cu = CY > 0 ? s.vy : -s.vy;
        const float h = __builtin_fmaf(s.r45, cu, s.r3);
        f = __builtin_fmaf(h, cu, s.a);
        g = __builtin_fmaf(s.r45, cu, h);
    }
}

// ... along (0, CY, CZ), from those along (0, CY, 0).
template <int CZ>
__device__ __forceinline__ void level_z(const Src& s, float& f, float& g) {
    if constexpr (CZ != 0) {
        const float tz = s.r45 * s.vz;
        const float q = __builtin_fmaf(tz, s.vz, f);
        f = __builtin_fmaf(CZ > 0 ? g : -g, s.vz, q);
        g = __builtin_fmaf(CZ > 0 ? 2.0f : -2.0f, tz, g);
    }
}

// f along (+1, CY, CZ) and (-1, CY, CZ).
__device__ __forceinline__ void level_x(const Src& s, float f, float g, float& fp, float& fm) {
    const float tx = s.r45 * s.vx;
    const float q = __builtin_fmaf(tx, s.vx, f);
    fp = __builtin_fmaf(g, s.vx, q);
    fm = __builtin_fmaf(-g, s.vx, q);
}

// Partial sums of one node of a destination plane (roles in the file header).
// t: T; s: C; x, y: momentum along x and y.
//
// Adds group (CY, CZ)'s density sum t and x-difference e (weights WG, WX) to
// the plane it goes to.  The first group a plane receives sets its sums: float at
// (0, +1), y at (+1, +1), x at the first group with c_x, C at (0, 0), and M
// (one plane's, of the current step only) at (0, -1).
template <int Q, int CY, int CZ>
__device__ __forceinline__ void add_group(float t, float e, float& pt, float& ps, float& px, float& py, float& m) {
    using G = Group<Q, CY, CZ>;
    if constexpr (CZ > 0) {
        if constexpr (CY == 0) pt = mul_w<G::wg>(t);
        else pt = add_w<G::wg>(pt, t);
        if constexpr (CY > 0) py = mul_w<G::wg>(t);
    } else if constexpr (CZ == 0) {
        if constexpr (CY == 0) ps = mul_w<G::wg>(t);
        else ps = add_w<G::wg>(ps, t);
        if constexpr (CY > 0) py = add_w<G::wg>(py, t);
    } else {
        if constexpr (CY == 0) m = mul_w<G::wg>(t);
        else m = add_w<G::wg>(m, t);
        if constexpr (CY > 0) py = add_w<G::wg>(py, t);
    }
    if constexpr (CY < 0) py = add_w<-G::wg>(py, t);
    if constexpr (G::hasx) {
        constexpr bool first = CZ > 0 && (CY == 0 || (CY > 0 && !Group<Q, 0, 1>::hasx));
        if constexpr (first) px = mul_w<G::wx>(e);
        else px = add_w<G::wx>(px, e);
    }
}

// A group's t from f_0 and the two arriving neighbours' values.
template <int Q, int CY, int CZ>
__device__ __forceinline__ float group_sum(float f0, float fp, float fm) {
    using G = Group<Q, CY, CZ>;
    if constexpr (!G::hasx) return f0;
    else if constexpr (!G::has0) return fp + fm;
    else return __builtin_fmaf((float)G::r, f0, fp + fm);
}

// Index of direction (x, y, z) in the lattice's order, or 0.
template <int Q>
constexpr int dir_index(int x, int y, int z) {
    for (int k = 1; k < Q; ++k)
        if (Lattice<Q>::c[k].x == x && Lattice<Q>::c[k].y == y && Lattice<Q>::c[k].z == z) return k;
    return 0;
}

// Halfway bounce-back (Eq. 11) at one node: every direction k whose neighbour
// x + c_k is solid returns the node's own equilibrium in k along -c_k.
// pick(k, u) is u where that neighbour is solid, else zero.  r: what is added to
// C (density less z-momentum), x, y and float (z-momentum), in units.
template <int Q, int CX, int CY, int CZ, typename Pick>
__device__ __forceinline__ void wall_dir(float f, const Pick& pick, float (&r)[4]) {
    constexpr int w = weight_units<Q>((CX != 0) + (CY != 0) + (CZ != 0));
    const float u = pick(std::integral_constant<int, dir_index<Q>(CX, CY, CZ)>{}, f);
    r[0] = add_w<w>(r[0], u);
    if constexpr (CX != 0) r[1] = add_w<-CX * w>(r[1], u);
    if constexpr (CY != 0) r[2] = add_w<-CY * w>(r[2], u);
    if constexpr (CZ != 0) r[3] = add_w<-CZ * w>(r[3], u);
}

template <int Q, int CY, int CZ, typename Pick>
__device__ __forceinline__ void wall_group(const Src& s, float f, float g, const Pick& pick, float (&r)[4]) {
    using G = Group<Q, CY, CZ>;
    level_z<CZ>(s, f, g);
    if constexpr (G::has0 && (CY != 0 || CZ != 0)) wall_dir<Q, 0, CY, CZ>(f, pick, r);
    if constexpr (G::hasx) {
        float fp, fm;
        level_x(s, f, g, fp, fm);
        wall_dir<Q, 1, CY, CZ>(fp, pick, r);
        wall_dir<Q, -1, CY, CZ>(fm, pick, r);
    }
}

template <int Q, int CY, typename Pick>
__device__ __forceinline__ void wall_row(const Src& s, const Pick& pick, float (&r)[4]) {
    float f, g;
    level_y<CY>(s, f, g);
    wall_group<Q, CY, 0>(s, f, g, pick, r);
    wall_group<Q, CY, 1>(s, f, g, pick, r);
    wall_group<Q, CY, -1>(s, f, g, pick, r);
}

template <int Q, typename Pick>
__device__ __forceinline__ void wall_sums(const Src& s, const Pick& pick, float (&r)[4]) {
    r[0] = r[1] = r[2] = r[3] = 0.0f;
    wall_row<Q, 0>(s, pick, r);
    wall_row<Q, 1>(s, pick, r);
    wall_row<Q, -1>(s, pick, r);
    r[0] -= r[3];
}

// New state of one node from its sums (file header): v = j / rho + g, with one
// correctly rounded division.  The unit as a float is too large by 7.5e-9 of its
// size, the same way in every step, which a flow of hundreds of steps would
// collect: density and velocity take the difference back.
template <int Q>
__device__ __forceinline__ void finish_node(float t, float c, float m, float jx, float jy, float gx,
                                            float gy, float gz, float& d, float& vx, float& vy,
                                            float& vz) {
    constexpr float unit = weight_unit<Q>();
    constexpr float off = (float)(1.0 / Lattice<Q>::units - (double)unit);
    const float tm = t + m, jz = t - m;
    d = __builtin_fmaf(unit, tm, __builtin_fmaf(unit, c, off * (tm + c)));
    const float r = unit / (1.0f + d);
    vx = __builtin_fmaf(jx, r, __builtin_fmaf(jx, off, gx));
    vy = __builtin_fmaf(jy, r, __builtin_fmaf(jy, off, gy));
    vz = __builtin_fmaf(jz, r, __builtin_fmaf(jz, off, gz));
}

}  // namespace tau1
