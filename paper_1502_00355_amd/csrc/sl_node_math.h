// Per-node arithmetic of the kernels that take one free node at a time (the
// node, lane-group, resident, class-tile and flow kernels): the two
// qualities of an incident triangle, the centroid's division and the
// minimum over a lane group.
#pragma once

#include <type_traits>

#include "sl_common.h"

namespace sl {

namespace {

// 2*sqrt(3) rounded to double: q = 4*sqrt(3)*A / sum(l^2) = (2*sqrt(3)*cr) / S.
constexpr double kTwoSqrt3 = 0x1.bb67ae8584caap+1;

// Old and new quality of the triangle whose stored order puts the node at
// position p, the vertex `a` at p+1 and `b` at p+2 (mod 3): the node at o,
// then at its candidate c.  With u = a - node, v = b - node and w = b - a,
// the stored order's edge vectors p1 - p0, p2 - p0, p2 - p1 are (u, v, w)
// for p = 0, (-v, -w, u) for p = 1 and (w, -u, -v) for p = 2.  A negation
// is exact and fl(y - x) = -fl(x - y), so the cross product is
// P.x Q.y - Q.x P.y with (P, Q) = (u, v), (v, w) or (u, w), and the sum of
// squared lengths (|p1-p0|^2 + |p2-p1|^2) + |p2-p0|^2 is (Lu + Lw) + Lv,
// (Lv + Lu) + Lw or (Lw + Lv) + Lu: the same roundings as evaluating the
// stored order directly, every operation one rounded double operation
// without contraction.  w and its length are shared by the
// two evaluations, and selects pick operands instead of rebuilding the
// order (the lanes of a wave hold different p: a branch per p made a wave
// run all three orders one after the other).
__device__ __forceinline__ void fan_qualities(int p, const double2 o, const double2 c, const double2 a,
                                              const double2 b, double& qold, double& qnew)
{
    const double wx = b.x - a.x, wy = b.y - a.y;
    const double Lw = wx * wx + wy * wy;
    auto one = [&](double px, double py) {
        const double ux = a.x - px, uy = a.y - py, vx = b.x - px, vy = b.y - py;
        const double Lu = ux * ux + uy * uy, Lv = vx * vx + vy * vy;
        const double Px = p == 1 ? vx : ux, Py = p == 1 ? vy : uy;
        const double Qx = p == 0 ? vx : wx, Qy = p == 0 ? vy : wy;
        const double X = p == 2 ? Lv : Lu, Y = p == 1 ? Lv : Lw, Z = p == 0 ? Lv : (p == 1 ? Lw : Lu);
        const double cr = Px * Qy - Qx * Py;
        const double S = (X + Y) + Z;
        const double q = (kTwoSqrt3 * cr) / S;
        return S == 0.0 ? 0.0 : q;
    };
    qold = one(o.x, o.y);
    qnew = one(c.x, c.y);
}

// The same for a stored position P known at compile time (the colour-class
// tiles list each node's fan entries grouped by position): no selects.
template <int P>
__device__ __forceinline__ void fan_qualities_p(const double2 o, const double2 c, const double2 a, const double2 b,
                                                double& qold, double& qnew)
{
    const double wx = b.x - a.x, wy = b.y - a.y;
    const double Lw = wx * wx + wy * wy;
    auto one = [&](double px, double py) {
        const double ux = a.x - px, uy = a.y - py, vx = b.x - px, vy = b.y - py;
        const double Lu = ux * ux + uy * uy, Lv = vx * vx + vy * vy;
        double cr, S;
        if (P == 0) {
            cr = ux * vy - vx * uy;
            S = (Lu + Lw) + Lv;
        } else if (P == 1) {
            cr = vx * wy - wx * vy;
            S = (Lu + Lv) + Lw;
        } else {
            cr = ux * wy - wx * uy;
            S = (Lv + Lw) + Lu;
        }
        const double q = (kTwoSqrt3 * cr) / S;
        return S == 0.0 ? 0.0 : q;
    };
    qold = one(o.x, o.y);
    qnew = one(c.x, c.y);
}

// a / d correctly rounded for an integer count d in [1, 127] with y = 1/d
// correctly rounded, while the quotient is a normal number (Markstein's
// correction step: q = a*y is within an ulp, the remainder a - q*d is
// exact, and a normal quotient by an integer below 2^7 lies at least
// ulp/254 from a rounding midpoint).  Callers divide instead when |a| is
// below 128 x the smallest normal.
__device__ __forceinline__ double div_small(double a, double d, double y)
{
    const double q = a * y;
    const double r = fma(-q, d, a);
    return fma(r, y, q);
}
constexpr double kStepMin = 0x1p-1015;   // 128 x the smallest normal double

// The minimum over the W lanes of each group (a group's lanes are active
// together): swaps of neighbouring lanes and of lane pairs inside each quad,
// then the mirror inside each half row (8 lanes) and each row (16 lanes).
template <int W>
__device__ __forceinline__ double group_min(double v)
{
    auto fold = [&v](auto ctrl) {
        constexpr int c = decltype(ctrl)::value;
        const long long b = __double_as_longlong(v);
        const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(b), c, 0xF, 0xF, false);
        const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(b >> 32), c, 0xF, 0xF, false);
        const double t = __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<uint32_t>(lo));
        v = t < v ? t : v;
    };
    if (W >= 2) fold(std::integral_constant<int, 0xB1>{});       // quad_perm [1,0,3,2]
    if (W >= 4) fold(std::integral_constant<int, 0x4E>{});       // quad_perm [2,3,0,1]
    if (W >= 8) fold(std::integral_constant<int, 0x141>{});      // row_half_mirror
    if (W >= 16) fold(std::integral_constant<int, 0x140>{});     // row_mirror
    return v;
}

}  // namespace

}  // namespace sl
