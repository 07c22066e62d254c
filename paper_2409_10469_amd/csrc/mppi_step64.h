// The FP64 dynamics step's leg: kinematics, mass-matrix and bias terms, foot contact and
// the terms they add to the trunk's rows, for the lane-split and the quad kernels.
//
// What bounds the FP64 step is the number of instructions a wave issues (one or two waves
// per SIMD, every value in registers), so the leg is written in the frame in which it has
// the fewest: the LEG FRAME, the trunk frame turned about x by the abduction angle with
// its origin at the hip.  There both links lie in the x-z plane, the flexion and knee axes
// are the unit vector y and the abduction axis is x, so cross products with an axis cost
// no arithmetic and about half of every product vanishes:
//   * composite inertia: xz-plane bodies have no xy and yz entries, and yy = xx + zz;
//   * the joint columns of the mass matrix hold 7 values instead of 18;
//   * a link is a uniform rod, whose inertia about its centre is that of two point masses,
//     so its inertial torque is d x (A d) with the same matrix A = [alpha x] + w w^T - |w|^2
//     that gives its centre's acceleration: no separate gyroscopic terms.
// Three 6-vectors (the joint rows), one wrench and 9 inertia values are then turned back
// into the trunk frame.  Divisions, square roots and the elementary functions are written
// out without branches (the device library's FP64 versions cost 2 to 4 times as many
// instructions); the results stay within about an ulp of the library's.
#pragma once
#include "mppi_device.h"

#ifndef __constant__
#define __constant__
#endif

namespace mppi {
namespace f64 {

// Coefficients of the series below.  Read from constant memory in every step, through a
// pointer that the compiler takes to depend on the step's number k, they arrive by a few
// scalar loads in scalar registers; as literals every one would be kept in two vector
// registers over the whole step loop, which costs the step more in register moves.  Each USE
// of the table loads for itself, so that its coefficients do not stay from one to the next.
enum { kSin = 0, kCos = 7, kRed = 14, kExp = 20 };
static __constant__ const double kTab[32] = {
    // sin: r^15 .. r^3
    -1.0 / 1307674368000.0, 1.0 / 6227020800.0, -1.0 / 39916800.0, 1.0 / 362880.0, -1.0 / 5040.0, 1.0 / 120.0, -1.0 / 6.0,
    // cos: r^16 .. r^4
    1.0 / 20922789888000.0, -1.0 / 87178291200.0, 1.0 / 479001600.0, -1.0 / 3628800.0, 1.0 / 40320.0, -1.0 / 720.0,
    1.0 / 24.0,
    // 2/pi, pi/2 in two parts; 1/ln 2, ln 2 in two parts
    0.63661977236758134308, 1.57079632679489655800, 6.12323399573676603587e-17, 1.44269504088896340736,
    0.69314718055994528623, 2.31904681384629955842e-17,
    // exp - 1: r^13 .. r^3
    1.0 / 6227020800.0, 1.0 / 479001600.0, 1.0 / 39916800.0, 1.0 / 3628800.0, 1.0 / 362880.0, 1.0 / 40320.0, 1.0 / 5040.0,
    1.0 / 720.0, 1.0 / 120.0, 1.0 / 24.0, 1.0 / 6.0, 0.0};
#if defined(__HIP_DEVICE_COMPILE__)
typedef const __attribute__((address_space(4))) double* TabPtr;
template <int USE>
__device__ __forceinline__ TabPtr fresh_table(int k)
{
    TabPtr p = (TabPtr)(&kTab[0]);
    asm("; %2" : "+s"(p) : "s"(k), "i"(USE));
    return p;
}
#else
typedef const double* TabPtr;
template <int USE>
__device__ __forceinline__ TabPtr fresh_table(int)
{
    return kTab;
}
#endif

// a x + c with the coefficient c in scalar registers (the compiler would move it to vector
// registers first to use the two-operand form)
__device__ __forceinline__ double horner(double a, double x, double c)
{
#if defined(__HIP_DEVICE_COMPILE__)
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(x), "s"(c));
    return d;
#else
    return fma(a, x, c);
#endif
}

// ------------------------------------------------------------------------------
// elementary functions
// ------------------------------------------------------------------------------
// 1/sqrt(x) and 1/x from the hardware's estimates (relative error below 2^-22) and one
// third-order step, which leaves the rounding of its own operations (about 1 ulp)
__device__ __forceinline__ double rsq(double x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const double y = __builtin_amdgcn_rsq(x);
#else
    const double y = 1.0 / sqrt(x);
#endif
    const double e = fma(-(x * y), y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}
__device__ __forceinline__ double rcp(double x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const double y = __builtin_amdgcn_rcp(x);
#else
    const double y = 1.0 / x;
#endif
    const double e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}
// sqrt of x >= 0, and 1/sqrt with 0 -> a large finite value
__device__ __forceinline__ double rsq_pos(double x) { return rsq(m_max(x, 1e-300)); }

// |x| from 2^40, the end of sincos64's range, up to the largest finite value, by its leading bits
// (as numbers in a table the bounds would be a wait for memory at the head of a step; and a state
// that is not finite, which stays so, takes no rare path)
__device__ __forceinline__ bool is_far(double x)
{
    constexpr unsigned lo = 0x42700000u, inf = 0x7ff00000u;
    return ((unsigned)__double2hiint(x) & 0x7fffffffu) - lo < inf - lo;
}

// An angle of the same sine and cosine as x, within 4, for an x beyond the range of sincos64:
// x 2/pi mod 4 from 159 bits of 2/pi, which the hardware looks up by x's exponent in
// segments of 53 (the bits before the first segment add multiples of 4), its products with x in
// two parts each.  Holds for any angle that an FP32 state and time step give (below 2^945, where
// the segments are scaled).
__device__ __forceinline__ double near_angle(TabPtr t, double x)
{
#pragma clang fp contract(off)
#if defined(__HIP_DEVICE_COMPILE__)
    const double p0 = __builtin_amdgcn_trig_preop(x, 0), p1 = __builtin_amdgcn_trig_preop(x, 1);
    const double h0 = x * p0, l0 = fma(x, p0, -h0), h1 = x * p1, l1 = fma(x, p1, -h1);
    const double a = fma(-4.0, rint(ldexp(h0, -2)), h0);
    const double s = l0 + h1, v = s - l0, e = ((l0 - (s - v)) + (h1 - v)) + (l1 + x * __builtin_amdgcn_trig_preop(x, 2));
    // quadrant k, the rest f + g of a quarter turn
    const double k = rint(a + s), n = a - k, f = n + s, u = f - n, g = ((n - (f - u)) + (s - u)) + e;
    const double r = fma(f, t[kRed + 1], fma(f, t[kRed + 2], g * t[kRed + 1]));
    return fma(fma(-4.0, rint(ldexp(k, -2)), k), t[kRed + 1], r);
#else
    return atan2(sin(x), cos(x));
#endif
}

// sine and cosine: x = k pi/2 + r with pi/2 in two parts (k pi/2's leading part leaves the
// fused multiply-add exact before its rounding), then the Taylor series on |r| <= pi/4 up
// to r^15 and r^16 (truncation below 6e-17 relative) and the quadrant's swap and signs.
// Good to |x| = 2^40; beyond it the rounded quotient misses its integer, r leaves the series'
// range, and the caller passes near_angle(x): by one test for all the angles of a step, where
// the code branches anyway (a test in each evaluation: 1-2% of a step).
__device__ __forceinline__ void sincos64(TabPtr t, double x, double* sn, double* cs)
{
    const double k = rint(x * t[kRed]);
    double r = fma(-k, t[kRed + 1], x);
    r = fma(-k, t[kRed + 2], r);
    const double z = r * r;
    double sp = fma(z, t[kSin], t[kSin + 1]), cp = fma(z, t[kCos], t[kCos + 1]);
#pragma unroll
    for (int i = 2; i < 7; ++i) {
        sp = horner(z, sp, t[kSin + i]);
        cp = horner(z, cp, t[kCos + i]);
    }
    sp = fma(r * z, sp, r);
    cp = fma(z, cp, -0.5);
    cp = fma(z, cp, 1.0);
    const int q = int(fma(-4.0, m_floor(0.25 * k), k));  // k mod 4
    const double s0 = (q & 1) ? cp : sp, c0 = (q & 1) ? sp : cp;
    *sn = (q & 2) ? -s0 : s0;
    *cs = ((q + 1) & 2) ? -c0 : c0;
}

// tanh(s) / s for s >= 0 through e = exp(-2s) - 1: -2s = k ln 2 + r, exp(r) - 1 by its
// Taylor series up to r^13 on |r| <= 0.35 (truncation below 1e-17), e = 2^k (exp(r) - 1) +
// (2^k - 1), which keeps its relative accuracy at small s (k = 0), tanh(s) = -e / (2 + e).
// Beyond s = 350 exp(-2s) is zero next to 1.
__device__ __forceinline__ double tanh_ratio64(TabPtr t, double s)
{
    const double x = -2.0 * m_min(s, 350.0);
    const double k = rint(x * t[kRed + 3]);
    double r = fma(-k, t[kRed + 4], x);
    r = fma(-k, t[kRed + 5], r);
    double p = fma(r, t[kExp], t[kExp + 1]);
#pragma unroll
    for (int i = 2; i < 11; ++i) p = horner(r, p, t[kExp + i]);
    p = fma(r, p, 0.5);
    p = fma(r * r, p, r);
    const double p2 = ldexp(1.0, int(k));
    const double e = fma(p2, p, p2 - 1.0);
    const double den = (2.0 + e) * s, y = rcp(den);
    const double q = -e * y;
    const double v = fma(fma(-q, den, -e), y, q);
    return s < 1e-8 ? 1.0 : v;
}

// quaternion update q <- normalize(q (x) exp(dt w / 2)): sin(a)/a and cos(a) of the half
// angle a by their Taylor series in a^2 while a <= 1/2 (up to a^12 and a^14, truncation
// below 5e-17: any |w| up to 1/dt), by sincos64 beyond (a rate that is not finite stays in the
// series, to the same end)
__device__ __forceinline__ void quat_step64(TabPtr t, double& qw, double& qx, double& qy, double& qz, V3<double> w,
                                            double dt)
{
    const V3<double> ph = (0.5 * dt) * w;
    const double z = dot(ph, ph);
    double sc = fma(z, t[kSin + 1], t[kSin + 2]), dw = fma(z, t[kCos + 1], t[kCos + 2]);
#pragma unroll
    for (int i = 3; i < 7; ++i) {
        sc = horner(z, sc, t[kSin + i]);
        dw = horner(z, dw, t[kCos + i]);
    }
    sc = fma(z, sc, 1.0);
    dw = fma(z, dw, -0.5);
    dw = fma(z, dw, 1.0);
    if (z > 0.25) {
        const double a = sqrt(z);
        double s;
        sincos64(t, is_far(a) ? near_angle(t, a) : a, &s, &dw);
        sc = s / a;
    }
    const double dx = sc * ph.x, dy = sc * ph.y, dz = sc * ph.z;
    const double nw = qw * dw - qx * dx - qy * dy - qz * dz;
    const double nx = qw * dx + qx * dw + qy * dz - qz * dy;
    const double ny = qw * dy - qx * dz + qy * dw + qz * dx;
    const double nz = qw * dz + qx * dy - qy * dx + qz * dw;
    const double inv = rsq(nw * nw + nx * nx + ny * ny + nz * nz);
    qw = nw * inv; qx = nx * inv; qy = ny * inv; qz = nz * inv;
}

// the penalty law of contact_law in FP64
template <typename MD>
__device__ __forceinline__ void contact_law64(TabPtr t, const MD& M, double delta, V3<double> n,
                                              V3<double> vrel, V3<double>& F, double& eta)
{
    const double vn = dot(n, vrel);
    const double Fn = M.ck * delta - M.cc * vn;
    const V3<double> vt = vrel - vn * n;
    const double v2 = dot(vt, vt);
    const double s = v2 * rsq_pos(v2) * M.inv_vs;
    eta = M.cmu * m_max(Fn, 0.0) * M.inv_vs * tanh_ratio64(t, s);
    F = Fn * n - eta * vt;
}

// terrain below a sphere (r > 0) or point (r = 0), as terrain<> of the device header
template <int SCENE, typename MD>
__device__ __forceinline__ bool terrain64(const MD& M, const float* __restrict__ hf, V3<double> c,
                                          double r, double& delta, V3<double>& n)
{
    if constexpr (SCENE != 1) {
        n = v3(0.0, 0.0, 1.0);
        delta = r - c.z;
        return delta > 0.0;
    } else {
        const int nx = M.hf_nx, ny = M.hf_ny;
        const double ux = (c.x - M.hf_x0) * M.hf_inv_cell, uy = (c.y - M.hf_y0) * M.hf_inv_cell;
        const double fx = m_min(m_max(ux, 0.0), double(nx - 1)), fy = m_min(m_max(uy, 0.0), double(ny - 1));
        int i0 = (int)m_floor(fx), j0 = (int)m_floor(fy);
        i0 = max(0, min(i0, nx - 2));
        j0 = max(0, min(j0, ny - 2));
        const double tx = fx - double(i0), ty = fy - double(j0);
        const double h00 = hf[j0 * nx + i0], h10 = hf[j0 * nx + i0 + 1];
        const double h01 = hf[(j0 + 1) * nx + i0], h11 = hf[(j0 + 1) * nx + i0 + 1];
        const double dx0 = h10 - h00, dx1 = h11 - h01, dy0 = h01 - h00;
        const double dxy = dx1 - dx0;
        const double h = h00 + tx * dx0 + ty * (dy0 + tx * dxy);
        // outside the grid the height is held, so its slope across the edge is zero; NaN
        // coordinates keep a zero slope as well
        const double gx = (fx == ux) ? (dx0 + ty * dxy) * M.hf_inv_cell : 0.0;
        const double gy = (fy == uy) ? (dy0 + tx * dxy) * M.hf_inv_cell : 0.0;
        const double inv = rsq(gx * gx + gy * gy + 1.0);
        n = v3(-gx * inv, -gy * inv, inv);
        delta = (h + r - c.z) * n.z;
        return delta > 0.0;
    }
}

// sphere against an axis-aligned box, as sphere_aabox of the device header
__device__ __forceinline__ bool sphere_aabox64(V3<double> l, double r, V3<double> bh, double& delta, V3<double>& n)
{
    const V3<double> q = v3(m_min(m_max(l.x, -bh.x), bh.x), m_min(m_max(l.y, -bh.y), bh.y),
                            m_min(m_max(l.z, -bh.z), bh.z));
    const V3<double> e = l - q;
    const double d2 = dot(e, e);
    const bool inside = m_abs(l.x) <= bh.x && m_abs(l.y) <= bh.y && m_abs(l.z) <= bh.z;
    if (!inside && !(d2 < r * r)) return false;
    const double id = rsq_pos(d2);
    const double dx = bh.x - m_abs(l.x), dy = bh.y - m_abs(l.y), dz = bh.z - m_abs(l.z);
    double depth = dx;
    V3<double> nf = v3(l.x >= 0.0 ? 1.0 : -1.0, 0.0, 0.0);
    if (dy < depth) { depth = dy; nf = v3(0.0, l.y >= 0.0 ? 1.0 : -1.0, 0.0); }
    if (dz < depth) { depth = dz; nf = v3(0.0, 0.0, l.z >= 0.0 ? 1.0 : -1.0); }
    delta = inside ? r + depth : r - d2 * id;
    n = inside ? nf : id * e;
    return true;
}

// ------------------------------------------------------------------------------
// 6x6 system: L D L^T of the packed upper triangle, solving Q x = r in place (Q is
// overwritten).  Reciprocals of the pivots instead of square roots.
// ------------------------------------------------------------------------------
// the pivots' sign bits, gathered, and v or, where one was set, NaN: a system that its rounding
// (a diverged sample) has made indefinite has no result, as with the square roots of a Cholesky
// factorisation (a pivot of 0 gives NaN by its reciprocal)
__device__ __forceinline__ int sign_of(double pivot) { return __double2hiint(pivot); }
__device__ __forceinline__ double nan_if(int signs, double v)
{
    return __hiloint2double(__double2hiint(v) | (signs >> 31), __double2loint(v));
}

__device__ __forceinline__ void ldl6_solve(double* Q, double* r)
{
    double inv[6];
    int signs = 0;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        inv[j] = rcp(Q[s6(j, j)]);
        signs |= sign_of(Q[s6(j, j)]);
        double l[6];
#pragma unroll
        for (int i = j + 1; i < 6; ++i) l[i] = Q[s6(j, i)] * inv[j];
#pragma unroll
        for (int i = j + 1; i < 6; ++i) {
#pragma unroll
            for (int k = i; k < 6; ++k) Q[s6(i, k)] -= l[i] * Q[s6(j, k)];
            r[i] -= l[i] * r[j];
        }
#pragma unroll
        for (int i = j + 1; i < 6; ++i) Q[s6(j, i)] = l[i];
    }
#pragma unroll
    for (int i = 5; i >= 0; --i) {
        double s = r[i] * inv[i];
        if (i == 5) s = nan_if(signs, s);
#pragma unroll
        for (int k = i + 1; k < 6; ++k) s -= Q[s6(i, k)] * r[k];
        r[i] = s;
    }
}

// 3x3 symmetric system, factored once and solved for several right sides
struct Ldl3 {
    double l10, l20, l21, i0, i1, i2;
};
__device__ __forceinline__ Ldl3 ldl3(double a00, double a10, double a11, double a20, double a21, double a22)
{
    Ldl3 f;
    f.i0 = rcp(a00);
    f.l10 = a10 * f.i0;
    f.l20 = a20 * f.i0;
    const double d1 = a11 - f.l10 * a10;
    f.i1 = rcp(d1);
    const double t = a21 - f.l20 * a10;
    f.l21 = t * f.i1;
    const double d2 = a22 - f.l20 * a20 - f.l21 * t;
    f.i2 = nan_if(sign_of(a00) | sign_of(d1) | sign_of(d2), rcp(d2));
    return f;
}
__device__ __forceinline__ void solve3(const Ldl3& f, double& b0, double& b1, double& b2)
{
    const double y1 = b1 - f.l10 * b0;
    const double y2 = b2 - f.l20 * b0 - f.l21 * y1;
    b2 = y2 * f.i2;
    b1 = y1 * f.i1 - f.l21 * b2;
    b0 = b0 * f.i0 - f.l10 * b1 - f.l20 * b2;
}

// ------------------------------------------------------------------------------
// the leg
// ------------------------------------------------------------------------------
struct LegFrame {
    double sa, ca;             // abduction
    double hx, hy;             // hip in the trunk frame (z = 0)
    double kx, kz, fx, fz;     // knee and foot in the leg frame (y = 0)
    V3<double> w1;             // angular velocity of the thigh, leg frame
    V3<double> vh;             // velocity of the hip, leg frame
    double dk;                 // knee rate
};
__device__ __forceinline__ V3<double> to_leg(const LegFrame& G, V3<double> v)
{
    return v3(v.x, G.ca * v.y + G.sa * v.z, G.ca * v.z - G.sa * v.y);
}
__device__ __forceinline__ V3<double> to_trunk(const LegFrame& G, V3<double> v)
{
    return v3(v.x, G.ca * v.y - G.sa * v.z, G.sa * v.y + G.ca * v.z);
}
// foot centre in the trunk frame
__device__ __forceinline__ V3<double> foot_trunk(const LegFrame& G)
{
    return v3(G.hx + G.fx, G.hy - G.sa * G.fz, G.ca * G.fz);
}

// the leg's rows of the implicit system: A (joints), C (joints x trunk: angular, linear,
// in the leg frame about the hip until rows_to_trunk), right side rl
struct LegRows {
    double A00, A01, A02, A11, A12, A22;
    V3<double> L[3], P[3];
    double rl[3];
};

// Mass-matrix, bias and joint-torque terms.  Q, rb receive the leg's share of the trunk
// rows (Q overwritten; the linear block and the hip offsets' own inertia, which are
// constant, are in the model's totals tr_I*).
template <typename MD>
__device__ __forceinline__ void leg_terms(const MD& M, int leg, double sa, double ca, double sf, double cf,
                                          double s12, double c12, const double* qd, const double* tau, double dt,
                                          double dtkd, V3<double> w, V3<double> vb, V3<double> gb, LegFrame& G,
                                          LegRows& S, double* Q, double* rb)
{
    const double hx = (leg < 2) ? M.hip_x : -M.hip_x, hy = (leg & 1) ? -M.hip_y : M.hip_y;
    G.sa = sa; G.ca = ca; G.hx = hx; G.hy = hy;
    const double kx = -M.l1 * sf, kz = -M.l1 * cf;
    const double rx = (-0.5 * M.l2) * s12, rz = (-0.5 * M.l2) * c12;  // calf centre from the knee
    const double cx = kx + rx, cz = kz + rz;                          // calf centre from the hip
    G.kx = kx; G.kz = kz;
    G.fx = cx + rx; G.fz = cz + rz;
    const double da = qd[0], df = qd[1], dk = qd[2];
    G.dk = dk;

    // hip: velocity and acceleration less gravity
    const V3<double> u = v3(-w.z * hy, w.z * hx, w.x * hy - w.y * hx);
    G.vh = to_leg(G, vb + u);
    const V3<double> a = to_leg(G, cross(w, u) - gb);
    const V3<double> wl = to_leg(G, w);
    const V3<double> w1 = v3(wl.x + da, wl.y + df, wl.z);
    G.w1 = w1;
    const V3<double> al1 = v3(-df * wl.z, da * wl.z, df * w1.x - da * wl.y);
    // columns x and z of [alpha x] + w w^T - |w|^2 for thigh (1) and calf (2)
    const double yy1 = w1.y * w1.y, xz1 = w1.x * w1.z;
    const V3<double> X1 = v3(-(w1.z * w1.z + yy1), w1.x * w1.y + al1.z, xz1 - al1.y);
    const V3<double> Z1 = v3(xz1 + al1.y, w1.y * w1.z - al1.x, -(w1.x * w1.x + yy1));
    const double w2y = w1.y + dk, a2x = al1.x - dk * w1.z, a2z = al1.z + dk * w1.x, yy2 = w2y * w2y;
    const V3<double> X2 = v3(-(w1.z * w1.z + yy2), w1.x * w2y + a2z, xz1 - al1.y);
    const V3<double> Z2 = v3(xz1 + al1.y, w2y * w1.z - a2x, -(w1.x * w1.x + yy2));
    const V3<double> E1 = kx * X1 + kz * Z1, E2 = rx * X2 + rz * Z2;
    // inertial forces: thigh F1, calf F2; G1, G2 carry the rods' own inertia as well
    const V3<double> m1a = M.m1 * a, ma = M.m2 * (a + E1);
    const V3<double> F1 = m1a + (0.5 * M.m1) * E1, G1 = 0.5 * m1a + M.leg_a1 * E1;
    const V3<double> F2 = ma + M.m2 * E2, G2 = ma + M.leg_a2 * E2;
    const V3<double> Fs = G1 + F2;
    const V3<double> Tk = v3(-rz * G2.y, rz * G2.x - rx * G2.z, rx * G2.y);
    const V3<double> Th = v3(Tk.x - kz * Fs.y, Tk.y + kz * Fs.x - kx * Fs.z, Tk.z + kx * Fs.y);
    S.rl[0] = dt * (tau[0] - Th.x);
    S.rl[1] = dt * (tau[1] - Th.y);
    S.rl[2] = dt * (tau[2] - Tk.y);
    {
        const V3<double> F = to_trunk(G, F1 + F2), T = to_trunk(G, Th);
        rb[0] = -dt * (T.x + hy * F.z);
        rb[1] = -dt * (T.y - hx * F.z);
        rb[2] = -dt * (T.z + hx * F.y - hy * F.x);
        rb[3] = -dt * F.x; rb[4] = -dt * F.y; rb[5] = -dt * F.z;
    }

    // composite inertia and first moment about the hip, leg frame
    const double k1c = M.leg_k1e * cf, k1s = M.leg_k1e * sf, k2c = M.k2 * c12, k2s = M.k2 * s12;
    const double mcx = M.m2 * cx, mcz = M.m2 * cz;
    const double xx = k1c * cf + k2c * c12 + mcz * cz;
    const double zz = k1s * sf + k2s * s12 + mcx * cx;
    const double xz = -(k1s * cf + k2s * c12 + mcx * cz);
    const double yy = xx + zz;
    const double lx = 0.5 * M.m1 * kx + mcx, lz = 0.5 * M.m1 * kz + mcz;
    const double bx = M.m2 * rx, bz = M.m2 * rz, Lk = M.k2 + cx * bx + cz * bz;
    S.L[0] = v3(xx, 0.0, xz);
    S.P[0] = v3(0.0, -lz, 0.0);
    S.L[1] = v3(0.0, yy, 0.0);
    S.P[1] = v3(lz, 0.0, -lx);
    S.L[2] = v3(0.0, Lk, 0.0);
    S.P[2] = v3(bz, 0.0, -bx);
    S.A00 = xx + dtkd; S.A01 = 0.0; S.A02 = 0.0;
    S.A11 = yy + dtkd; S.A12 = Lk; S.A22 = M.leg_kk + dtkd;

    // the trunk's rows: turned, then moved from the hip to the trunk's centre
    const double s2 = sa * sa, c2 = ca * ca;
    const double ly = -sa * lz, l2 = ca * lz;
    const double hl = hx * lx, hm = hy * ly;
    Q[s6(0, 0)] = xx + 2.0 * hm;
    Q[s6(0, 1)] = -sa * xz - (hx * ly + hy * lx);
    Q[s6(0, 2)] = ca * xz - hx * l2;
    Q[s6(1, 1)] = c2 * yy + s2 * zz + 2.0 * hl;
    Q[s6(1, 2)] = (ca * sa) * (yy - zz) - hy * l2;
    Q[s6(2, 2)] = s2 * yy + c2 * zz + 2.0 * (hl + hm);
    Q[s6(0, 3)] = 0.0; Q[s6(0, 4)] = -l2; Q[s6(0, 5)] = ly;
    Q[s6(1, 3)] = l2;  Q[s6(1, 4)] = 0.0; Q[s6(1, 5)] = -lx;
    Q[s6(2, 3)] = -ly; Q[s6(2, 4)] = lx;  Q[s6(2, 5)] = 0.0;
#pragma unroll
    for (int i = 15; i < 21; ++i) Q[i] = 0.0;
}

// A contact on the foot with weight wgt (1: applied, 0: nothing added): nt the normal
// toward the robot and vo the other body's velocity, both in the trunk frame.  Adds the
// terms of the joint rows and of the trunk's rows; returns force (trunk frame) and secant.
template <typename MD>
__device__ __forceinline__ void foot_contact(TabPtr t, const MD& M, const LegFrame& G, double delta,
                                             V3<double> nt, V3<double> vo, double dt, double wgt, LegRows& S, double* Q, double* rb,
                                             V3<double>& Ft, double& eta)
{
    const V3<double> n = to_leg(G, nt);
    const V3<double> r = v3(G.fx - M.foot_r * n.x, -M.foot_r * n.y, G.fz - M.foot_r * n.z);
    const double px = r.x - G.kx, pz = r.z - G.kz;
    const V3<double> vl = G.vh - to_leg(G, vo) + cross(G.w1, r);
    V3<double> F;
    contact_law64(t, M, delta, n, v3(vl.x + G.dk * pz, vl.y, vl.z - G.dk * px), F, eta);
    F = wgt * F;
    eta = wgt * eta;
    const double c = wgt * M.cc;
    const double de = dt * eta, dce = dt * (c - eta);
    Ft = to_trunk(G, F);
    base_contact_folded(eta, c, foot_trunk(G) - M.foot_r * nt, nt, Ft, dt, Q, rb);
    // the joints' columns at the contact: abduction (0, -rz, ry), flexion (rz, 0, -rx),
    // knee (pz, 0, -px); D j = de j + dce (j . n) n
    const double gA = r.y * n.z - r.z * n.y, gF = r.z * n.x - r.x * n.z, gK = pz * n.x - px * n.z;
    const double ex = de * r.x, ey = de * r.y, ez = de * r.z, fx = de * px, fz = de * pz;
    const double hA = dce * gA, hF = dce * gF, hK = dce * gK;
    const V3<double> DA = v3(hA * n.x, hA * n.y - ez, hA * n.z + ey);
    const V3<double> DF = v3(hF * n.x + ez, hF * n.y, hF * n.z - ex);
    const V3<double> DK = v3(hK * n.x + fz, hK * n.y, hK * n.z - fx);
    S.A00 += r.y * DA.z - r.z * DA.y;
    S.A01 += r.z * DA.x - r.x * DA.z;
    S.A02 += pz * DA.x - px * DA.z;
    S.A11 += r.z * DF.x - r.x * DF.z;
    S.A12 += pz * DF.x - px * DF.z;
    S.A22 += pz * DK.x - px * DK.z;
    S.rl[0] += dt * (r.y * F.z - r.z * F.y);
    S.rl[1] += dt * (r.z * F.x - r.x * F.z);
    S.rl[2] += dt * (pz * F.x - px * F.z);
    S.L[0] = S.L[0] + cross(r, DA); S.P[0] = S.P[0] + DA;
    S.L[1] = S.L[1] + cross(r, DF); S.P[1] = S.P[1] + DF;
    S.L[2] = S.L[2] + cross(r, DK); S.P[2] = S.P[2] + DK;
}

// the joint rows over the trunk's six velocities, trunk frame about its centre
__device__ __forceinline__ void rows_to_trunk(const LegFrame& G, const LegRows& S, double C[3][6])
{
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const V3<double> P = to_trunk(G, S.P[j]), L = to_trunk(G, S.L[j]);
        C[j][0] = L.x + G.hy * P.z;
        C[j][1] = L.y - G.hx * P.z;
        C[j][2] = L.z + G.hx * P.y - G.hy * P.x;
        C[j][3] = P.x; C[j][4] = P.y; C[j][5] = P.z;
    }
}

// ------------------------------------------------------------------------------
// the step of one sample on a quad of lanes (this lane owns leg `leg`), as quad_step: same
// contacts and discretisation.  M: the model in constant memory (ConstModel), read in every
// step k where it is used.  With the chip full (batched serving) the time is the instruction
// count and the waves a SIMD holds: the step is arranged so that few values live long (two
// waves per SIMD need 256 registers), robot first, then the box, with the contacts that are
// rare (trunk corners, the box against the robot) in blocks entered only where a lane of the
// wave has one.
// ------------------------------------------------------------------------------
#if defined(__HIP_DEVICE_COMPILE__)
typedef const __attribute__((address_space(4))) ModelT<double> ConstModel;
__device__ __forceinline__ ConstModel& fresh_const_model(ConstModel* m, int k)
{
    asm("" : "+s"(m) : "s"(k));
    return *m;
}
#else
typedef const ModelT<double> ConstModel;
__device__ __forceinline__ ConstModel& fresh_const_model(ConstModel* m, int) { return *m; }
#endif

template <int SCENE>
__device__ __forceinline__ void quad_step64(int k, ConstModel& M, const float* __restrict__ hf, double dt, double kp,
                                            double kd, int leg, Base<double>& b, Leg<double>& lg, BoxS<double>& bx,
                                            const double u[3], double& tau2)
{
    double tau[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) tau[j] = kp * (u[j] - lg.q[j]) - kd * lg.qd[j];

    const M33<double> Rm = quat_R(b.qw, b.qx, b.qy, b.qz);
    const V3<double> w = b.w, zero = v3(0.0, 0.0, 0.0), up = v3(0.0, 0.0, 1.0);
    const V3<double> vb = mulT(Rm, b.vw);
    [[maybe_unused]] M33<double> Rb;
    [[maybe_unused]] V3<double> bh, th;
    [[maybe_unused]] bool near_box = false;  // the trunk's and the box's bounding spheres can overlap
    if constexpr (SCENE == 3) {
        Rb = quat_R(bx.qw, bx.qx, bx.qy, bx.qz);
        bh = v3<double>(M.bx_hx, M.bx_hy, M.bx_hz);
        th = v3<double>(0.5 * M.tsx, 0.5 * M.tsy, 0.5 * M.tsz);
        const V3<double> dc = b.p - bx.p;
        near_box = dot(dc, dc) <= 2.001 * (dot(th, th) + dot(bh, bh));
    }
    [[maybe_unused]] auto box_vel = [&](V3<double> x) { return bx.vw + mul(Rb, cross(bx.w, mulT(Rb, x - bx.p))); };

    double Q[21], rb[6], W[3][6], y0, y1, y2;
    V3<double> F;
    double eta;
    // the foot's contact with the box, for the box's system below
    [[maybe_unused]] V3<double> fb_x = zero, fb_n = up, fb_F = zero;
    [[maybe_unused]] double fb_eta = 0.0, fb_c = 0.0;
    [[maybe_unused]] bool fb = false;
    {
        LegFrame G;
        LegRows S;
        {
            const V3<double> gb = (-M.g) * v3(Rm.m[6], Rm.m[7], Rm.m[8]);
            double sa, ca, sf, cf, s12, c12;
            const TabPtr t = fresh_table<0>(k);
            double qa = lg.q[0], qf = lg.q[1], q12 = lg.q[1] + lg.q[2];
            if (__builtin_amdgcn_ballot_w64(is_far(qa) | is_far(qf) | is_far(q12))) {  // a scalar branch
                if (is_far(qa)) qa = near_angle(t, qa);
                if (is_far(qf)) qf = near_angle(t, qf);
                if (is_far(q12)) q12 = near_angle(t, q12);
            }
            sincos64(t, qa, &sa, &ca);
            sincos64(t, qf, &sf, &cf);
            sincos64(t, q12, &s12, &c12);
            leg_terms(M, leg, sa, ca, sf, cf, s12, c12, lg.qd, tau, dt, dt * kd, w, vb, gb, G, S, Q, rb);
        }
        const V3<double> pfw = b.p + mul(Rm, foot_trunk(G));
        double dT, dB = 0.0;
        V3<double> nT, nB = zero;
        const bool hitT = terrain64<SCENE>(M, hf, pfw, M.foot_r, dT, nT);
        bool hitB = false;
        if constexpr (SCENE == 2)
            hitB = sphere_aabox64(pfw - v3<double>(M.sb_cx, M.sb_cy, M.sb_cz), M.foot_r,
                                  v3<double>(M.sb_hx, M.sb_hy, M.sb_hz), dB, nB);
        if constexpr (SCENE == 3) {
            // outside the sphere around the box there is no contact ((r + |h|)^2 <= 2 (r^2 + |h|^2),
            // with a margin for the rounding)
            const V3<double> d = pfw - bx.p;
            if (dot(d, d) <= 2.001 * (M.foot_r * M.foot_r + dot(bh, bh))) {
                V3<double> nl = up;
                hitB = sphere_aabox64(mulT(Rb, d), M.foot_r, bh, dB, nl);
                nB = mul(Rb, nl);  // box -> foot (world)
            }
        }
        // first contact: terrain if touched, else the box
        const bool on = hitT || hitB, isB = !hitT && hitB;
        if (on) {
            V3<double> n, vo = zero;
            if constexpr (SCENE == 0) {
                n = v3(Rm.m[6], Rm.m[7], Rm.m[8]);
            } else {
                const V3<double> nw = selv(isB, nB, nT);
                if constexpr (SCENE == 3) {
                    if (isB) vo = mulT(Rm, box_vel(pfw - M.foot_r * nw));
                }
                n = mulT(Rm, nw);
            }
            foot_contact(fresh_table<1>(k), M, G, isB ? dB : dT, n, vo, dt, 1.0, S, Q, rb, F, eta);
        }
        if constexpr (SCENE == 2 || SCENE == 3) {
            if (hitT && hitB) {
                V3<double> vo = zero;
                if constexpr (SCENE == 3) vo = mulT(Rm, box_vel(pfw - M.foot_r * nB));
                foot_contact(fresh_table<4>(k), M, G, dB, mulT(Rm, nB), vo, dt, 1.0, S, Q, rb, F, eta);
            }
            if constexpr (SCENE == 3) {
                if (hitB) {
                    fb = true;
                    fb_x = pfw - M.foot_r * nB;
                    fb_n = nB;
                    fb_F = -1.0 * mul(Rm, F);
                    fb_eta = eta;
                    fb_c = M.cc;
                }
            }
        }
        // eliminate the leg
        double C[3][6];
        rows_to_trunk(G, S, C);
        const Ldl3 f3 = ldl3(S.A00, S.A01, S.A11, S.A02, S.A12, S.A22);
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            double x0 = C[0][i], x1 = C[1][i], x2 = C[2][i];
            f64::solve3(f3, x0, x1, x2);
            W[0][i] = x0; W[1][i] = x1; W[2][i] = x2;
#pragma unroll
            for (int j = 0; j <= i; ++j) Q[s6(j, i)] -= C[0][j] * x0 + C[1][j] * x1 + C[2][j] * x2;
        }
        y0 = S.rl[0]; y1 = S.rl[1]; y2 = S.rl[2];
        f64::solve3(f3, y0, y1, y2);
#pragma unroll
        for (int i = 0; i < 6; ++i) rb[i] -= C[0][i] * y0 + C[1][i] * y1 + C[2][i] * y2;
    }
    // ---- two trunk corners per lane against terrain, static box and free box, and two box
    // corners against the trunk (its side of the contact)
#pragma unroll 1
    for (int cc = 0; cc < 2; ++cc) {
        const int ci = 2 * leg + cc;
        const V3<double> r = v3((ci & 1 ? 0.5 : -0.5) * M.tsx, (ci & 2 ? 0.5 : -0.5) * M.tsy,
                                (ci & 4 ? 0.5 : -0.5) * M.tsz);
        const V3<double> pw = b.p + mul(Rm, r);
        double delta;
        V3<double> nw;
        if (terrain64<SCENE>(M, hf, pw, 0.0, delta, nw)) {
            const V3<double> n = mulT(Rm, nw);
            contact_law64(fresh_table<3>(k), M, delta, n, vb + cross(w, r), F, eta);
            base_contact_folded(eta, M.cc, r, n, F, dt, Q, rb);
        }
        if constexpr (SCENE == 2) {
            if (point_aabox(pw - v3<double>(M.sb_cx, M.sb_cy, M.sb_cz), v3<double>(M.sb_hx, M.sb_hy, M.sb_hz), delta,
                            nw)) {
                const V3<double> n = mulT(Rm, nw);
                contact_law64(fresh_table<3>(k), M, delta, n, vb + cross(w, r), F, eta);
                base_contact_folded(eta, M.cc, r, n, F, dt, Q, rb);
            }
        }
        if constexpr (SCENE == 3) {
            if (near_box) {
                V3<double> nl;
                if (point_aabox(mulT(Rb, pw - bx.p), bh, delta, nl)) {
                    const V3<double> n = mulT(Rm, mul(Rb, nl));
                    contact_law64(fresh_table<3>(k), M, delta, n, vb + cross(w, r) - mulT(Rm, box_vel(pw)), F, eta);
                    base_contact_folded(eta, M.cc, r, n, F, dt, Q, rb);
                }
                const V3<double> cl = v3(ci & 1 ? bh.x : -bh.x, ci & 2 ? bh.y : -bh.y, ci & 4 ? bh.z : -bh.z);
                const V3<double> xw = bx.p + mul(Rb, cl), lt = mulT(Rm, xw - b.p);
                if (point_aabox(lt, th, delta, nl)) {  // nl: trunk face normal, toward the box corner
                    contact_law64(fresh_table<3>(k), M, delta, -1.0 * nl, vb + cross(w, lt) - mulT(Rm, box_vel(xw)), F,
                                  eta);
                    base_contact_folded(eta, M.cc, lt, -1.0 * nl, F, dt, Q, rb);
                }
            }
        }
    }

    // ---- sum over the four legs, the trunk's own terms, solve
#pragma unroll
    for (int i = 0; i < 21; ++i) Q[i] = quad_sum(Q[i]);
#pragma unroll
    for (int i = 0; i < 6; ++i) rb[i] = quad_sum(rb[i]);
    tau2 = quad_sum(tau[0] * tau[0] + tau[1] * tau[1] + tau[2] * tau[2]);
    Q[s6(0, 0)] += M.tr_Ix; Q[s6(1, 1)] += M.tr_Iy; Q[s6(2, 2)] += M.tr_Iz;
    Q[s6(3, 3)] += M.mtot; Q[s6(4, 4)] += M.mtot; Q[s6(5, 5)] += M.mtot;
    {
        const V3<double> gy = cross(w, v3(M.I0x * w.x, M.I0y * w.y, M.I0z * w.z));
        const double dm = -dt * M.m0 * M.g;
        rb[0] -= dt * gy.x; rb[1] -= dt * gy.y; rb[2] -= dt * gy.z;
        rb[3] += dm * Rm.m[6]; rb[4] += dm * Rm.m[7]; rb[5] += dm * Rm.m[8];
    }
    ldl6_solve(Q, rb);
    double dq[3] = {y0, y1, y2};
#pragma unroll
    for (int j = 0; j < 3; ++j) {
#pragma unroll
        for (int i = 0; i < 6; ++i) dq[j] -= W[j][i] * rb[i];
        lg.qd[j] += dq[j];
        lg.q[j] += dt * lg.qd[j];
    }
    const V3<double> dw = v3(rb[0], rb[1], rb[2]), dvw = mul(Rm, v3(rb[3], rb[4], rb[5]));

    // ---- the box: its corners on the ground, its side of the contacts above, its system
    if constexpr (SCENE == 3) {
        double Qb[21], rx[6];
#pragma unroll
        for (int i = 0; i < 21; ++i) Qb[i] = 0.0;
#pragma unroll
        for (int i = 0; i < 6; ++i) rx[i] = 0.0;
        const V3<double> nz = v3(Rb.m[6], Rb.m[7], Rb.m[8]), vl = mulT(Rb, bx.vw);
        if (fb) base_contact_folded(fb_eta, fb_c, mulT(Rb, fb_x - bx.p), mulT(Rb, fb_n), mulT(Rb, fb_F), dt, Qb, rx);
#pragma unroll 1
        for (int cc = 0; cc < 2; ++cc) {
            const int ci = 2 * leg + cc;
            const V3<double> cl = v3(ci & 1 ? bh.x : -bh.x, ci & 2 ? bh.y : -bh.y, ci & 4 ? bh.z : -bh.z);
            const V3<double> xw = bx.p + mul(Rb, cl);
            if (-xw.z > 0.0) {
                contact_law64(fresh_table<5>(k), M, -xw.z, nz, vl + cross(bx.w, cl), F, eta);
                base_contact_folded(eta, M.cc, cl, nz, F, dt, Qb, rx);
            }
            if (near_box) {
                const V3<double> r = v3((ci & 1 ? 0.5 : -0.5) * M.tsx, (ci & 2 ? 0.5 : -0.5) * M.tsy,
                                        (ci & 4 ? 0.5 : -0.5) * M.tsz);
                const V3<double> pw = b.p + mul(Rm, r), lb = mulT(Rb, pw - bx.p);
                double delta;
                V3<double> nl;
                if (point_aabox(lb, bh, delta, nl)) {
                    const V3<double> n = mulT(Rm, mul(Rb, nl));
                    contact_law64(fresh_table<5>(k), M, delta, n, vb + cross(w, r) - mulT(Rm, box_vel(pw)), F, eta);
                    base_contact_folded(eta, M.cc, lb, nl, mulT(Rb, -1.0 * mul(Rm, F)), dt, Qb, rx);
                }
                const V3<double> lt = mulT(Rm, xw - b.p);
                if (point_aabox(lt, th, delta, nl)) {
                    contact_law64(fresh_table<5>(k), M, delta, -1.0 * nl, vb + cross(w, lt) - mulT(Rm, box_vel(xw)), F,
                                  eta);
                    base_contact_folded(eta, M.cc, cl, mulT(Rb, mul(Rm, nl)), mulT(Rb, -1.0 * mul(Rm, F)), dt, Qb, rx);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 21; ++i) Qb[i] = quad_sum(Qb[i]);
#pragma unroll
        for (int i = 0; i < 6; ++i) rx[i] = quad_sum(rx[i]);
        Qb[s6(0, 0)] += M.bx_Ix; Qb[s6(1, 1)] += M.bx_Iy; Qb[s6(2, 2)] += M.bx_Iz;
        Qb[s6(3, 3)] += M.bx_m; Qb[s6(4, 4)] += M.bx_m; Qb[s6(5, 5)] += M.bx_m;
        const V3<double> gy = cross(bx.w, v3(M.bx_Ix * bx.w.x, M.bx_Iy * bx.w.y, M.bx_Iz * bx.w.z));
        const double dm = -dt * M.bx_m * M.g;
        rx[0] -= dt * gy.x; rx[1] -= dt * gy.y; rx[2] -= dt * gy.z;
        rx[3] += dm * nz.x; rx[4] += dm * nz.y; rx[5] += dm * nz.z;
        ldl6_solve(Qb, rx);
        bx.w = bx.w + v3(rx[0], rx[1], rx[2]);
        bx.vw = bx.vw + mul(Rb, v3(rx[3], rx[4], rx[5]));
        bx.p = bx.p + dt * bx.vw;
    }
    b.w = w + dw;
    b.vw = b.vw + dvw;
    b.p = b.p + dt * b.vw;
    if constexpr (SCENE != 3) {
        quat_step64(fresh_table<2>(k), b.qw, b.qx, b.qy, b.qz, b.w, dt);
    } else {
        // one quaternion step per lane: the trunk's on even lanes, the box's on odd lanes
        const bool odd = (leg & 1) != 0;
        double q0 = odd ? bx.qw : b.qw, q1 = odd ? bx.qx : b.qx, q2 = odd ? bx.qy : b.qy, q3 = odd ? bx.qz : b.qz;
        quat_step64(fresh_table<2>(k), q0, q1, q2, q3, selv(odd, bx.w, b.w), dt);
        b.qw = dpp<0x00>(q0); b.qx = dpp<0x00>(q1); b.qy = dpp<0x00>(q2); b.qz = dpp<0x00>(q3);
        bx.qw = dpp<0x55>(q0); bx.qx = dpp<0x55>(q1); bx.qy = dpp<0x55>(q2); bx.qz = dpp<0x55>(q3);
    }
}

}  // namespace f64
}  // namespace mppi
