// Lane-split rollout for gfx950: one sample per 16 lanes (four per leg), four samples per
// 64-lane workgroup, so that K = 4096 samples occupy 1024 waves -- one on every SIMD of
// the chip -- where the quad kernel (one lane per leg) leaves three SIMDs in four idle.
//
// The per-step instruction stream of a wave is what sets the time on a SIMD that holds
// one wave, so the split pays only where the 16 lanes run the same instructions on
// different data:
//   * knot interpolation: lane s < 3 of a leg interpolates joint s; the three targets are
//     broadcast in the quad (DPP quad_perm);
//   * trigonometry: lane s evaluates the sine and cosine of the leg's angle s (abduction,
//     flexion, flexion + knee) and broadcasts them;
//   * contacts with the trunk corners and the free box's corners: lane g < 8 takes trunk
//     corner g, lane g >= 8 box corner g - 8 (the quad kernel takes two of each per lane);
//   * the two 6x6 solves of the pushing scene: even lanes solve the trunk's system, odd
//     lanes the box's, from selected operands, and swap results with their neighbour.
// The leg's kinematics, mass-matrix and bias terms and its foot contacts run in all four
// lanes of the leg; each lane eliminates two of the leg's columns.  The trunk and box systems
// (Sec. III-A's dynamics step: (M + dt D) dv = dt f, the legs eliminated first) are summed over
// the 16 lanes through LDS in a fixed order: one lane writes a leg's terms and each lane its
// columns', or, while a wave has a rare contact, every lane all its terms.  The results do not
// depend on timing.
//
// The step computes the same discretisation as the quad kernel in the same arithmetic
// type R (the state is FP32 between steps); only summation orders differ.
#include "mppi_device.h"
#include "mppi_launch.h"
#include "mppi_step64.h"

namespace mppi {
namespace r16 {

struct alignas(16) Quad {
    float v[4];
};

constexpr int kSamples = 4;     // samples per workgroup (one wave)
constexpr int kNVMax = 55;      // summed values: trunk system 21 + 6, torque^2, box system 21 + 6
constexpr int kPitch = 20;      // LDS row pitch of one summed value over the 16 lanes (16 used)
constexpr int kSumPitch = 64;   // per-sample row of the sums

template <int SCENE>
__device__ __forceinline__ constexpr int n_summed()
{
    return SCENE == 3 ? 55 : 28;
}

// LDS per sample (values of type S): [0, kBoxRow) a region used in turn for the trunk corners'
// rows (27 x kPitch) and for the legs' values (4 x kLegPitch) and eliminated columns (4 x
// kElimPitch); in the pushing scene the box's rows follow at kBoxRow (27 x kPitch)
constexpr int kLegPitch = 28, kElimPitch = 50, kElimRow = 4 * kLegPitch, kBoxRow = 28 * kPitch;

// where lane g's summed values g and g + 16 of the trunk's 28 (21 + 6 + torque^2) stand in a
// leg's eliminated columns (6 rows x 8 columns; column 6 is the right side, 7 zeros)
__device__ __forceinline__ int elim_slot(int e)
{
    if (e >= 27) return 7;
    if (e >= 21) return (e - 21) * 8 + 6;
    int i = 0, first = 0;
    while (e - first >= 6 - i) first += 6 - i++;
    return i * 8 + i + (e - first);
}

// bounding spheres of two bodies: (r1 + r2)^2 <= 2 (r1^2 + r2^2), with a margin for the rounding
constexpr double kNear = 2.001;

// fixed-order sum of the 16 partials of one value
template <typename R>
__device__ __forceinline__ R sum16(const R* p)
{
    R a[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = p[2 * i] + p[2 * i + 1];
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = a[2 * i] + a[2 * i + 1];
    return (a[0] + a[1]) + (a[2] + a[3]);
}

// the same for 8 of them
template <typename R>
__device__ __forceinline__ R sum8(const R* p)
{
    R a[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = p[2 * i] + p[2 * i + 1];
    return (a[0] + a[1]) + (a[2] + a[3]);
}

template <typename R>
__device__ __forceinline__ R sel(bool c, R a, R b)
{
    return c ? a : b;
}

// pose and velocity of a rigid body (the trunk or the free box): rotation to world,
// position, world linear velocity, body-frame angular velocity
template <typename R>
struct Pose {
    M33<R> Rt;
    V3<R> p, vw, w;
};
template <typename R>
__device__ __forceinline__ V3<R> pose_point_vel(const Pose<R>& B, V3<R> x)
{
    return B.vw + mul(B.Rt, cross(B.w, mulT(B.Rt, x - B.p)));
}
template <typename R>
__device__ __forceinline__ Pose<R> sel_pose(bool c, const Pose<R>& a, const Pose<R>& b)
{
    Pose<R> o;
#pragma unroll
    for (int i = 0; i < 9; ++i) o.Rt.m[i] = c ? a.Rt.m[i] : b.Rt.m[i];
    o.p = selv(c, a.p, b.p);
    o.vw = selv(c, a.vw, b.vw);
    o.w = selv(c, a.w, b.w);
    return o;
}

template <typename T, typename U>
__device__ __forceinline__ V3<T> cv(V3<U> a)
{
    return V3<T>{T(a.x), T(a.y), T(a.z)};
}

// A a with the products added in a stated order: the compiler's choice of the products it
// fuses would otherwise move FP32 roundings when the code around it changes
template <typename R>
__device__ __forceinline__ V3<R> mul_ordered(const M33<R>& A, V3<R> a)
{
    return v3(R(fma(A.m[2], a.z, fma(A.m[1], a.y, A.m[0] * a.x))), R(fma(A.m[5], a.z, fma(A.m[4], a.y, A.m[3] * a.x))),
              R(fma(A.m[8], a.z, fma(A.m[7], a.y, A.m[6] * a.x))));
}

// Vector operations with the zeros of ex = (1, 0, 0), ey = (0, cos, sin) and the hip (x, y, 0)
// left out, which the compiler has to multiply by (0 times an infinity is not 0): about 90 of a
// step's 1500 instructions and more.  Every product and sum is rounded as in the full form, whose
// order is stated: fma of the first product on the second, sums from the left, and a product whose
// other terms were zeros by itself (`lone`, never fused into a sum).  Full form / here, MI355X:
// climbing K = 1001, H = 47, mixed, 212 / 206 us; pushing K = 4096, H = 60, FP32, whole control
// step, 274 / 264; terrain walk with a proposal, K = 1024 + 256, H = 50, FP32, 221 / 214.
template <typename R>
__device__ __forceinline__ R lone(R a, R b)
{
#pragma clang fp contract(off)
    return a * b;
}
template <typename R>
__device__ __forceinline__ R mad(R a, R b, R c)
{
    return R(fma(a, b, c));
}
template <typename R>
__device__ __forceinline__ V3<R> lonev(R a, V3<R> b)
{
    return v3(lone(a, b.x), lone(a, b.y), lone(a, b.z));
}
template <typename R>
__device__ __forceinline__ V3<R> madv(R a, V3<R> b, V3<R> c)
{
    return v3(mad(a, b.x, c.x), mad(a, b.y, c.y), mad(a, b.z, c.z));
}
template <typename R>
__device__ __forceinline__ V3<R> crossf(V3<R> a, V3<R> b)
{
    return v3(mad(a.y, b.z, -lone(a.z, b.y)), mad(a.z, b.x, -lone(a.x, b.z)), mad(a.x, b.y, -lone(a.y, b.x)));
}
template <typename R>
__device__ __forceinline__ R dotf(V3<R> a, V3<R> b)
{
    return mad(a.z, b.z, mad(a.x, b.x, lone(a.y, b.y)));
}
template <typename R>
__device__ __forceinline__ V3<R> ex_cross(V3<R> a)  // ex x a
{
    return v3(R(0), -a.z, a.y);
}
template <typename R>
__device__ __forceinline__ V3<R> x0_cross(V3<R> e, V3<R> a)  // e x a, e.x = 0
{
    return v3(mad(e.y, a.z, -lone(e.z, a.y)), lone(e.z, a.x), -lone(e.y, a.x));
}
template <typename R>
__device__ __forceinline__ V3<R> cross_x0(V3<R> a, V3<R> e)  // a x e, e.x = 0
{
    return v3(mad(a.y, e.z, -lone(a.z, e.y)), -lone(a.x, e.z), lone(a.x, e.y));
}
template <typename R>
__device__ __forceinline__ V3<R> cross_z0(V3<R> a, V3<R> h)  // a x h, h.z = 0
{
    return v3(-lone(a.z, h.y), lone(a.z, h.x), mad(a.x, h.y, -lone(a.y, h.x)));
}
template <typename R>
__device__ __forceinline__ V3<R> hip_cross(V3<R> h, V3<R> e)  // h x e, h.z = e.x = 0
{
    return v3(lone(h.y, e.z), -lone(h.x, e.z), lone(h.x, e.y));
}
template <typename R>
__device__ __forceinline__ R dot_x0(V3<R> e, V3<R> a)  // e . a, e.x = 0
{
    return mad(e.z, a.z, lone(e.y, a.y));
}
// (I - d d^T) applied to ex and to e (e.x = 0): rod_I without its factor
template <typename R>
__device__ __forceinline__ V3<R> rod_ex(V3<R> d)
{
    return v3(mad(-d.x, d.x, R(1)), -lone(d.x, d.y), -lone(d.x, d.z));
}
template <typename R>
__device__ __forceinline__ V3<R> rod_x0(V3<R> d, V3<R> e)
{
    const R t = dot_x0(d, e);
    return v3(-lone(t, d.x), mad(-t, d.y, e.y), mad(-t, d.z, e.z));
}

// Factor of the leg's 3x3 system and solution of the body's 6x6 in the system type: in FP64 the
// factorisation without square roots and with reciprocals from the hardware's estimate, a step's
// 9 general divisions and 9 square roots less (climbing K = 1001, H = 47, mixed: 206 / 185 us).
__device__ __forceinline__ Chol3<float> leg_factor(const LegSys<float>& L)
{
    return chol3(L.A00, L.A01, L.A11, L.A02, L.A12, L.A22);
}
__device__ __forceinline__ f64::Ldl3 leg_factor(const LegSys<double>& L)
{
    return f64::ldl3(L.A00, L.A01, L.A11, L.A02, L.A12, L.A22);
}
__device__ __forceinline__ void body_solve(float* Q, float* r) { chol6_solve(Q, r); }
__device__ __forceinline__ void body_solve(double* Q, double* r) { f64::ldl6_solve(Q, r); }

// a contact on the leg's calf with weight wgt (1: applied, 0: nothing added).  The contact
// velocity and the law are evaluated in the geometry type R; the force and damping terms
// on the trunk's base rows and on the leg's joint rows accumulate in the system type S.
template <typename R, typename S>
__device__ __forceinline__ void leg_contact_w(const ModelT<R>& M, const LegGeo<R>& G, V3<R> vb, V3<R> w,
                                              const R qd[3], R delta, V3<R> n, V3<R> r, V3<R> vo, S dt, R wgt, S* Q,
                                              S* rb, LegSys<S>& L, V3<R>& F, R& eta)
{
    // ja in full: with its zeros left out, FP32 contacts were rounded differently (the cause was
    // not found)
    const V3<R> ex = v3(R(1), R(0), R(0));
    const V3<R> ja = cross(ex, r - G.h), jf = cross(G.ey, r - G.h), jk = cross(G.ey, r - G.pk);
    V3<R> vc = vb + crossf(w, r);
    vc.y = mad(qd[0], ja.y, vc.y);
    vc.z = mad(qd[0], ja.z, vc.z);
    vc = madv(qd[2], jk, madv(qd[1], jf, vc)) - vo;
    contact_law(M, delta, n, vc, F, eta);
    F = wgt * F;
    eta = wgt * eta;
    const S e = S(eta), cw = S(wgt) * S(M.cc);
    const S ce = cw - e;
    const V3<S> rs = cv<S>(r), ns = cv<S>(n), Fs = cv<S>(F);
    base_contact_folded(e, cw, rs, ns, Fs, dt, Q, rb);
    // the leg's rows: dt (e J_l^T J + ce g_l g^T) with g_l = J_l^T n, dt e and dt ce folded
    // into the operands
    const S de = dt * e;
    const V3<S> jv[3] = {cv<S>(ja), cv<S>(jf), cv<S>(jk)};
    const S gj[3] = {dot_x0(jv[0], ns), dotf(jv[1], ns), dotf(jv[2], ns)};
    const S dg[3] = {dt * ce * gj[0], dt * ce * gj[1], dt * ce * gj[2]};
    const V3<S> gA = cross(rs, ns);
    const S g0[6] = {gA.x, gA.y, gA.z, ns.x, ns.y, ns.z};
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const V3<S> rxj = j ? crossf(rs, jv[j]) : cross_x0(rs, jv[j]);
        const S jb[6] = {rxj.x, rxj.y, rxj.z, jv[j].x, jv[j].y, jv[j].z};
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const S t = lone(dg[j], g0[i]);
            L.C[j][i] += j == 0 && i == 3 ? t : mad(de, jb[i], t);
        }
        L.rl[j] = mad(dt, j ? dotf(jv[j], Fs) : dot_x0(jv[j], Fs), L.rl[j]);
    }
    L.A00 += mad(de, dot_x0(jv[0], jv[0]), lone(dg[0], gj[0]));
    L.A01 += mad(de, dot_x0(jv[0], jv[1]), lone(dg[0], gj[1]));
    L.A02 += mad(de, dot_x0(jv[0], jv[2]), lone(dg[0], gj[2]));
    L.A11 += mad(de, dotf(jv[1], jv[1]), lone(dg[1], gj[1]));
    L.A12 += mad(de, dotf(jv[1], jv[2]), lone(dg[1], gj[2]));
    L.A22 += mad(de, dotf(jv[2], jv[2]), lone(dg[2], gj[2]));
}

// contact terms of a force F at body-frame point r with normal n and secant eta (all in
// the geometry type R) on a 6x6 body system accumulated in S
template <typename R, typename S>
__device__ __forceinline__ void body_contact(R eta, R c, V3<R> r, V3<R> n, V3<R> F, S dt, S* Q, S* rb)
{
    base_contact_folded(S(eta), S(c), cv<S>(r), cv<S>(n), cv<S>(F), dt, Q, rb);
}

// ------------------------------------------------------------------------------
// one dynamics step of one sample; lane g (0..15) of the sample, leg g >> 2, sub-lane
// g & 3.  R: the geometry type (kinematics, contact detection and law, state); S: the
// system type (mass matrix, bias, contact damping and forces as terms of the implicit
// system, the leg elimination, the sums and the 6x6 solves).  MR / MS: the model in
// both.  uj: the joint target this lane interpolated (joint g & 3 of its leg, lanes 3
// repeat joint 2).  red / sred: this sample's LDS rows.  tau2 receives sum tau^2.
// ------------------------------------------------------------------------------
template <int SCENE, typename R, typename S>
__device__ __forceinline__ void step16(const ModelT<R>& MR, const ModelT<S>& MS, const float* __restrict__ hf, S dt,
                                       S kp, S kd, int g, int eo0, int eo1, Base<R>& b, Leg<R>& lg, BoxS<R>& bx,
                                       R uj, S* red, S* sred, R& tau2)
{
    const int leg = g >> 2, sub = g & 3;
    const R dtr = R(dt);
    const R u[3] = {dpp<0x00>(uj), dpp<0x55>(uj), dpp<0xAA>(uj)};
    S tau[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) tau[j] = kp * (S(u[j]) - S(lg.q[j])) - kd * S(lg.qd[j]);
    const S t2 = tau[0] * tau[0] + tau[1] * tau[1] + tau[2] * tau[2];

    const M33<R> Rm = quat_R(b.qw, b.qx, b.qy, b.qz);
    const V3<R> w = b.w;
    const V3<R> vb = mulT(Rm, b.vw);
    const V3<R> gb = (-MR.g) * v3(Rm.m[6], Rm.m[7], Rm.m[8]);

    // ---- leg kinematics: lane `sub` evaluates angle sub of the leg, the quad shares them
    R sn, cs;
    {
        const R ang = (sub == 0) ? lg.q[0] : (sub == 1) ? lg.q[1] : lg.q[1] + lg.q[2];
        m_sincos(ang, &sn, &cs);
    }
    const R sa = dpp<0x00>(sn), ca = dpp<0x00>(cs);
    const R sf = dpp<0x55>(sn), cf = dpp<0x55>(cs);
    const R s12 = dpp<0xAA>(sn), c12 = dpp<0xAA>(cs);
    LegGeo<R> G;
    G.ey = v3(R(0), ca, sa);
    G.d1 = v3(-sf, sa * cf, -ca * cf);
    G.d2 = v3(-s12, sa * c12, -ca * c12);
    G.h = v3((leg < 2) ? MR.hip_x : -MR.hip_x, (leg & 1) ? -MR.hip_y : MR.hip_y, R(0));
    G.pk = G.h + MR.l1 * G.d1;
    G.pf = G.pk + MR.l2 * G.d2;
    G.c1 = G.h + (R(0.5) * MR.l1) * G.d1;
    G.c2 = G.pk + (R(0.5) * MR.l2) * G.d2;

    // the leg's geometry and velocities in the system type
    const V3<S> ex = v3(S(1), S(0), S(0));
    const V3<S> ey = cv<S>(G.ey), d1 = cv<S>(G.d1), d2 = cv<S>(G.d2), h = cv<S>(G.h), pk = cv<S>(G.pk),
                c1 = cv<S>(G.c1), c2 = cv<S>(G.c2);
    const V3<S> ws = cv<S>(w), gbs = cv<S>(gb);
    const S dqa = S(lg.qd[0]), dqf = S(lg.qd[1]), dqk = S(lg.qd[2]);

    // ---- the leg's mass-matrix terms: base block, coupling columns, leg block
    S Q[21];
#pragma unroll
    for (int i = 0; i < 21; ++i) Q[i] = S(0);
    {
        const S r1 = dot(c1, c1), r2 = dot(c2, c2);
        const S cv1[3] = {c1.x, c1.y, c1.z}, cv2[3] = {c2.x, c2.y, c2.z};
        const S d1v[3] = {d1.x, d1.y, d1.z}, d2v[3] = {d2.x, d2.y, d2.z};
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = i; j < 3; ++j) {
                const S I = (i == j) ? S(1) : S(0);
                Q[s6(i, j)] = MS.k1 * (I - d1v[i] * d1v[j]) + MS.k2 * (I - d2v[i] * d2v[j]) +
                              MS.m1 * (r1 * I - cv1[i] * cv1[j]) + MS.m2 * (r2 * I - cv2[i] * cv2[j]);
            }
        const V3<S> hl = MS.m1 * c1 + MS.m2 * c2;
        Q[s6(0, 4)] = -hl.z; Q[s6(0, 5)] = hl.y;
        Q[s6(1, 3)] = hl.z;  Q[s6(1, 5)] = -hl.x;
        Q[s6(2, 3)] = -hl.y; Q[s6(2, 4)] = hl.x;
    }
    LegSys<S> L;
    {
        const V3<S> ua1 = ex_cross(c1 - h), ua2 = ex_cross(c2 - h);
        const V3<S> uf1 = x0_cross(ey, c1 - h), uf2 = x0_cross(ey, c2 - h);
        const V3<S> uk2 = x0_cross(ey, c2 - pk), z2 = rod_x0(d2, ey);
        const V3<S> Pa = madv(MS.m1, ua1, lonev(MS.m2, ua2));
        const V3<S> La = madv(MS.k2, rod_ex(d2), madv(MS.k1, rod_ex(d1), madv(MS.m1, cross_x0(c1, ua1),
                                                                              lonev(MS.m2, cross_x0(c2, ua2)))));
        const V3<S> Pf = madv(MS.m1, uf1, lonev(MS.m2, uf2));
        const V3<S> Lf = madv(MS.k2, z2, madv(MS.k1, rod_x0(d1, ey), madv(MS.m1, crossf(c1, uf1),
                                                                          lonev(MS.m2, crossf(c2, uf2)))));
        const V3<S> Pk = lonev(MS.m2, uk2);
        const V3<S> Lk = madv(MS.m2, crossf(c2, uk2), lonev(MS.k2, z2));
        const V3<S> Ls[3] = {La, Lf, Lk}, Ps[3] = {Pa, Pf, Pk};
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            L.C[j][0] = Ls[j].x; L.C[j][1] = Ls[j].y; L.C[j][2] = Ls[j].z;
            L.C[j][3] = Ps[j].x; L.C[j][4] = Ps[j].y; L.C[j][5] = Ps[j].z;
        }
        // ex . L + (h x ex) . P and ey . L + (o x ey) . P
        const V3<S> oxa_f = hip_cross(h, ey), oxa_k = cross_x0(pk, ey);
        L.A00 = La.x - lone(h.y, Pa.z);
        L.A01 = Lf.x - lone(h.y, Pf.z);
        L.A02 = Lk.x - lone(h.y, Pk.z);
        L.A11 = dot_x0(ey, Lf) + dotf(oxa_f, Pf);
        L.A12 = dot_x0(ey, Lk) + dotf(oxa_f, Pk);
        L.A22 = dot_x0(ey, Lk) + dotf(oxa_k, Pk);
    }

    // ---- bias forces of the leg (zero generalized acceleration, gravity)
    S rb[6];
    {
        const V3<S> wa = v3(ws.x + dqa, ws.y, ws.z);
        const V3<S> w1 = v3(wa.x, mad(dqf, ey.y, wa.y), mad(dqf, ey.z, wa.z));
        const V3<S> we = cross_x0(wa, ey);
        const V3<S> al1 = v3(lone(dqf, we.x), mad(dqa, ws.z, lone(dqf, we.y)), mad(dqa, -ws.y, lone(dqf, we.z)));
        const V3<S> ah = crossf(ws, cross_z0(ws, h));
        const V3<S> r1 = c1 - h, rk = pk - h;
        const V3<S> ac1 = ah + cross(al1, r1) + cross(w1, cross(w1, r1));
        const V3<S> apk = ah + cross(al1, rk) + cross(w1, cross(w1, rk));
        const V3<S> w2 = v3(w1.x, mad(dqk, ey.y, w1.y), mad(dqk, ey.z, w1.z));
        const V3<S> al2 = madv(dqk, cross_x0(w1, ey), al1);
        const V3<S> r2 = c2 - pk;
        const V3<S> ac2 = apk + cross(al2, r2) + cross(w2, cross(w2, r2));
        const V3<S> F1 = MS.m1 * (ac1 - gbs), F2 = MS.m2 * (ac2 - gbs);
        const V3<S> N1 = rod_I(MS.k1, d1, al1) + cross(w1, rod_I(MS.k1, d1, w1));
        const V3<S> N2 = rod_I(MS.k2, d2, al2) + cross(w2, rod_I(MS.k2, d2, w2));
        const V3<S> Tk = N2 + cross(r2, F2);
        const V3<S> Th = N1 + cross(r1, F1) + N2 + cross(c2 - h, F2);
        const V3<S> Tb = N1 + N2 + cross(c1, F1) + cross(c2, F2);
        const V3<S> Fb = F1 + F2;
        rb[0] = -dt * Tb.x; rb[1] = -dt * Tb.y; rb[2] = -dt * Tb.z;
        rb[3] = -dt * Fb.x; rb[4] = -dt * Fb.y; rb[5] = -dt * Fb.z;
        L.rl[0] = dt * (tau[0] - Th.x);
        L.rl[1] = dt * (tau[1] - dot_x0(ey, Th));
        L.rl[2] = dt * (tau[2] - dot_x0(ey, Tk));
    }
    L.A00 += dt * kd; L.A11 += dt * kd; L.A22 += dt * kd;

    [[maybe_unused]] BoxFrame<R> bf;
    const V3<R> zero = v3(R(0), R(0), R(0));
    V3<R> F;
    R eta;
    if constexpr (SCENE == 3) bf.Rb = quat_R(bx.qw, bx.qx, bx.qy, bx.qz);

    // ---- the leg's foot against terrain and the static or free box.  Each lane lists its
    // foot's contacts (terrain, box) and the wave runs one contact body per listed entry:
    // usually one pass, a second only where a foot touches both.
    [[maybe_unused]] bool foot_box = false;   // some lane of the wave has its foot on the box
    [[maybe_unused]] R fb_eta = R(0), fb_c = R(0);
    [[maybe_unused]] V3<R> fb_r = zero, fb_n = zero, fb_F = zero;  // this lane's share for the box's system
    {
        const V3<R> pfw = b.p + mul(Rm, G.pf);
        R dT, dB = R(0);
        V3<R> nT, nB = zero;
        const bool hitT = terrain<SCENE>(MR, hf, pfw, MR.foot_r, dT, nT);
        bool hitB = false;
        if constexpr (SCENE == 2) {
            hitB = sphere_aabox(pfw - v3(MR.sb_cx, MR.sb_cy, MR.sb_cz), MR.foot_r, v3(MR.sb_hx, MR.sb_hy, MR.sb_hz),
                                dB, nB);
        }
        if constexpr (SCENE == 3) {
            // outside the sphere around the box there is no contact
            const V3<R> d = pfw - bx.p, bh = v3(MR.bx_hx, MR.bx_hy, MR.bx_hz);
            if (__builtin_amdgcn_ballot_w64(dot(d, d) <= R(kNear) * (MR.foot_r * MR.foot_r + dot(bh, bh)))) {
                V3<R> nl = v3(R(0), R(0), R(1));  // left as is when the foot misses the box
                hitB = sphere_aabox(mulT(bf.Rb, d), MR.foot_r, bh, dB, nl);
                nB = mul(bf.Rb, nl);  // box -> foot (world)
            }
        }
        const int cnt = int(hitT) + int(hitB);
#pragma unroll
        for (int it = 0; it < ((SCENE == 2 || SCENE == 3) ? 2 : 1); ++it) {
            if (!__builtin_amdgcn_ballot_w64(it < cnt)) break;
            const bool isB = (it == 0) ? !hitT : true;  // pass 0: terrain if touched, else the box
            // a lane without a contact in this pass takes a neutral one (zero depth, upward
            // normal, zero weight), so nothing it adds can be non-finite
            const bool on = it < cnt;
            const R wgt = on ? R(1) : R(0);
            const R delta = on ? (isB ? dB : dT) : R(0);
            const V3<R> nw = on ? selv(isB, nB, nT) : v3(R(0), R(0), R(1));
            const V3<R> n = mulT(Rm, nw);
            V3<R> vo = zero;
            // the box's velocity and its share of the contact, only while a foot of the wave
            // touches it
            [[maybe_unused]] V3<R> pcw;
            [[maybe_unused]] bool box_pass = false;
            if constexpr (SCENE == 3) {
                box_pass = __builtin_amdgcn_ballot_w64(isB && on) != 0;
                if (box_pass) {
                    pcw = pfw - MR.foot_r * nw;
                    vo = selv(isB && on, mulT(Rm, box_point_vel(bx, bf, pcw)), zero);
                }
            }
            leg_contact_w(MR, G, vb, w, lg.qd, delta, n, G.pf - MR.foot_r * n, vo, dt, wgt, Q, rb, L, F, eta);
            if constexpr (SCENE == 3) {
                if (box_pass) {
                    // the box's share in its frame (added below; a lane has one box contact at most)
                    foot_box = true;
                    const bool mine = isB && on;
                    const R wb = isB ? wgt : R(0);
                    fb_eta = sel(mine, eta, fb_eta);
                    fb_c = sel(mine, MR.cc, fb_c);
                    fb_r = selv(mine, mulT(bf.Rb, pcw - bx.p), fb_r);
                    fb_n = selv(mine, mulT(bf.Rb, nw), fb_n);
                    fb_F = selv(mine, mulT(bf.Rb, (-wb) * mul(Rm, F)), fb_F);
                }
            }
        }
    }

    // ---- one corner per lane: trunk corner g (g < 8), free-box corner g - 8 (g >= 8).  Contacts
    // with the trunk (a fallen robot, the box against the robot) are rare: without one, and
    // with no foot on the box, the sums below take the short way (`plain`).
    bool hitG = false, hitP = false, plain = true;
    R dG = R(0), dP = R(0);
    V3<R> nG = zero, nlq = zero, cl = zero, x = zero;
    [[maybe_unused]] V3<R> lq = zero, rloc = zero;
    [[maybe_unused]] const bool own_trunk = g < 8;
    [[maybe_unused]] Pose<R> PT, PB;
    PT.Rt = Rm; PT.p = b.p; PT.vw = b.vw; PT.w = b.w;
    if constexpr (SCENE != 3) {
        rloc = v3((g & 1 ? R(0.5) : R(-0.5)) * MR.tsx, (g & 2 ? R(0.5) : R(-0.5)) * MR.tsy,
                  (g & 4 ? R(0.5) : R(-0.5)) * MR.tsz);
        const V3<R> pw = b.p + mul(Rm, rloc);
        hitG = terrain<SCENE>(MR, hf, pw, R(0), dG, nG) && g < 8;
        if constexpr (SCENE == 2)
            hitP = point_aabox(pw - v3(MR.sb_cx, MR.sb_cy, MR.sb_cz), v3(MR.sb_hx, MR.sb_hy, MR.sb_hz), dP, nlq) &&
                   g < 8;
        plain = __builtin_amdgcn_ballot_w64(hitG || hitP) == 0;
    } else {
        PB.Rt = bf.Rb; PB.p = bx.p; PB.vw = bx.vw; PB.w = bx.w;
        const int ci = g & 7;
        const V3<R> th = v3(R(0.5) * MR.tsx, R(0.5) * MR.tsy, R(0.5) * MR.tsz), bh = v3(MR.bx_hx, MR.bx_hy, MR.bx_hz);
        const V3<R> hP = selv(own_trunk, th, bh);
        cl = v3(ci & 1 ? hP.x : -hP.x, ci & 2 ? hP.y : -hP.y, ci & 4 ? hP.z : -hP.z);
        x = selv(own_trunk, b.p + mul(Rm, cl), bx.p + mul(bf.Rb, cl));
        hitG = terrain<SCENE>(MR, hf, x, R(0), dG, nG);
        // the corner inside the other body, only while the bounding spheres can overlap
        const V3<R> dc = b.p - bx.p;
        if (__builtin_amdgcn_ballot_w64(dot(dc, dc) <= R(kNear) * (dot(th, th) + dot(bh, bh)))) {
            lq = selv(own_trunk, mulT(bf.Rb, x - bx.p), mulT(Rm, x - b.p));
            hitP = point_aabox(lq, selv(own_trunk, bh, th), dP, nlq);  // nlq: Q's face normal toward the corner
        }
        plain = __builtin_amdgcn_ballot_w64(hitP || (hitG && own_trunk)) == 0 && !foot_box;
    }

    // ---- eliminate the leg, A_ll^-1 [A_l0 | r_l]: lane `sub` solves columns sub and sub + 4 (the
    // fifth and sixth velocity, the right side, and a zero column)
    const auto L3 = leg_factor(L);
    S W0[3], W1[3];
    const bool sub1 = (sub & 1) != 0, sub2 = (sub & 2) != 0;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        W0[j] = sel(sub2, sel(sub1, L.C[j][3], L.C[j][2]), sel(sub1, L.C[j][1], L.C[j][0]));
        W1[j] = sel(sub2, sel(sub1, S(0), L.rl[j]), sel(sub1, L.C[j][5], L.C[j][4]));
    }
    solve3(L3, W0[0], W0[1], W0[2]);
    solve3(L3, W1[0], W1[1], W1[2]);

    // ---- sum the trunk (and box) systems and the squared torques over the 16 lanes
    const bool keep = sub == 0;
    if (plain) {
        // the leg's values from its first lane and the eliminated parts from the lanes that have
        // them: value by value the same sums as below, whose other terms are zeros
        if (keep) {
            S* o = red + leg * kLegPitch;
#pragma unroll
            for (int i = 0; i < 21; ++i) o[i] = Q[i];
#pragma unroll
            for (int i = 0; i < 6; ++i) o[21 + i] = rb[i];
            o[27] = t2;
        }
        {
            S* o = red + kElimRow + leg * kElimPitch + sub;
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                if (i < 4) o[8 * i] = L.C[0][i] * W0[0] + L.C[1][i] * W0[1] + L.C[2][i] * W0[2];
                o[8 * i + 4] = L.C[0][i] * W1[0] + L.C[1][i] * W1[1] + L.C[2][i] * W1[2];
            }
        }
        if constexpr (SCENE == 3) {
            // the box's corners against the ground (lanes 8-15)
            S Qb[21], rbx[6];
#pragma unroll
            for (int i = 0; i < 21; ++i) Qb[i] = S(0);
#pragma unroll
            for (int i = 0; i < 6; ++i) rbx[i] = S(0);
            if (__builtin_amdgcn_ballot_w64(hitG)) {
                const R wgt = hitG ? R(1) : R(0);
                const V3<R> n = hitG ? nG : v3(R(0), R(0), R(1));
                contact_law(MR, hitG ? dG : R(0), n, hitG ? pose_point_vel(PB, x) : zero, F, eta);
                F = wgt * F;
                eta = wgt * eta;
                body_contact(eta, wgt * MR.cc, cl, mulT(bf.Rb, n), mulT(bf.Rb, F), dt, Qb, rbx);
            }
            if (g >= 8) {
#pragma unroll
                for (int e = 0; e < 21; ++e) red[kBoxRow + e * kPitch + g] = Qb[e];
#pragma unroll
                for (int e = 0; e < 6; ++e) red[kBoxRow + (21 + e) * kPitch + g] = rbx[e];
            }
        }
        __syncthreads();
        {
            // every lane reads (lanes past the last value a valid one, unused), so that the
            // reads wait together
            const S* v = red + g;
            const S* xe = red + kElimRow;
            S s0[4], s1[4];
#pragma unroll
            for (int l = 0; l < 4; ++l) {
                s0[l] = v[l * kLegPitch] - xe[l * kElimPitch + eo0];
                s1[l] = v[l * kLegPitch + 16] - xe[l * kElimPitch + eo1];
            }
            const S a0 = (s0[0] + s0[1]) + (s0[2] + s0[3]), a1 = (s1[0] + s1[1]) + (s1[2] + s1[3]);
            [[maybe_unused]] S b0, b1;
            if constexpr (SCENE == 3) {
                b0 = sum8(red + kBoxRow + g * kPitch + 8);
                b1 = sum8(red + kBoxRow + min(g + 16, 26) * kPitch + 8);
                sred[28 + g] = b0;
            }
            sred[g] = a0;
            if (g < 12) {
                sred[g + 16] = a1;
                if constexpr (SCENE == 3) sred[28 + 16 + g] = b1;  // the twelfth to a place that is not read
            }
        }
        __syncthreads();
    } else {
        // all columns in every lane, each lane's corner terms added to its own (the leg's values
        // in its first lane), then the 16 lanes' values in a fixed order
        S W[3][6];
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            S x0 = L.C[0][i], x1 = L.C[1][i], x2 = L.C[2][i];
            solve3(L3, x0, x1, x2);
            W[0][i] = x0; W[1][i] = x1; W[2][i] = x2;
        }
        S y0 = L.rl[0], y1 = L.rl[1], y2 = L.rl[2];
        solve3(L3, y0, y1, y2);
#pragma unroll
        for (int i = 0; i < 6; ++i) {
#pragma unroll
            for (int j = i; j < 6; ++j)
                Q[s6(i, j)] -= L.C[0][i] * W[0][j] + L.C[1][i] * W[1][j] + L.C[2][i] * W[2][j];
            rb[i] -= L.C[0][i] * y0 + L.C[1][i] * y1 + L.C[2][i] * y2;
        }
#pragma unroll
        for (int i = 0; i < 21; ++i) Q[i] = sel(keep, Q[i], S(0));
#pragma unroll
        for (int i = 0; i < 6; ++i) rb[i] = sel(keep, rb[i], S(0));
        [[maybe_unused]] S Qb[21], rbx[6];
        if constexpr (SCENE != 3) {
            if (hitG) {
                const V3<R> n = mulT(Rm, nG);
                contact_law(MR, dG, n, vb + cross(w, rloc), F, eta);
                body_contact(eta, MR.cc, rloc, n, F, dt, Q, rb);
            }
            if constexpr (SCENE == 2) {
                if (hitP) {
                    const V3<R> n = mulT(Rm, nlq);
                    contact_law(MR, dP, n, vb + cross(w, rloc), F, eta);
                    body_contact(eta, MR.cc, rloc, n, F, dt, Q, rb);
                }
            }
        } else {
            // A corner of body P (the trunk on lanes 0-7, the box on lanes 8-15) against the
            // other body Q (a point inside Q's box, normal out of Q's nearest face) and against
            // the terrain.  The same code serves both roles: each contact adds its terms to the
            // trunk's and the box's 6x6 systems in their own frames, with zero weight where a
            // body is not part of the contact.
#pragma unroll
            for (int i = 0; i < 21; ++i) Qb[i] = S(0);
#pragma unroll
            for (int i = 0; i < 6; ++i) rbx[i] = S(0);
            body_contact(sel(keep, fb_eta, R(0)), sel(keep, fb_c, R(0)), fb_r, fb_n, selv(keep, fb_F, zero), dt, Qb, rbx);
            const Pose<R> own = sel_pose(own_trunk, PT, PB), oth = sel_pose(own_trunk, PB, PT);
            const int cnt = int(hitP) + int(hitG);
            if (__builtin_amdgcn_ballot_w64(cnt > 0)) {
                const V3<R> vP = pose_point_vel(own, x), vQ = pose_point_vel(oth, x);
                const V3<R> nPw = mul(oth.Rt, nlq);
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    if (!__builtin_amdgcn_ballot_w64(it < cnt)) break;
                    const bool pair = (it == 0) && hitP;  // pass 0: the pair if touching, else the terrain
                    // a lane without a contact in this pass takes a neutral one (zero depth and
                    // velocity, zero weight), so nothing it adds can be non-finite
                    const bool on = it < cnt;
                    const R wgt = on ? R(1) : R(0);
                    const R wq = pair ? wgt : R(0);
                    const V3<R> n = on ? selv(pair, nPw, nG) : v3(R(0), R(0), R(1));
                    contact_law(MR, on ? (pair ? dP : dG) : R(0), n, on ? selv(pair, vP - vQ, vP) : zero, F, eta);
                    F = wgt * F;
                    eta = wgt * eta;
                    // P's side in P's frame (force +F), Q's side in Q's frame (force -F)
                    const V3<R> nP = mulT(own.Rt, n), FP = mulT(own.Rt, F);
                    const V3<R> FQ = R(-1) * mulT(oth.Rt, F);
                    const R cP = wgt * MR.cc, cQ = wq * MR.cc, eQ = wq * eta;
                    body_contact(sel(own_trunk, eta, eQ), sel(own_trunk, cP, cQ), selv(own_trunk, cl, lq),
                                 selv(own_trunk, nP, nlq), selv(own_trunk, FP, wq * FQ), dt, Q, rb);
                    body_contact(sel(own_trunk, eQ, eta), sel(own_trunk, cQ, cP), selv(own_trunk, lq, cl),
                                 selv(own_trunk, nlq, nP), selv(own_trunk, wq * FQ, FP), dt, Qb, rbx);
                }
            }
        }
        constexpr int NV = n_summed<SCENE>();
        {
            S v[NV];
#pragma unroll
            for (int i = 0; i < 21; ++i) v[i] = Q[i];
#pragma unroll
            for (int i = 0; i < 6; ++i) v[21 + i] = rb[i];
            v[27] = sel(keep, t2, S(0));
            if constexpr (SCENE == 3) {
#pragma unroll
                for (int i = 0; i < 21; ++i) v[28 + i] = Qb[i];
#pragma unroll
                for (int i = 0; i < 6; ++i) v[49 + i] = rbx[i];
            }
#pragma unroll
            for (int e = 0; e < NV; ++e) red[e * kPitch + g] = v[e];
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < (NV + 15) / 16; ++m) {
            const int e = g + 16 * m;
            if (e < NV) sred[e] = sum16(red + e * kPitch);
        }
        __syncthreads();
    }

    // ---- the body's system: sums, own inertia, mass, gyroscopic and gravity bias; one 6x6
    // solve per lane: the trunk's, in the pushing scene on odd lanes the box's
    tau2 = R(sred[27]);
    const bool odd = SCENE == 3 && (g & 1) != 0;
    {
        const S* s = sred + (odd ? 28 : 0);
#pragma unroll
        for (int i = 0; i < 21; ++i) Q[i] = s[i];
#pragma unroll
        for (int i = 0; i < 6; ++i) rb[i] = s[21 + i];
        V3<S> I = v3(MS.I0x, MS.I0y, MS.I0z), wo = ws, go = gbs;
        S mo = MS.m0, mt = MS.mtot;
        if constexpr (SCENE == 3) {
            I = selv(odd, v3(MS.bx_Ix, MS.bx_Iy, MS.bx_Iz), I);
            wo = selv(odd, cv<S>(bx.w), ws);
            go = selv(odd, cv<S>((-MR.g) * v3(bf.Rb.m[6], bf.Rb.m[7], bf.Rb.m[8])), gbs);
            mo = sel(odd, MS.bx_m, mo);
            mt = sel(odd, MS.bx_m, mt);
        }
        Q[s6(0, 0)] += I.x; Q[s6(1, 1)] += I.y; Q[s6(2, 2)] += I.z;
        Q[s6(3, 3)] += mt; Q[s6(4, 4)] += mt; Q[s6(5, 5)] += mt;
        const V3<S> gy = cross(wo, v3(I.x * wo.x, I.y * wo.y, I.z * wo.z));
        rb[0] -= dt * gy.x; rb[1] -= dt * gy.y; rb[2] -= dt * gy.z;
        rb[3] += dt * mo * go.x; rb[4] += dt * mo * go.y; rb[5] += dt * mo * go.z;
    }
    body_solve(Q, rb);  // rb <- the body's increment [d omega; d v_b]
    [[maybe_unused]] S rbx[6];
    if constexpr (SCENE == 3) {
        // lanes 0 and 1 of every quad hold the trunk's and the box's increments
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            rbx[i] = dpp<0x55>(rb[i]);
            rb[i] = dpp<0x00>(rb[i]);
        }
    }

    // ---- back-substitute the leg and integrate (semi-implicit Euler): velocities add the
    // increments in S, positions take dt times the new velocities in R.  The columns come from
    // their lanes: in FP32 one after the other (the order of the terms is the rounding), in
    // FP64 each lane adds its two and the quad adds the lanes.
    S dq[3];
    if constexpr (sizeof(S) == 4) {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            dq[j] = dpp<0xAA>(W1[j]);
            dq[j] -= dpp<0x00>(W0[j]) * rb[0];
            dq[j] -= dpp<0x55>(W0[j]) * rb[1];
            dq[j] -= dpp<0xAA>(W0[j]) * rb[2];
            dq[j] -= dpp<0xFF>(W0[j]) * rb[3];
            dq[j] -= dpp<0x00>(W1[j]) * rb[4];
            dq[j] -= dpp<0x55>(W1[j]) * rb[5];
        }
    } else {
        const S x0 = sel(sub2, sel(sub1, rb[3], rb[2]), sel(sub1, rb[1], rb[0]));
        const S x1 = sel(sub2, sel(sub1, S(0), S(-1)), sel(sub1, rb[5], rb[4]));
#pragma unroll
        for (int j = 0; j < 3; ++j) dq[j] = -quad_sum(W0[j] * x0 + W1[j] * x1);
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        lg.qd[j] = R(S(lg.qd[j]) + dq[j]);
        lg.q[j] += dtr * lg.qd[j];
    }
    M33<S> Rs;
#pragma unroll
    for (int i = 0; i < 9; ++i) Rs.m[i] = S(Rm.m[i]);
    b.w = cv<R>(ws + v3(rb[0], rb[1], rb[2]));
    if constexpr (SCENE == 3) b.vw = cv<R>(cv<S>(b.vw) + mul_ordered(Rs, v3(rb[3], rb[4], rb[5])));
    else b.vw = cv<R>(cv<S>(b.vw) + mul(Rs, v3(rb[3], rb[4], rb[5])));
    b.p = b.p + dtr * b.vw;
    if constexpr (SCENE != 3) {
        quat_step(b.qw, b.qx, b.qy, b.qz, b.w, dtr);
    } else {
        M33<S> Rbs;
#pragma unroll
        for (int i = 0; i < 9; ++i) Rbs.m[i] = S(bf.Rb.m[i]);
        bx.w = cv<R>(cv<S>(bx.w) + v3(rbx[0], rbx[1], rbx[2]));
        bx.vw = cv<R>(cv<S>(bx.vw) + mul_ordered(Rbs, v3(rbx[3], rbx[4], rbx[5])));
        bx.p = bx.p + dtr * bx.vw;
        // one quaternion step per lane: the trunk's on even lanes, the box's on odd lanes
        R q[4] = {sel(odd, bx.qw, b.qw), sel(odd, bx.qx, b.qx), sel(odd, bx.qy, b.qy), sel(odd, bx.qz, b.qz)};
        const V3<R> ph = (R(0.5) * dtr) * selv(odd, bx.w, b.w);
        // in a stated order (see mul_ordered)
        quat_turn(q[0], q[1], q[2], q[3], ph, m_sqrt(R(fma(ph.z, ph.z, fma(ph.y, ph.y, ph.x * ph.x)))));
        b.qw = dpp<0x00>(q[0]); b.qx = dpp<0x00>(q[1]); b.qy = dpp<0x00>(q[2]); b.qz = dpp<0x00>(q[3]);
        bx.qw = dpp<0x55>(q[0]); bx.qx = dpp<0x55>(q[1]); bx.qy = dpp<0x55>(q[2]); bx.qz = dpp<0x55>(q[3]);
    }
}

// ------------------------------------------------------------------------------
// The step in FP64: the same lanes, sums and discretisation as step16, arranged for fewer
// instructions (a step's time on a SIMD with one wave is its instruction stream):
//   * the leg is written in its own frame (mppi_step64.h), with divisions, square roots and
//     elementary functions without branches;
//   * lane `sub` of a leg eliminates two columns of the trunk's system, sub and sub + 4 (the
//     fifth and sixth velocity, the right side, and a zero column); the back-substitution adds
//     the four lanes' parts;
//   * the leg's own terms and the eliminated parts go to the sum from where they are: one
//     lane writes a leg's 28 values, each lane its two columns, so lane g adds 4 legs;
//   * corner contacts of the trunk are rare (a fallen robot, the box against the trunk):
//     their 16-lane sum runs only in steps in which some lane of the wave has one, and the
//     tests of trunk against box only while their bounding spheres overlap;
//   * in the pushing scene each lane reads the sums of the one body whose 6x6 system it solves.
// Per call, step16 with all columns in every lane / here (MI355X): heightfield walk K = 1024, H = 50: 318 / 197 us; box push
// K = 4096, H = 60: 560 / 343 us; flat walk K = 64, H = 25, whole control step: 135 / 96 us.
// ------------------------------------------------------------------------------
// the model in LDS through an offset (always zero) that the compiler takes to depend on the
// step's number, so that a step reads its constants where it uses them instead of keeping
// about 35 doubles in registers over the whole step loop
__device__ __forceinline__ const ModelT<double>& fresh_model(const ModelT<double>* m, int k)
{
    int o = 0;
#if defined(__HIP_DEVICE_COMPILE__)
    asm("" : "+v"(o) : "s"(k));
#endif
    return m[o];
}

template <int SCENE>
__device__ __forceinline__ void step16_64(int k, const ModelT<double>& M, const float* __restrict__ hf, double dt,
                                          double kp, double kd, int g, int eo0, int eo1, Base<double>& b,
                                          Leg<double>& lg, BoxS<double>& bx, double uj, double* red, double* sred, double& tau2)
{
    using namespace f64;
    const int leg = g >> 2, sub = g & 3;
    const bool sub1 = (sub & 1) != 0, sub2 = (sub & 2) != 0;
    const M33<double> Rm = quat_R(b.qw, b.qx, b.qy, b.qz);
    const V3<double> w = b.w;
    const V3<double> vb = mulT(Rm, b.vw);
    const V3<double> zero = v3(0.0, 0.0, 0.0), up = v3(0.0, 0.0, 1.0);
    [[maybe_unused]] M33<double> Rb;
    if constexpr (SCENE == 3) Rb = quat_R(bx.qw, bx.qx, bx.qy, bx.qz);

    // lane `sub` evaluates angle sub of the leg; one beyond the range of sincos64 is brought into
    // it where the step branches for its rare contacts
    double ang = (sub == 0) ? lg.q[0] : (sub == 1) ? lg.q[1] : lg.q[1] + lg.q[2];
    const bool far = is_far(ang);

    // ---- trunk corner g (g < 8) or box corner g - 8 (g >= 8), first, so that their terms leave
    // the registers before the leg's: the trunk's through a sum of their own where there are
    // any, the box's as rows of the sum below
    double c0 = 0.0, c1 = 0.0;  // the trunk corners' part of the values this lane sums
    {
        double Qc[21], rc[6];
#pragma unroll
        for (int i = 0; i < 21; ++i) Qc[i] = 0.0;
#pragma unroll
        for (int i = 0; i < 6; ++i) rc[i] = 0.0;
        bool corner;
        V3<double> F;
        double eta;
        if constexpr (SCENE != 3) {
            const V3<double> rloc = v3((g & 1 ? 0.5 : -0.5) * M.tsx, (g & 2 ? 0.5 : -0.5) * M.tsy,
                                       (g & 4 ? 0.5 : -0.5) * M.tsz);
            const V3<double> pw = b.p + mul(Rm, rloc);
            double dT, dB = 0.0;
            V3<double> nT, nB = zero;
            const bool hitT = terrain64<SCENE>(M, hf, pw, 0.0, dT, nT) && g < 8;
            bool hitB = false;
            if constexpr (SCENE == 2)
                hitB = point_aabox(pw - v3(M.sb_cx, M.sb_cy, M.sb_cz), v3(M.sb_hx, M.sb_hy, M.sb_hz), dB, nB) && g < 8;
            corner = __builtin_amdgcn_ballot_w64(hitT || hitB || far) != 0;
            if (corner) {
                const V3<double> vc = vb + cross(w, rloc);
                if (hitT) {
                    const V3<double> n = mulT(Rm, nT);
                    contact_law64(fresh_table<3>(k), M, dT, n, vc, F, eta);
                    base_contact_folded(eta, M.cc, rloc, n, F, dt, Qc, rc);
                }
                if (hitB) {
                    const V3<double> n = mulT(Rm, nB);
                    contact_law64(fresh_table<3>(k), M, dB, n, vc, F, eta);
                    base_contact_folded(eta, M.cc, rloc, n, F, dt, Qc, rc);
                }
            }
        } else {
            const bool own_trunk = g < 8;
            const int ci = g & 7;
            const V3<double> th = v3(0.5 * M.tsx, 0.5 * M.tsy, 0.5 * M.tsz), bh = v3(M.bx_hx, M.bx_hy, M.bx_hz);
            const V3<double> hP = selv(own_trunk, th, bh);
            const V3<double> cl = v3(ci & 1 ? hP.x : -hP.x, ci & 2 ? hP.y : -hP.y, ci & 4 ? hP.z : -hP.z);
            const V3<double> x = selv(own_trunk, b.p + mul(Rm, cl), bx.p + mul(Rb, cl));
            const double dG = -x.z;  // the corner against the ground
            const bool hitG = dG > 0.0;
            // the corner inside the other body, only while the bounding spheres can overlap
            bool hitP = false;
            double dP = 0.0;
            V3<double> lq = zero, nlq = zero;
            const V3<double> dc = b.p - bx.p;
            if (__builtin_amdgcn_ballot_w64(dot(dc, dc) <= kNear * (dot(th, th) + dot(bh, bh)))) {
                lq = selv(own_trunk, mulT(Rb, x - bx.p), mulT(Rm, x - b.p));
                hitP = point_aabox(lq, selv(own_trunk, bh, th), dP, nlq);
            }
            double Qb[21], rbx[6];
#pragma unroll
            for (int i = 0; i < 21; ++i) Qb[i] = 0.0;
#pragma unroll
            for (int i = 0; i < 6; ++i) rbx[i] = 0.0;
            // the box's corners against the ground
            if (__builtin_amdgcn_ballot_w64(hitG && !own_trunk)) {
                const double wgt = hitG && !own_trunk ? 1.0 : 0.0;
                const V3<double> n = v3(Rb.m[6], Rb.m[7], Rb.m[8]);  // up, box frame
                const V3<double> vc = mulT(Rb, bx.vw) + cross(bx.w, cl);
                contact_law64(fresh_table<3>(k), M, wgt * dG, n, wgt * vc, F, eta);
                base_contact_folded(wgt * eta, wgt * M.cc, cl, n, wgt * F, dt, Qb, rbx);
            }
            // rare: the trunk's corners against the ground, and either body's in the other
            corner = __builtin_amdgcn_ballot_w64(hitP || (hitG && own_trunk) || far) != 0;
            if (__builtin_expect(corner, 0)) {  // out of the step's straight way
                const V3<double> lt = own_trunk ? cl : mulT(Rm, x - b.p), lb = own_trunk ? mulT(Rb, x - bx.p) : cl;
                const V3<double> vtr = b.vw + mul(Rm, cross(w, lt)), vbx = bx.vw + mul(Rb, cross(bx.w, lb));
                if (hitG && own_trunk) {
                    const V3<double> n = v3(Rm.m[6], Rm.m[7], Rm.m[8]);
                    contact_law64(fresh_table<3>(k), M, dG, n, mulT(Rm, vtr), F, eta);
                    base_contact_folded(eta, M.cc, lt, n, F, dt, Qc, rc);
                }
                if (hitP) {
                    // force +F on the corner's body, -F on the other
                    const V3<double> n = selv(own_trunk, mul(Rb, nlq), mul(Rm, nlq));
                    contact_law64(fresh_table<3>(k), M, dP, n, selv(own_trunk, vtr - vbx, vbx - vtr), F, eta);
                    const double st = own_trunk ? 1.0 : -1.0;
                    base_contact_folded(eta, M.cc, lt, mulT(Rm, n), st * mulT(Rm, F), dt, Qc, rc);
                    base_contact_folded(eta, M.cc, lb, mulT(Rb, n), (-st) * mulT(Rb, F), dt, Qb, rbx);
                }
            }
#pragma unroll
            for (int e = 0; e < 21; ++e) red[kBoxRow + e * kPitch + g] = Qb[e];
#pragma unroll
            for (int e = 0; e < 6; ++e) red[kBoxRow + (21 + e) * kPitch + g] = rbx[e];
        }
        if (__builtin_expect(corner, 0)) {
            if (far) ang = near_angle(fresh_table<0>(k), ang);
#pragma unroll
            for (int e = 0; e < 21; ++e) red[e * kPitch + g] = Qc[e];
#pragma unroll
            for (int e = 0; e < 6; ++e) red[(21 + e) * kPitch + g] = rc[e];
            __syncthreads();
            c0 = sum16(red + g * kPitch);
            c1 = sel(g < 11, sum16(red + min(g + 16, 26) * kPitch), 0.0);
            __syncthreads();
        }
    }

    // ---- the leg: torques, kinematics, mass-matrix and bias terms
    const double u[3] = {dpp<0x00>(uj), dpp<0x55>(uj), dpp<0xAA>(uj)};
    double tau[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) tau[j] = kp * (u[j] - lg.q[j]) - kd * lg.qd[j];
    const V3<double> gb = (-M.g) * v3(Rm.m[6], Rm.m[7], Rm.m[8]);
    LegFrame G;
    LegRows S;
    {
        double Q[21], rb[6];
        double sn, cs;
        sincos64(fresh_table<0>(k), ang, &sn, &cs);
        leg_terms(M, leg, dpp<0x00>(sn), dpp<0x00>(cs), dpp<0x55>(sn), dpp<0x55>(cs), dpp<0xAA>(sn), dpp<0xAA>(cs),
                  lg.qd, tau, dt, dt * kd, w, vb, gb, G, S, Q, rb);

        // its foot against terrain and the static or free box: the first contact (terrain if
        // touched, else the box) in line, with zero weight where there is none; the second
        // (a foot that touches both) and the box's share in blocks that are rarely entered
        const V3<double> pfw = b.p + mul(Rm, foot_trunk(G));
        double dT, dB = 0.0;
        V3<double> nT, nB = zero;
        const bool hitT = terrain64<SCENE>(M, hf, pfw, M.foot_r, dT, nT);
        bool hitB = false;
        if constexpr (SCENE == 2)
            hitB = sphere_aabox64(pfw - v3(M.sb_cx, M.sb_cy, M.sb_cz), M.foot_r, v3(M.sb_hx, M.sb_hy, M.sb_hz), dB, nB);
        if constexpr (SCENE == 3) {
            // outside the sphere around the box there is no contact
            const V3<double> d = pfw - bx.p;
            const V3<double> bh = v3(M.bx_hx, M.bx_hy, M.bx_hz);
            if (__builtin_amdgcn_ballot_w64(dot(d, d) <= kNear * (M.foot_r * M.foot_r + dot(bh, bh)))) {
                V3<double> nl = up;
                hitB = sphere_aabox64(mulT(Rb, d), M.foot_r, bh, dB, nl);
                nB = mul(Rb, nl);  // box -> foot (world)
            }
        }
        // the box at the contact point: its velocity there, and its share of the contact added
        // to this lane's row of the box's sum (once per leg)
        [[maybe_unused]] auto box_velocity = [&](V3<double> nw) {
            return mulT(Rm, bx.vw + mul(Rb, cross(bx.w, mulT(Rb, pfw - M.foot_r * nw - bx.p))));
        };
        [[maybe_unused]] auto box_share = [&](double wgt, V3<double> nw, V3<double> F, double eta) {
            double Qf[21], rf[6];
#pragma unroll
            for (int i = 0; i < 21; ++i) Qf[i] = 0.0;
#pragma unroll
            for (int i = 0; i < 6; ++i) rf[i] = 0.0;
            const double wb = sub == 0 ? wgt : 0.0;
            base_contact_folded(wb * eta, wb * M.cc, mulT(Rb, pfw - M.foot_r * nw - bx.p), mulT(Rb, nw),
                       mulT(Rb, (-wb) * mul(Rm, F)), dt, Qf, rf);
#pragma unroll
            for (int e = 0; e < 21; ++e) red[kBoxRow + e * kPitch + g] += Qf[e];
#pragma unroll
            for (int e = 0; e < 6; ++e) red[kBoxRow + (21 + e) * kPitch + g] += rf[e];
        };
        V3<double> F;
        double eta;
        {
            const bool on = hitT || hitB, isB = !hitT && hitB;
            const double wgt = on ? 1.0 : 0.0;
            V3<double> n, vo = zero;
            if constexpr (SCENE == 0) {
                n = v3(Rm.m[6], Rm.m[7], Rm.m[8]);
                foot_contact(fresh_table<1>(k), M, G, on ? dT : 0.0, n, vo, dt, wgt, S, Q, rb, F, eta);
            } else {
                const V3<double> nw = isB ? nB : nT;
                if constexpr (SCENE == 3) {
                    if (__builtin_amdgcn_ballot_w64(isB)) vo = selv(isB, box_velocity(nw), zero);
                }
                n = mulT(Rm, nw);
                foot_contact(fresh_table<1>(k), M, G, on ? (isB ? dB : dT) : 0.0, n, vo, dt, wgt, S, Q, rb, F, eta);
                if constexpr (SCENE == 3) {
                    if (__builtin_amdgcn_ballot_w64(isB)) box_share(isB ? 1.0 : 0.0, nw, F, eta);
                }
            }
        }
        // the leg's values to the sum
        double* o = red + leg * kLegPitch;
        if (sub == 0) {
#pragma unroll
            for (int e = 0; e < 21; ++e) o[e] = Q[e];
#pragma unroll
            for (int e = 0; e < 6; ++e) o[21 + e] = rb[e];
            o[27] = tau[0] * tau[0] + tau[1] * tau[1] + tau[2] * tau[2];
        }
        if constexpr (SCENE == 2 || SCENE == 3) {
            const bool both = hitT && hitB;
            if (__builtin_amdgcn_ballot_w64(both)) {
                const double wgt = both ? 1.0 : 0.0;
                const V3<double> nw = both ? nB : up;
                V3<double> vo = zero;
                if constexpr (SCENE == 3) vo = selv(both, box_velocity(nw), zero);
#pragma unroll
                for (int i = 0; i < 21; ++i) Q[i] = 0.0;
#pragma unroll
                for (int i = 0; i < 6; ++i) rb[i] = 0.0;
                foot_contact(fresh_table<1>(k), M, G, both ? dB : 0.0, mulT(Rm, nw), vo, dt, wgt, S, Q, rb, F, eta);
                if (sub == 0) {
#pragma unroll
                    for (int e = 0; e < 21; ++e) o[e] += Q[e];
#pragma unroll
                    for (int e = 0; e < 6; ++e) o[21 + e] += rb[e];
                }
                if constexpr (SCENE == 3) box_share(wgt, nw, F, eta);
            }
        }
    }

    // ---- its elimination: lane `sub` solves columns sub and sub + 4
    double W0[3], W1[3];
    {
        double C[3][6];
        rows_to_trunk(G, S, C);
        const Ldl3 f3 = ldl3(S.A00, S.A01, S.A11, S.A02, S.A12, S.A22);
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            W0[j] = sel(sub2, sel(sub1, C[j][3], C[j][2]), sel(sub1, C[j][1], C[j][0]));
            W1[j] = sel(sub2, sel(sub1, 0.0, S.rl[j]), sel(sub1, C[j][5], C[j][4]));
        }
        f64::solve3(f3, W0[0], W0[1], W0[2]);
        f64::solve3(f3, W1[0], W1[1], W1[2]);
        double* o = red + kElimRow + leg * kElimPitch + sub;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            if (i < 4) o[8 * i] = C[0][i] * W0[0] + C[1][i] * W0[1] + C[2][i] * W0[2];
            o[8 * i + 4] = C[0][i] * W1[0] + C[1][i] * W1[1] + C[2][i] * W1[2];
        }
    }
    __syncthreads();
    {
        const double* v = red + g;
        const double* x = red + kElimRow;
        double s0 = c0, s1 = c1;
        // every lane reads (lanes past the last value a valid one, unused), so that the reads
        // wait together
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            s0 += v[l * kLegPitch] - x[l * kElimPitch + eo0];
            s1 += v[l * kLegPitch + 16] - x[l * kElimPitch + eo1];
        }
        [[maybe_unused]] double b0, b1;
        if constexpr (SCENE == 3) {
            b0 = sum16(red + kBoxRow + g * kPitch);
            b1 = sum16(red + kBoxRow + min(g + 16, 26) * kPitch);
            sred[28 + g] = b0;
        }
        sred[g] = s0;
        if (g < 12) {
            sred[g + 16] = s1;
            if constexpr (SCENE == 3) sred[28 + 16 + g] = b1;  // the twelfth to a place that is not read
        }
    }
    __syncthreads();

    // ---- the body's system: sums, own inertia, mass, gyroscopic and gravity bias; one 6x6
    // solve per lane (the trunk's, on odd lanes of the pushing scene the box's)
    tau2 = sred[27];
    const bool odd = SCENE == 3 && sub1;
    double dv[6];
    {
        double Q[21];
        const double* s = sred + (odd ? 28 : 0);
#pragma unroll
        for (int i = 0; i < 21; ++i) Q[i] = s[i];
#pragma unroll
        for (int i = 0; i < 6; ++i) dv[i] = s[21 + i];
        V3<double> I = v3(M.I0x, M.I0y, M.I0z), It = v3(M.tr_Ix, M.tr_Iy, M.tr_Iz), wo = w, go = gb;
        double m0 = M.m0, mt = M.mtot;
        if constexpr (SCENE == 3) {
            const V3<double> Ib = v3(M.bx_Ix, M.bx_Iy, M.bx_Iz);
            I = selv(odd, Ib, I);
            It = selv(odd, Ib, It);
            m0 = sel(odd, M.bx_m, m0);
            mt = sel(odd, M.bx_m, mt);
            wo = selv(odd, bx.w, w);
            go = selv(odd, (-M.g) * v3(Rb.m[6], Rb.m[7], Rb.m[8]), gb);
        }
        Q[s6(0, 0)] += It.x; Q[s6(1, 1)] += It.y; Q[s6(2, 2)] += It.z;
        Q[s6(3, 3)] += mt; Q[s6(4, 4)] += mt; Q[s6(5, 5)] += mt;
        const V3<double> gy = cross(wo, v3(I.x * wo.x, I.y * wo.y, I.z * wo.z));
        const double dm = dt * m0;
        dv[0] -= dt * gy.x; dv[1] -= dt * gy.y; dv[2] -= dt * gy.z;
        dv[3] += dm * go.x; dv[4] += dm * go.y; dv[5] += dm * go.z;
        ldl6_solve(Q, dv);
    }
    [[maybe_unused]] double db[6];
    if constexpr (SCENE == 3) {
        // lanes 0 and 1 of every quad hold the trunk's and the box's increments
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            db[i] = dpp<0x55>(dv[i]);
            dv[i] = dpp<0x00>(dv[i]);
        }
    }

    // ---- back-substitute the leg (each lane its two columns, added over the quad) and integrate
    {
        const double x0 = sel(sub2, sel(sub1, dv[3], dv[2]), sel(sub1, dv[1], dv[0]));
        const double x1 = sel(sub2, sel(sub1, 0.0, -1.0), sel(sub1, dv[5], dv[4]));
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            lg.qd[j] -= quad_sum(W0[j] * x0 + W1[j] * x1);
            lg.q[j] += dt * lg.qd[j];
        }
    }
    b.w = w + v3(dv[0], dv[1], dv[2]);
    b.vw = b.vw + mul(Rm, v3(dv[3], dv[4], dv[5]));
    b.p = b.p + dt * b.vw;
    if constexpr (SCENE != 3) {
        quat_step64(fresh_table<2>(k), b.qw, b.qx, b.qy, b.qz, b.w, dt);
    } else {
        bx.w = bx.w + v3(db[0], db[1], db[2]);
        bx.vw = bx.vw + mul(Rb, v3(db[3], db[4], db[5]));
        bx.p = bx.p + dt * bx.vw;
        // one quaternion step per lane: the trunk's on even lanes, the box's on odd lanes
        double q[4] = {sel(odd, bx.qw, b.qw), sel(odd, bx.qx, b.qx), sel(odd, bx.qy, b.qy), sel(odd, bx.qz, b.qz)};
        quat_step64(fresh_table<2>(k), q[0], q[1], q[2], q[3], selv(odd, bx.w, b.w), dt);
        b.qw = dpp<0x00>(q[0]); b.qx = dpp<0x00>(q[1]); b.qy = dpp<0x00>(q[2]); b.qz = dpp<0x00>(q[3]);
        bx.qw = dpp<0x55>(q[0]); bx.qx = dpp<0x55>(q[1]); bx.qy = dpp<0x55>(q[2]); bx.qz = dpp<0x55>(q[3]);
    }
}

}  // namespace r16

// ------------------------------------------------------------------------------
// rollout kernel: workgroup of 64 lanes = 4 samples x 16 lanes.  R: geometry and state
// type, S: system type (FP32/FP32, FP64/FP64, or FP32 geometry with the FP64 system).
// LDS: the summation rows [4][NV][kPitch] (NV summed values of the scene) and sums
// [4][kSumPitch] (type S), then the heightfield (scene 1).  eps addressing as in the quad kernel: eps_in[n * eps_sn + d *
// eps_sd] when given, otherwise Philox noise stored to eps_out[d * K + n].  DIRECT: one
// value per control step (the direct representation, whose noise is drawn inside the step
// loop; the `direct` argument equals it); a separate instantiation, so that the knot
// representations carry no per-step sampling code and its registers in their step loop.
// ------------------------------------------------------------------------------
template <int SCENE, typename R, typename S, bool DIRECT>
__global__ __launch_bounds__(64) void rollout16_kernel(ModelT<R> Mr, ModelT<S> Ms, DevParams P,
                                                       const double* __restrict__ gB,
                                                       const float* __restrict__ ghf, const float* __restrict__ mu,
                                                       const float* __restrict__ x0,
                                                       const float* __restrict__ eps_in, int eps_sn, int eps_sd,
                                                       float* __restrict__ eps_out, float* __restrict__ costs,
                                                       float* __restrict__ traj, int direct,
                                                       const int* __restrict__ skip, int* __restrict__ input_status)
{
    // a plain fallback rollout whose proposal the gate took: nothing to do
    if (skip && skip[0]) return;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    // the model's constants are read from LDS (values in vector registers), which keeps the
    // scalar registers for the kernel's pointers and loop state
    __shared__ ModelT<R> sMr;
    __shared__ ModelT<S> sMs;
    constexpr int NV = r16::n_summed<SCENE>();
    S* red = reinterpret_cast<S*>(lds_raw);
    S* sred = red + r16::kSamples * NV * r16::kPitch;
    float* sHF = reinterpret_cast<float*>(sred + r16::kSamples * r16::kSumPitch);
    if (threadIdx.x == 0) {
        sMr = Mr;
        sMs = Ms;
    }
    if constexpr (SCENE == 1) {
        // 16 bytes a lane and several loads in flight (both sides are 16-byte aligned): one
        // value at a time, the 64 x 64 field took 64 round trips
        const int cells = Mr.hf_nx * Mr.hf_ny, quads = cells >> 2;
        const r16::Quad* __restrict__ src = reinterpret_cast<const r16::Quad*>(ghf);
        r16::Quad* dst = reinterpret_cast<r16::Quad*>(sHF);
#pragma unroll 8
        for (int i = threadIdx.x; i < quads; i += 64) dst[i] = src[i];
        for (int i = 4 * quads + threadIdx.x; i < cells; i += 64) sHF[i] = ghf[i];
    }
    __syncthreads();
    const ModelT<R>& MR = sMr;
    const ModelT<S>& MS = sMs;

    const int tid = threadIdx.x;
    const int g = tid & 15, grp = tid >> 4;
    const int leg = g >> 2, sub = g & 3;
    const int jl = sub < 3 ? sub : 2;  // this lane's joint of its leg
    const int n = blockIdx.x * r16::kSamples + grp;
    const bool valid = n < P.K;
    const int ns = valid ? n : P.K - 1;
    const int nk = P.nk;
    const R sigma = P.sigma;

    // knots of this lane's joint, theta = mu + sigma eps (sample 0 is the nominal); the
    // direct representation draws one value per step inside the step loop instead
    R th[kMaxKnots];
#pragma unroll
    for (int i = 0; i < kMaxKnots; ++i) {
        th[i] = R(0);
        if (!DIRECT && i < nk) {
            const int d = (3 * leg + jl) * nk + i;
            R e;
            if (eps_in) {
                e = eps_in[(size_t)ns * eps_sn + (size_t)d * eps_sd];
            } else {
                e = gauss_elem<R>(P, (uint32_t)ns, (uint32_t)d);
                if (valid && sub < 3 && eps_out) eps_out[(size_t)d * P.K + n] = (float)e;
            }
            th[i] = R(mu[d]) + (ns ? sigma * e : R(0));
        }
    }

    // a start state that is not finite: no rollout, every cost +inf, and the flag set
    {
        bool bad = false;
        for (int i = tid; i < P.nx; i += 64) bad |= !(fabsf(x0[i]) <= 3.0e38f);
        const bool any_bad = __builtin_amdgcn_ballot_w64(bad) != 0;
        if (input_status && blockIdx.x == 0 && tid == 0) input_status[0] = any_bad ? 1 : 0;
        if (any_bad) {
            if (valid && g == 0) costs[n] = __int_as_float(0x7f800000);
            return;
        }
    }
    Base<R> b;
    Leg<R> lg;
    BoxS<R> bx{};
    load_state(x0, leg, b, lg);
    if constexpr (SCENE == 3) load_box(x0, bx);
    float* tr = (traj && valid && sub == 0) ? traj + (size_t)n * (P.H + 1) * P.nx : nullptr;
    if (tr) {
        store_state(tr, leg, b, lg);
        if (SCENE == 3 && leg == 0) store_box(tr, bx);
    }

    S* my_red = red + grp * NV * r16::kPitch;
    S* my_sum = sred + grp * r16::kSumPitch;
    const S dt = P.dt, kp = P.kp, kd = P.kd;
    // the spline basis' row of the coming step, read before the cost of the last one: its
    // scalar loads make one round trip to memory together and behind that work, where reading
    // them knot by knot at their use made one after the other
    [[maybe_unused]] double brow[kMaxKnots];
    if constexpr (!DIRECT) {
#pragma unroll
        for (int i = 0; i < kMaxKnots; ++i) brow[i] = gB[min(i, nk - 1)];
    }
    [[maybe_unused]] const int eo0 = r16::elim_slot(g), eo1 = r16::elim_slot(g + 16);
    R L = R(0);
    for (int k = 0; k < P.H; ++k) {
        R uj = R(0);
        if constexpr (DIRECT) {
            // value k of this lane's joint (nk == H): theta = mu + sigma eps
            const int d = (3 * leg + jl) * nk + k;
            R e;
            if (eps_in) {
                e = eps_in[(size_t)ns * eps_sn + (size_t)d * eps_sd];
            } else {
                e = gauss_elem<R>(P, (uint32_t)ns, (uint32_t)d);
                if (valid && sub < 3 && eps_out) eps_out[(size_t)d * P.K + n] = (float)e;
            }
            uj = R(mu[d]) + (ns ? sigma * e : R(0));
        } else {
            // every term (those past the last knot are zero), from the row read a step ago
#pragma unroll
            for (int i = 0; i < kMaxKnots; ++i) uj += R(brow[i]) * th[i];
        }
        R tau2;
        if constexpr (sizeof(R) == 8)
            r16::step16_64<SCENE>(k, r16::fresh_model(&sMs, k), sHF, dt, kp, kd, g, eo0, eo1, b, lg, bx, uj, my_red,
                                  my_sum, tau2);
        else
            r16::step16<SCENE, R, S>(MR, MS, sHF, dt, kp, kd, g, eo0, eo1, b, lg, bx, uj, my_red, my_sum,
                                        tau2);
        if constexpr (!DIRECT) {
            const double* nrow = gB + min(k + 1, P.H - 1) * nk;
#pragma unroll
            for (int i = 0; i < kMaxKnots; ++i) brow[i] = nrow[min(i, nk - 1)];
        }
        round_state(b, lg);
        if constexpr (SCENE == 3) round_box(bx);
        L += R(dt) * stage_cost<SCENE>(P, b, bx, tau2);
        if (tr) {
            store_state(tr + (size_t)(k + 1) * P.nx, leg, b, lg);
            if (SCENE == 3 && leg == 0) store_box(tr + (size_t)(k + 1) * P.nx, bx);
        }
    }
    float Lf = (float)L;
    if (!(fabsf(Lf) <= 3.0e38f)) Lf = __int_as_float(0x7f800000);  // non-finite -> +inf
    if (valid && g == 0) costs[n] = Lf;
}

namespace r16 {

template <typename S>
size_t lds_bytes(int scene, int hf_cells)
{
    const size_t nv = scene == 3 ? 55 : 28;  // n_summed<scene>()
    size_t b = sizeof(S) * ((size_t)kSamples * nv * kPitch + (size_t)kSamples * kSumPitch);
    if (scene == 1) b += sizeof(float) * (size_t)hf_cells;
    return b;
}

template <typename R, typename S>
hipError_t launch_t(const ModelT<R>& Mr, const ModelT<S>& Ms, const DevParams& P, const RolloutArgs& a,
                    hipStream_t st)
{
    const int blocks = (P.K + kSamples - 1) / kSamples;
    const size_t lds = lds_bytes<S>(Mr.scene, Mr.hf_nx * Mr.hf_ny);
    if (lds > 65536) return hipErrorInvalidValue;
#define MPPI_LAUNCH_R16_D(SC, D)                                                                               \
    hipLaunchKernelGGL((rollout16_kernel<SC, R, S, D>), dim3(blocks), dim3(64), lds, st, Mr, Ms, P, a.B, a.hf,     \
                       a.mu, a.x0, a.eps_in, a.eps_sn, a.eps_sd, a.eps_out, a.costs, a.traj, a.direct, a.skip,     \
                       a.input_status)
#define MPPI_LAUNCH_R16(SC)          \
    if (a.direct)                    \
        MPPI_LAUNCH_R16_D(SC, true); \
    else                             \
        MPPI_LAUNCH_R16_D(SC, false)
    switch (Mr.scene) {
    case 0: MPPI_LAUNCH_R16(0); break;
    case 1: MPPI_LAUNCH_R16(1); break;
    case 2: MPPI_LAUNCH_R16(2); break;
    case 3: MPPI_LAUNCH_R16(3); break;
    default: return hipErrorInvalidValue;
    }
#undef MPPI_LAUNCH_R16
#undef MPPI_LAUNCH_R16_D
    return hipGetLastError();
}

}  // namespace r16

bool rollout16_fits(int arith, int scene, int hf_cells)
{
    const size_t b = arith == 1 ? r16::lds_bytes<float>(scene, hf_cells) : r16::lds_bytes<double>(scene, hf_cells);
    return b <= 65536;
}

// arith: 0 FP64, 1 FP32, 2 FP32 geometry with the FP64 implicit system
hipError_t launch_rollout16(const DevModelF& Mf, const DevModelD& Md, int arith, const DevParams& P,
                            const RolloutArgs& a, hipStream_t st)
{
    if (arith == 1) return r16::launch_t(Mf, Mf, P, a, st);
    if (arith == 2) return r16::launch_t(Mf, Md, P, a, st);
    return r16::launch_t(Md, Md, P, a, st);
}

}  // namespace mppi
