// Stage records of the two-launch discretize forms (classical RK4 in
// cis_split.hip, Runge-Kutta-Fehlberg in cis_rkf.hip): the nominal recursion
// with four intervals per wave, and what it leaves for the tangent columns
// (arxiv 2604.09993, Sec. IV-B eq. intg-aug-sys-param; sensitivities by
// internal numerical differentiation, Sec. VI).
//
// Structure used.  Joint forces are controls, so the translation of a body
// that carries no contact is driven by the controls alone, and on flat ground
// (fixed contact frame) so is that of every body: its rows of Z = [Phi_x | B- |
// B+] and its position and velocity columns are the same scalar RK solutions
// for every interval (1, s tau, and the responses to the two hold weights) up
// to factors s and 1/m, and they enter the rest of Z only through the integral
// rows, linearly.  What is left to integrate column by column are the angle
// rows (and, on a sinusoid, the feet's translation) for the columns that touch
// them: quad13 on flat ground 26 + 5 rows x 122 columns instead of 83 x 174.
// The integral rows' share of the translation is a weighted sum of their
// coefficients over the stages (PackRec::SUM), formed here on body lanes.
#pragma once
#include <hip/hip_runtime.h>

#include "cis_body.hpp"
#include "cis_model.hpp"

namespace cis {

// Layout of the workspace (elements of T), FLAT: flat ground.  An interval's
// part holds HDR constants and one record of STAGE elements per RK stage; the
// sums of all n intervals follow as SUM arrays of n elements, sum q of
// interval i at [q * n + i].
template <class TP, bool FLAT>
struct PackRec {
    static_assert(TP::L >= 1 && TP::D >= 1, "legs with links");
    static constexpr int NB = TP::NB, NJ = TP::NJ, NC = TP::NC, M = TP::M;
    // constants: s, h, 0 x6, 1/m, 1/I per body, per joint s k/I and s d/I of the
    // parent and -s k/I, -s d/I of the child
    static constexpr int MINV = 8, IINV = MINV + NB, KC = IINV + NB;
    static constexpr int NVK = (4 * NJ + 15) / 16;
    static constexpr int HDR = (KC + 16 * NVK + 7) / 8 * 8;
    // stage record: per body s dT/dth / I and the violation row's angle
    // coefficient, per foot the integral rows' and contact coefficients (field
    // f of foot i at FT + NFOOT i + f), then the forcing entries.  Coefficients
    // of the integral rows carry the RK weight of the stage.  The tangent lanes
    // read the first NV vectors of 16 elements (KC: NVK) lane by lane.
    static constexpr int CTH = 0, CV = NB, FT = 2 * NB;
    enum { F_CTH = 0, F_COM, F_CX, F_CY, F_CVX, F_CVY, F_XX, F_XT, F_YX, F_YT, F_TX, F_ZX, F_ZY };
    static constexpr int NFOOT = FLAT ? 2 : 13;
    static constexpr int NSC = FT + NFOOT * NC, NV = (NSC + 15) / 16;
    static constexpr int FORCE = (NSC + 1) / 2 * 2;
    // joint j, field f (parent x, parent y, child x, child y of the theta row) at
    // FORCE + f NJ + j; contact i, field f at CF + f NC + i: theta row by
    // lambda_n, t+, t- (flat), or rows x, y, theta by them (f = 3 row + control)
    static constexpr int CF = FORCE + 4 * NJ, NCF = FLAT ? 3 : 9;
    static constexpr int NF = 4 * NJ + NCF * NC;
    static constexpr int STAGE = (cmax(FORCE + NF, 16 * NV) + 7) / 8 * 8;
    // sums: violation row by the x and y translation of body b against {1, tau,
    // X-, X+}: RX + q NB + b; cross-complementarity row of foot i by its y
    // translation: EY + q NC + i, by its x velocity against {1, V-, V+}: EX, by its
    // y velocity: EV, by its own forces: GC + q NC + i; then zeros that are NaN
    // when an angle state, the violation row, or foot i's row (PZ + 2 + i) is not
    // finite
    static constexpr int RX = 0, RY = 4 * NB, EY = 8 * NB, EX = EY + 4 * NC, EV = EX + 3 * NC;
    static constexpr int GC = EV + NC, PZ = GC + 3 * NC, SUM = PZ + 2 + NC;
    static constexpr int64_t records(int K, int R) { return HDR + (int64_t)R * K * STAGE; }
    static constexpr int64_t per_interval(int K, int R) { return records(K, R) + SUM; }
};

// DPP inside rows of 16 lanes (one interval's bodies): lane N of the row.  In
// FP64 the broadcast is one 64-bit move, and a sum over lanes uses the FMA's DPP
// form with a factor 1 (a DPP operand needs two wait states after its write).
template <int N>
__device__ __forceinline__ float row_lane(float v) { return dpp_row<0x150 + N>(v); }
template <int N>
__device__ __forceinline__ double row_lane(double v) {
    double r;
    asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf"
        : "=v"(r) : "v"(v), "n"(N));
    return r;
}
// v at lanes A, B, C, D of the row, summed in this order (the first NL of them)
template <int NL, int A, int B, int C, int D>
__device__ __forceinline__ float row_sum_of(float v) {
    float t = row_lane<A>(v);
    if constexpr (NL > 1) t += row_lane<B>(v);
    if constexpr (NL > 2) t += row_lane<C>(v);
    if constexpr (NL > 3) t += row_lane<D>(v);
    return t;
}
template <int NL, int A, int B, int C, int D>
__device__ __forceinline__ double row_sum_of(double v) {
    static_assert(NL == 1 || NL == 2 || NL == 4, "one, two or four legs");
    if constexpr (NL == 1) return row_lane<A>(v);
    double t;
    const double one = 1.0;
    if constexpr (NL == 2)
        asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%3 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %0, %1, %2 row_newbcast:%4 row_mask:0xf bank_mask:0xf"
            : "=&v"(t) : "v"(v), "v"(one), "n"(A), "n"(B));
    if constexpr (NL == 4)
        asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%3 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %0, %1, %2 row_newbcast:%4 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %0, %1, %2 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %0, %1, %2 row_newbcast:%6 row_mask:0xf bank_mask:0xf"
            : "=&v"(t) : "v"(v), "v"(one), "n"(A), "n"(B), "n"(C), "n"(D));
    return t;
}
template <int N, class T>
__device__ __forceinline__ T row_ror(T v) { return dpp_row<0x120 + N>(v); }    // row_ror:N
template <class T>
__device__ __forceinline__ T row_sum(T v) {
    v += row_ror<8>(v);
    v += row_ror<4>(v);
    v += row_ror<2>(v);
    v += row_ror<1>(v);
    return v;
}

// the first N lanes of the row, in their order
template <int N, class T, int E = 1>
__device__ __forceinline__ T row_sum_first(T v, T acc) {
    if constexpr (E < N) return row_sum_first<N, T, E + 1>(v, acc + row_lane<E>(v));
    else return acc;
}
template <int N, class T>
__device__ __forceinline__ T row_sum_first(T v) { return row_sum_first<N, T>(v, row_lane<0>(v)); }

// A double constant in scalar registers, formed where it is used: as ordinary
// constants the compiler keeps the 22 coefficients of sin and cos in vector
// registers across the stage loop (44 of them) and spills others for it.
template <uint64_t BITS>
__device__ __forceinline__ double scalar_const() {
    int lo, hi;
    asm volatile("s_mov_b32 %0, %1" : "=s"(lo) : "i"((int)(uint32_t)BITS));
    asm volatile("s_mov_b32 %0, %1" : "=s"(hi) : "i"((int)(uint32_t)(BITS >> 32)));
    return __builtin_bit_cast(double, make_int2(lo, hi));
}
// sincos_t with the constants of sincos_cw (same arithmetic) in scalar registers
__device__ __forceinline__ void sincos_pack(double a, double* s, double* c) {
    if (__any(fabs(a) > 1e5)) {
        sincos(a, s, c);
        return;
    }
#define CIS_SC(V) scalar_const<__builtin_bit_cast(uint64_t, (double)(V))>()
    const double k = rint(a * CIS_SC(0.6366197723675814));
    double r = fma(-k, CIS_SC(1.570796325802803), a);
    r = fma(-k, CIS_SC(9.920935791635221e-10), r);
    r = fma(-k, CIS_SC(5.170182981794105e-19), r);
    const double z = r * r;
    double ps = CIS_SC(1.0 / 355687428096000.0);
    double pc = CIS_SC(-1.0 / 6402373705728000.0);
    ps = fma(ps, z, CIS_SC(-1.0 / 1307674368000.0));
    pc = fma(pc, z, CIS_SC(1.0 / 20922789888000.0));
    ps = fma(ps, z, CIS_SC(1.0 / 6227020800.0));
    pc = fma(pc, z, CIS_SC(-1.0 / 87178291200.0));
    ps = fma(ps, z, CIS_SC(-1.0 / 39916800.0));
    pc = fma(pc, z, CIS_SC(1.0 / 479001600.0));
    ps = fma(ps, z, CIS_SC(1.0 / 362880.0));
    pc = fma(pc, z, CIS_SC(-1.0 / 3628800.0));
    ps = fma(ps, z, CIS_SC(-1.0 / 5040.0));
    pc = fma(pc, z, CIS_SC(1.0 / 40320.0));
    ps = fma(ps, z, CIS_SC(1.0 / 120.0));
    pc = fma(pc, z, CIS_SC(-1.0 / 720.0));
    ps = fma(ps, z, CIS_SC(-1.0 / 6.0));
    pc = fma(pc, z, CIS_SC(1.0 / 24.0));
#undef CIS_SC
    const double sr = fma(r * z, ps, r);
    const double cr = fma(z * z, pc, fma(-0.5, z, 1.0));
    const int q = (int)k;
    const double s1 = (q & 1) ? cr : sr;
    const double c1 = (q & 1) ? sr : cr;
    *s = (q & 2) ? -s1 : s1;
    *c = ((q + 1) & 2) ? -c1 : c1;
}
__device__ __forceinline__ void sincos_pack(float a, float* s, float* c) { sincosf(a, s, c); }

// Constants of a body lane that a stage reads once, kept in LDS (one slot per
// lane of the wave): 44 registers less per lane.
template <class T>
struct PackConst {
    enum { CP, CQ, CFX, CFY, CTQ, RP, RC, RX, KD, LN, FT, LB, LS, N };
    struct Pair { T a, b; };
    Pair v[N][64];
};

// a <- a^-1 (symmetric positive definite, without pivoting)
template <int N>
__device__ __forceinline__ void spd_inverse(double (&a)[N][N]) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const double p = 1.0 / a[k][k];
        a[k][k] = p;
#pragma unroll
        for (int j = 0; j < N; ++j)
            if (j != k) a[k][j] *= p;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (i == k) continue;
            const double t = a[i][k];
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (j != k) a[i][j] = fma(-t, a[k][j], a[i][j]);
            a[i][k] = -t * p;
        }
    }
}

// Whether a link is much heavier than the torso or a body between them (or a mass is
// infinite, NaN or not positive).  A leg eliminated from its tip by angular rates then cancels:
// what the torso feels of it is a difference of its masses.  Errors of the
// paper-faithful A against 64 bits, a tip 100, 1,000, 1e6 times heavier than the
// rest: 5e-16, 4e-15, 5e-8 (the joint rows' system, which takes 1/m: 1e-16).
template <class TP>
__device__ __forceinline__ bool heavy_link(const double* mass) {
    bool ok = mass[0] > 0.0 && mass[0] < 1e300;
#pragma unroll
    for (int l = 0; l < TP::L; ++l) {
        double lo = mass[0];
#pragma unroll
        for (int e = 0; e < TP::D; ++e) {
            const double m = mass[1 + l * TP::D + e];
            ok = ok && m > 0.0 && m < 16.0 * lo;
            lo = m < lo ? m : lo;
        }
    }
    return __builtin_amdgcn_readfirstlane(ok ? 0 : 1) != 0;
}

// Body lane of one of the wave's four intervals (lane & 15 is the body) and its
// place in the tree.
template <class T, class TP>
struct PackTree {
    int b, p, j, i;
    bool body, joint, contact, pt, torso, inner;   // inner: its child is the next lane
    __device__ __forceinline__ void place(int lane) {
        body = lane < TP::NB;
        b = body ? lane : 0;
        joint = b >= 1;
        contact = joint && b % TP::D == 0;
        j = joint ? b - 1 : 0;
        i = contact ? b / TP::D - 1 : 0;
        pt = !joint || j % TP::D == 0;
        p = pt ? 0 : j;
        torso = b == 0;
        inner = joint && !contact;
    }
    __device__ __forceinline__ T parent(T v) const {
        const T t = row_lane<0>(v);
        const T q = prev_lane(v);
        return pt ? t : q;
    }
    // sum over the legs of a value held by their first links
    static __device__ __forceinline__ T legs(T v) {
        constexpr int D = TP::D;
        return row_sum_of<TP::L, 1, 1 + (TP::L > 1) * D, 1 + (TP::L > 2) * 2 * D,
                          1 + (TP::L > 3) * 3 * D>(v);
    }
    // sum over the children of a value held by the child lanes
    __device__ __forceinline__ T children(T v) const {
        const T t = legs(v);
        if constexpr (TP::D > 1) {
            const T q = next_lane(v);
            return torso ? t : (inner ? q : T(0));
        } else {
            return torso ? t : T(0);
        }
    }
};

template <class T, class TP, bool FLAT>
struct PackBody : PackTree<T, TP> {
    using Tree = PackTree<T, TP>;
    using Tree::b;
    using Tree::p;
    using Tree::j;
    using Tree::i;
    using Tree::body;
    using Tree::joint;
    using Tree::contact;
    using Tree::pt;
    using Tree::torso;
    using Tree::inner;
    using Tree::parent;
    using Tree::children;
    T mi, ii, s, mu, ipar;   // ipar: 1/I of the parent
    // LDS, pairs: hold values at the two nodes of the joint force on the body, of
    // the moment terms P = sum r x lambda, Q = sum r . lambda in body axes (signed
    // by side; with the contact force on flat ground) and of the joint torque;
    // joint anchors, contact point, stiffness and damping; contact force (n, t) at
    // the nodes and its hold means (n, t+), (t-, friction slack)
    typename PackConst<T>::Pair* lc;
    __device__ __forceinline__ typename PackConst<T>::Pair get(int q) const { return lc[64 * q]; }

    // FORCES: keep the forces themselves, not their sums (pack_accel)
    template <bool FORCES = false>
    __device__ __forceinline__ void load(const FwdArgs<T>& a,
                                         const MConst<TP::NB, TP::NJ, TP::NC>& mc, int k,
                                         int lane) {
        constexpr int NJ = TP::NJ;
        Tree::place(lane);
        const int64_t ld = a.ldn;
        s = a.s[k];
        mu = a.prm[0];
        const T m = a.prm[2 + b];
        mi = T(1) / m;
        ii = T(1) / (m * T(mc.ipm[b]));
        ipar = parent(ii);
        T rp[2] = {T(0), T(0)}, rc[2] = {T(0), T(0)}, kd[2] = {T(0), T(0)}, r[2] = {T(0), T(0)};
        if (joint) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                rp[e] = T(mc.rp[j][e]);
                rc[e] = T(mc.rc[j][e]);
            }
            kd[0] = T(mc.ks[j]);
            kd[1] = T(mc.ds[j]);
        }
        if (contact) {
            r[0] = T(mc.cr[i][0]);
            r[1] = T(mc.cr[i][1]);
        }
        T cm[3] = {T(0), T(0), T(0)};
        T F[2][2], P[2], Q[2], tq[2], ln[2], ft[2];
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const T* u = a.U + k + n;
            T lx = T(0), ly = T(0), tau = T(0);
            if (joint) {
                tau = u[j * ld];
                lx = u[(NJ + 2 * j) * ld];
                ly = u[(NJ + 2 * j + 1) * ld];
            }
            T w[3] = {T(0), T(0), T(0)};
            if (contact)
#pragma unroll
                for (int q = 0; q < 3; ++q) w[q] = u[(3 * NJ + 3 * i + q) * ld];
#pragma unroll
            for (int q = 0; q < 3; ++q) cm[q] += T(0.5) * w[q];
            ln[n] = w[0];
            ft[n] = w[1] - w[2];
            if constexpr (FORCES) {
                P[n] = lx;
                Q[n] = ly;
                tq[n] = tau;
                F[n][0] = w[1];
                F[n][1] = w[2];
                continue;
            }
            F[n][0] = children(lx) - lx;
            F[n][1] = children(ly) - ly;
            P[n] = children(rp[0] * ly - rp[1] * lx) - (rc[0] * ly - rc[1] * lx);
            Q[n] = children(rp[0] * lx + rp[1] * ly) - (rc[0] * lx + rc[1] * ly);
            tq[n] = tau - children(tau);
            if constexpr (FLAT) {
                // (0 x the other component: its NaN spreads as in the rotated frame)
                F[n][0] += ft[n] + T(0) * ln[n];
                F[n][1] += ln[n] + T(0) * ft[n];
                P[n] += r[0] * ln[n] - r[1] * ft[n];
                Q[n] += r[0] * ft[n] + r[1] * ln[n];
            }
        }
        using C = PackConst<T>;
        auto put = [&](int q, T x, T y) { lc[64 * q] = typename C::Pair{x, y}; };
        put(C::CP, P[0], P[1]);
        put(C::CQ, Q[0], Q[1]);
        put(C::CFX, F[0][0], F[1][0]);
        put(C::CFY, F[0][1], F[1][1]);
        put(C::CTQ, tq[0], tq[1]);
        put(C::RP, rp[0], rp[1]);
        put(C::RC, rc[0], rc[1]);
        put(C::RX, r[0], r[1]);
        put(C::KD, kd[0], kd[1]);
        put(C::LN, ln[0], ln[1]);
        put(C::FT, ft[0], ft[1]);
        put(C::LB, cm[0], cm[1]);
        put(C::LS, cm[2], mu * cm[0] - cm[1] - cm[2]);
    }
};

// Scalar responses at a stage: tau, the weight w of the stage in the integral
// rows (0: none) and s w, and the velocities and positions (per s, s^2 / m) of
// a mass under the hold weights 1 - tau and tau at the stage input.
template <class T>
struct StageHold {
    T tau, w, sw, vm, vp, xm, xp;
};

// What the state wave hands to the coefficient wave, per stage (two slots, in
// turn; a third for a stage of its own) and lane: the stage input, its rotation
// and its S column; at the end, a flag sum and the error estimate.
template <class T, int SLOTS = 2>
struct PackShared {
    using Pair = typename PackConst<T>::Pair;
    PackConst<T> lc;
    T v[SLOTS][3][64];                  // velocities
    Pair cs[SLOTS][64], xy[SLOTS][64];  // also read by the children
    T z[2][6][64];
    T fin[64], err[64];
    __device__ __forceinline__ void put(int slot, int me, const T (&x)[6], T cb, T sb) {
        cs[slot][me] = Pair{cb, sb};
        xy[slot][me] = Pair{x[0], x[1]};
#pragma unroll
        for (int q = 0; q < 3; ++q) v[slot][q][me] = x[3 + q];
    }
};

template <class T>
__device__ __forceinline__ T mul_add(T a, T b, T c) { return __builtin_elementwise_fma(a, b, c); }

// State wave: accelerations f of the stage input xs, derivative kz of the S
// column's velocity rows at zs, the own-angle coefficient cth and the rotation.
template <class T, class TP, bool FLAT>
__device__ __forceinline__ void pack_state(const PackBody<T, TP, FLAT>& c,
                                           const MConst<TP::NB, TP::NJ, TP::NC>& mc,
                                           const T (&xs)[6], const T (&zs)[6], T tau, T (&f)[3],
                                           T (&kz)[3], T& cth, T& cb, T& sb) {
    using C = PackConst<T>;
    asm volatile("" ::: "memory");   // read the constants in every stage, keep none
    const T omt = T(1) - tau;
    auto hold = [&](int q) {
        const auto v = c.get(q);
        return omt * v.a + tau * v.b;
    };
    const T P = hold(C::CP), Q = hold(C::CQ);
    T Fx = hold(C::CFX), Fy = hold(C::CFY), Tq = hold(C::CTQ);
    const auto kd = c.get(C::KD);
    // spring-damper torque of the own joint (zero without one), also the S column's
    const T ts = kd.a * (xs[2] - c.parent(xs[2])) + kd.b * (xs[5] - c.parent(xs[5]));
    const T tz = kd.a * (zs[2] - c.parent(zs[2])) + kd.b * (zs[5] - c.parent(zs[5]));
    Tq += c.children(ts) - ts;
    const T dz = c.children(tz) - tz;
    sincos_pack(xs[2], &sb, &cb);
    Tq += cb * P - sb * Q;
    T dT = -(sb * P + cb * Q);
    const T si = c.s * c.ii;
    T fxx = T(0), fyx = T(0), ftx = T(0), ay = T(0);
    if constexpr (!FLAT) {
        // contact point, frame and force (lanes without a contact: none)
        const auto cr = c.get(C::RX);
        const T ax = cb * cr.a - sb * cr.b;
        ay = sb * cr.a + cb * cr.b;
        const Frame<T> fr = terrain<T>(mc, xs[0] + ax, xs[1] + ay);
        const T ln = hold(C::LN), ft = hold(C::FT);
        auto own = [&](T v) { return c.contact ? v : T(0); };
        const T fx = own(fr.tx * ft + fr.nx * ln), fy = own(fr.ty * ft + fr.ny * ln);
        const T dfx = own(fr.dny * ft + fr.dnx * ln), dfy = own(-fr.dnx * ft + fr.dny * ln);
        Fx += fx;
        Fy += fy;
        Tq += ax * fy - ay * fx;
        dT -= ax * fx + ay * fy;
        fxx = dfx * (c.s * c.mi);
        fyx = dfy * (c.s * c.mi);
        ftx = (ax * dfy - ay * dfx) * si;
    }
    f[0] = Fx * c.mi;
    f[1] = Fy * c.mi - T(mc.g);
    f[2] = Tq * c.ii;
    cth = si * dT;
    if constexpr (!FLAT) cth -= ftx * ay;
    kz[0] = f[0];
    kz[1] = f[1];
    kz[2] = f[2] + cth * zs[2] + si * dz;
    if constexpr (!FLAT) {
        auto own = [&](T v) { return c.contact ? v : T(0); };
        kz[0] += own(fxx * (zs[0] - ay * zs[2]));
        kz[1] += own(fyx * (zs[0] - ay * zs[2]));
        kz[2] += own(ftx * zs[0]);
    }
}

// As pack_state from the forces themselves (PackBody::load<true>), the
// accelerations in a fixed arithmetic: an embedded error estimate is a difference of
// nearly equal sums, down to their rounding, so which product of a sum is rounded
// is written out (mul_add) and not left to the compiler.
template <class T, class TP, bool FLAT>
__device__ __forceinline__ void pack_accel(const PackBody<T, TP, FLAT>& c,
                                           const MConst<TP::NB, TP::NJ, TP::NC>& mc,
                                           const T (&xs)[6], const T (&zs)[6], T tau, T (&f)[3],
                                           T (&kz)[3], T& cth, T& cb, T& sb) {
    using C = PackConst<T>;
    asm volatile("" ::: "memory");   // read the constants in every stage, keep none
    const T omt = T(1) - tau;
    auto hold = [&](int q) {
        const auto v = c.get(q);
        return mul_add(tau, v.b, omt * v.a);
    };
    sincos_pack(xs[2], &sb, &cb);
    const T thp = c.parent(xs[2]), omp = c.parent(xs[5]);
    const T sp = c.parent(sb), cp = c.parent(cb);
    const auto kd = c.get(C::KD);
    T Fx = T(0), Fy = T(0), Tq = T(0), dT = T(0);
    T wx = T(0), wy = T(0), wt = T(0), dp = T(0);   // parent-side wrench of the own joint
    if (c.joint) {
        const auto jp = c.get(C::RP), jc = c.get(C::RC);
        const T apx = mul_add(cp, jp.a, -(sp * jp.b)), apy = mul_add(sp, jp.a, cp * jp.b);
        const T acx = mul_add(cb, jc.a, -(sb * jc.b)), acy = mul_add(cb, jc.b, sb * jc.a);
        const T tq = hold(C::CTQ), lx = hold(C::CP), ly = hold(C::CQ);
        const T tt = mul_add(-kd.b, xs[5] - omp, mul_add(-kd.a, xs[2] - thp, tq));
        Fx -= lx;
        Fy -= ly;
        Tq += tt - mul_add(acx, ly, -(acy * lx));
        wx = lx;
        wy = ly;
        wt = mul_add(apx, ly, -(apy * lx)) - tt;
        dT = acx * lx + acy * ly;
        dp = apx * lx + apy * ly;
    }
    const T si = c.s * c.ii;
    T fxx = T(0), fyx = T(0), ftx = T(0), ay = T(0);
    if (c.contact) {
        const auto cr = c.get(C::RX);
        const T ax = mul_add(cb, cr.a, -(sb * cr.b));
        ay = mul_add(cb, cr.b, sb * cr.a);
        const Frame<T> fr = FLAT ? Frame<T>{xs[1] + ay, T(0), T(1), T(1), T(0), T(0), T(1), T(0), T(0)}
                                 : terrain<T>(mc, xs[0] + ax, xs[1] + ay);
        const T ln = hold(C::LN), ft = hold(C::CFX) - hold(C::CFY);
        const T fx = mul_add(fr.nx, ln, fr.tx * ft), fy = mul_add(fr.ty, ft, fr.ny * ln);
        Fx += fx;
        Fy += fy;
        Tq += mul_add(ax, fy, -(ay * fx));
        dT -= ax * fx + ay * fy;
        if constexpr (!FLAT) {
            const T dfx = fr.dny * ft + fr.dnx * ln, dfy = -fr.dnx * ft + fr.dny * ln;
            fxx = dfx * (c.s * c.mi);
            fyx = dfy * (c.s * c.mi);
            ftx = (ax * dfy - ay * dfx) * si;
        }
    }
    Fx += c.children(wx);
    Fy += c.children(wy);
    Tq += c.children(wt);
    f[0] = Fx * c.mi;
    f[1] = mul_add(Fy, c.mi, -T(mc.g));
    f[2] = Tq * c.ii;
    cth = si * (dT - c.children(dp));
    if constexpr (!FLAT) cth -= ftx * ay;
    const T tz = kd.a * (zs[2] - c.parent(zs[2])) + kd.b * (zs[5] - c.parent(zs[5]));
    kz[0] = f[0];
    kz[1] = f[1];
    kz[2] = f[2] + cth * zs[2] + si * (c.children(tz) - tz);
    if constexpr (!FLAT) {   // (no 0 x NaN on bodies without a contact)
        auto own = [&](T v) { return c.contact ? v : T(0); };
        kz[0] += own(fxx * (zs[0] - ay * zs[2]));
        kz[1] += own(fyx * (zs[0] - ay * zs[2]));
        kz[2] += own(ftx * zs[0]);
    }
}

// Coefficient wave: sums over the stages of the coefficients of the integral
// rows (PackRec::SUM), and the integral rows of the state and of S.
template <class T, class TP, bool FLAT>
struct PackSums {
    T rx[4], ry[4], ey[4], ex[3], ev, gc[3];
    T zcc, zct;
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int q = 0; q < 4; ++q) rx[q] = ry[q] = ey[q] = T(0);
#pragma unroll
        for (int q = 0; q < 3; ++q) ex[q] = gc[q] = T(0);
        ev = zcc = zct = T(0);
    }
};

// One stage of the coefficient wave (slot: the state wave's; the integrands in a
// fixed arithmetic, as pack_accel): the integrands cc
// and ct, and with COEF the sums and the stage record (all but CTH).
template <class T, class TP, bool FLAT, bool COEF, int SLOTS>
__device__ __forceinline__ void pack_coef(const PackBody<T, TP, FLAT>& c,
                                          const MConst<TP::NB, TP::NJ, TP::NC>& mc,
                                          const PackShared<T, SLOTS>& sh, int slot, const StageHold<T>& hd,
                                          T& cc, T& ct, PackSums<T, TP, FLAT>& sm,
                                          T* __restrict__ rec, bool write) {
    using R = PackRec<TP, FLAT>;
    using C = PackConst<T>;
    constexpr int NJ = TP::NJ, NC = TP::NC;
    asm volatile("" ::: "memory");
    const int me = threadIdx.x & 63, up = (me & 48) + c.p;
    const T vx = sh.v[slot][0][me], vy = sh.v[slot][1][me], om = sh.v[slot][2][me];
    const auto csb = sh.cs[slot][me], xyb = sh.xy[slot][me];
    const auto csp = sh.cs[slot][up], xyp = sh.xy[slot][up];
    const T cb = csb.a, sb = csb.b, xb = xyb.a, yb = xyb.b;
    const T cp = csp.a, sp = csp.b, xp = xyp.a, yp = xyp.b;
    const auto cr = c.get(C::RX), jp = c.get(C::RP), jc = c.get(C::RC);
    const auto lb = c.get(C::LB), ls = c.get(C::LS);   // (lnb, ltpb), (ltmb, slack)
    // contact point and frame
    const T ax = mul_add(cb, cr.a, -(sb * cr.b)), ay = mul_add(cb, cr.b, sb * cr.a);
    const Frame<T> f = FLAT ? Frame<T>{yb + ay, T(0), T(1), T(1), T(0), T(0), T(1), T(0), T(0)}
                            : terrain<T>(mc, xb + ax, yb + ay);
    const T Pdx = mul_add(-om, ay, vx), Pdy = mul_add(om, ax, vy);
    // smooth functions: |h|_s of the own joint, |v_t|_s and ramp_s(-sd) of the contact
    const T apx = mul_add(cp, jp.a, -(sp * jp.b)), apy = mul_add(cp, jp.b, sp * jp.a);
    const T acx = mul_add(cb, jc.a, -(sb * jc.b)), acy = mul_add(cb, jc.b, sb * jc.a);
    const T vt = FLAT ? Pdx + T(0) * Pdy : mul_add(f.ty, Pdy, f.tx * Pdx);   // (a NaN of v_y too)
    T v0, d0, v1, d1, av, dav, v3, d3;
    sabs_d(xp + apx - xb - acx, v0, d0);
    sabs_d(yp + apy - yb - acy, v1, d1);
    sabs_d(vt, av, dav);
    sabs_d(-f.sd, v3, d3);
    const T rp = vt > T(0) ? av : T(0), rm = vt < T(0) ? av : T(0);
    const bool pen = c.contact && -f.sd > T(0);
    cc = mul_add(ls.b, av, mul_add(ls.a, rm, mul_add(lb.a, f.sd, lb.b * rp)));
    ct = (c.joint ? v0 + v1 : T(0)) + (pen ? v3 : T(0));
    if constexpr (COEF) {
        const T s = c.s, sw = hd.sw, tau = hd.tau;
        const T gv = lb.b * (vt > T(0) ? dav : T(0)) + ls.a * (vt < T(0) ? dav : T(0)) +
                     ls.b * dav;
        if (!c.joint) d0 = d1 = T(0);
        const T Dg = pen ? -d3 : T(0);
        const T si = s * c.ii, sm_ = s * c.mi;
        T epx = T(0), epy = lb.a, exd = gv, eyd = T(0), eom = -gv * ay, eth = -gv * om * ax;
        T zpx = T(0), zpy = Dg;
        if constexpr (!FLAT) {
            epx = lb.a * f.dsd_px + gv * (f.dny * Pdx - f.dnx * Pdy);
            epy = lb.a * f.dsd_py;
            exd = gv * f.tx;
            eyd = gv * f.ty;
            eom = gv * (f.ty * ax - f.tx * ay);
            eth = -gv * om * (f.tx * ax + f.ty * ay);
            zpx = c.contact ? Dg * f.dsd_px : T(0);
            zpy = c.contact ? Dg * f.dsd_py : T(0);
        }
        // integral rows by the body's pose and velocity, with the stage weight
        const T cvx = sw * (c.children(d0) - d0 + zpx), cvy = sw * (c.children(d1) - d1 + zpy);
        const T cvt = sw * (c.children(d1 * apx - d0 * apy) + (d0 * acy - d1 * acx) +
                            (zpy * ax - zpx * ay));
        const T wpx = sw * epx, wpy = sw * epy, wxd = sw * exd, wyd = sw * eyd, wom = sw * eom;
        const T wth = sw * eth + (wpy * ax - wpx * ay);
        // stage record
        if (write && c.body) {
            rec[R::CV + c.b] = cvt;
            if (c.joint) {
                T* w = rec + R::FORCE + c.j;
                const T ip = s * c.ipar;
                w[0] = -apy * ip;
                w[NJ] = apx * ip;
                w[2 * NJ] = acy * si;
                w[3 * NJ] = -acx * si;
            }
            if (c.contact) {
                T* w = rec + R::FT + R::NFOOT * c.i;
                T* g = rec + R::CF + c.i;
                w[R::F_CTH] = wth;
                w[R::F_COM] = wom;
                if constexpr (FLAT) {
                    g[0] = ax * si;
                    g[NC] = -ay * si;
                    g[2 * NC] = ay * si;
                } else {
                    // the contact force's derivatives along the surface
                    const T omt = T(1) - tau;
                    const auto l0 = c.get(C::LN), l1 = c.get(C::FT);
                    const T ln = omt * l0.a + tau * l0.b, ft = omt * l1.a + tau * l1.b;
                    const T dfx = f.dny * ft + f.dnx * ln, dfy = -f.dnx * ft + f.dny * ln;
                    const T fxx = dfx * sm_, fyx = dfy * sm_;
                    w[R::F_CX] = wpx;
                    w[R::F_CY] = wpy;
                    w[R::F_CVX] = wxd;
                    w[R::F_CVY] = wyd;
                    w[R::F_XX] = fxx;
                    w[R::F_XT] = -fxx * ay;
                    w[R::F_YX] = fyx;
                    w[R::F_YT] = -fyx * ay;
                    w[R::F_TX] = (ax * dfy - ay * dfx) * si;
                    w[R::F_ZX] = cvx;
                    w[R::F_ZY] = cvy;
                    const T tn = (ax * f.ny - ay * f.nx) * si, tt = (ax * f.ty - ay * f.tx) * si;
                    const T row[9] = {f.nx * sm_, f.tx * sm_, -f.tx * sm_, f.ny * sm_, f.ty * sm_,
                                      -f.ty * sm_, tn, tt, -tt};
#pragma unroll
                    for (int q = 0; q < 9; ++q) g[q * NC] = row[q];
                }
            }
        }
        // sums over the stages
        sm.rx[0] += cvx;
        sm.rx[1] += cvx * tau;
        sm.rx[2] += cvx * hd.xm;
        sm.rx[3] += cvx * hd.xp;
        sm.ry[0] += cvy;
        sm.ry[1] += cvy * tau;
        sm.ry[2] += cvy * hd.xm;
        sm.ry[3] += cvy * hd.xp;
        sm.ey[0] += wpy;
        sm.ey[1] += wpy * tau;
        if constexpr (FLAT) {
            sm.ey[2] += wpy * hd.xm;
            sm.ey[3] += wpy * hd.xp;
            sm.ex[0] += wxd;
            sm.ex[1] += wxd * hd.vm;
            sm.ex[2] += wxd * hd.vp;
        } else {
            sm.ev += wyd;
        }
        sm.gc[0] += (T(0.5) * sw) * (f.sd + c.mu * av);
        sm.gc[1] += (T(0.5) * sw) * (rp - av);
        sm.gc[2] += (T(0.5) * sw) * (rm - av);
        // integral rows of S
        auto z = [&](int q) { return sh.z[slot][q][me]; };
        const T z0 = z(0), z1 = z(1), z2 = z(2);
        sm.zcc += wpx * z0 + wpy * z1 + wth * z2 + wxd * z(3) + wyd * z(4) + wom * z(5) + hd.w * cc;
        sm.zct += cvx * z0 + cvy * z1 + cvt * z2 + hd.w * ct;
    }
}

// Constants of the interval for the tangent launch (body and joint lanes).
template <class T, class TP, bool FLAT>
__device__ __forceinline__ void pack_header(const PackBody<T, TP, FLAT>& c, T h, T* rec) {
    using R = PackRec<TP, FLAT>;
    if (!c.body) return;
    if (c.torso) {
        rec[0] = c.s;
        rec[1] = h;
    }
    rec[R::MINV + c.b] = c.mi;
    rec[R::IINV + c.b] = c.ii;
    if (c.joint) {
        T* w = rec + R::KC + 4 * c.j;
        const auto kd = c.get(PackConst<T>::KD);
        w[0] = c.s * kd.a * c.ipar;
        w[1] = c.s * kd.b * c.ipar;
        w[2] = -(c.s * kd.a * c.ii);
        w[3] = -(c.s * kd.b * c.ii);
    }
}

// Sums of the interval at sums[q * n].
template <class T, class TP, bool FLAT>
__device__ __forceinline__ void pack_sums(const PackBody<T, TP, FLAT>& c,
                                          const PackSums<T, TP, FLAT>& sm, T angles, T zct,
                                          T* sums, int64_t n) {
    using R = PackRec<TP, FLAT>;
    if (!c.body) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        sums[(R::RX + q * TP::NB + c.b) * n] = sm.rx[q];
        sums[(R::RY + q * TP::NB + c.b) * n] = sm.ry[q];
    }
    if (c.contact) {
#pragma unroll
        for (int q = 0; q < 4; ++q) sums[(R::EY + q * TP::NC + c.i) * n] = sm.ey[q];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            sums[(R::EX + q * TP::NC + c.i) * n] = sm.ex[q];
            sums[(R::GC + q * TP::NC + c.i) * n] = sm.gc[q];
        }
        sums[(R::EV + c.i) * n] = sm.ev;
        // a coefficient of the row that is no number leaves one in these two
        sums[(R::PZ + 2 + c.i) * n] = T(0) * (sm.ey[0] + (FLAT ? sm.ex[0] : sm.ev));
    }
    if (c.torso) {
        sums[R::PZ * n] = T(0) * angles;
        sums[(R::PZ + 1) * n] = T(0) * zct;
    }
}

// Outputs of one row of the nominal state (F~, defect) and of S.
template <class T>
__device__ __forceinline__ void pack_output(const FwdArgs<T>& a, int k, int r, T x, T z) {
    if (a.xprop) a.xprop[r * a.ldi + k] = x;
    a.defect[r * a.ldi + k] = x - a.X[r * a.ldn + k + 1];
    a.S[r * a.ldi + k] = z;
}

// n / d with the reciprocal r of d: quotient estimate and one residual step
// (three instructions where the division takes about ten).
template <class T>
__device__ __forceinline__ T quotient(T n, T d, T r) {
    const T q = n * r;
    return __builtin_elementwise_fma(__builtin_elementwise_fma(-q, d, n), r, q);
}

// Response of a unit-mass translation to the hold weights at t (exact for the
// RK methods used, whose nodes integrate cubics exactly).
template <class T>
__device__ __forceinline__ void hold_nodes(T t, T& vm, T& vp, T& xm, T& xp) {
    vp = T(0.5) * t * t;
    vm = t - vp;
    xp = t * vp / T(3);
    xm = vp - xp;
}

}  // namespace cis
