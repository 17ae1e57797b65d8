// Discretize step of the paper-faithful dynamics variant (arxiv 2604.09993):
// joint reaction forces eliminated at the acceleration level (Sec. II-A,
// eq. joint-cnstr-acc), controls u = (tau, (phi_t, phi_n, gamma) per contact)
// (the state-space form after it), and the auxiliary system of eq. aux-dynamics
// with four integral states per contact (phi_n, lambda_c, gamma, rho_c) and one
// violation state summing ramp_s(g) over g = (-phi_n, -sd, -gamma, -rho_c).
// Classical RK4 with K substeps and the variational equations through the same
// stages (Sec. IV-B, Sec. VI), FP64.
//
// The joint forces are eliminated leg by leg instead of through A = grad h M^-1 grad
// h^T: the joint rows grad h v' + c = 0 give every link's translation from the
// torso's acceleration a0 = (v'_0, w'_0) and the angular accelerations of its leg,
//     v'_l = v'_0 + w'_0 E a_p1 + sum_{i<=l} (gamma_i + w'_i E r_li),
//     r_li = a_p,i+1 - a_c,i (i < l),  r_ll = -a_c,l,  E a = (-a_y, a_x),
//     gamma_i = -w_p^2 a_p + w_c^2 a_c,
// and virtual work along the w'_i leaves, per leg, H w' = f - H0 a0 (H symmetric, as
// many rows as the leg has links) and a 3 x 3 system of the torso,
//     w' = H^-1 f - G a0,  G = H^-1 H0,  (M0 + sum_legs (M_leg - H0^T G)) a0 = ... .
// A direction of the state or of the controls moves v' by the same elimination
// with perturbed forces u = dF + dgrad_h^T lambda and joint terms d = dgrad_h v' +
// dc in the place of F and gamma.  Two kernels:
//   k_paper_rec : four intervals per wave on rows of 16 body lanes; the nominal RK4,
//                 and per stage and leg the coefficients of u, d, H^-1, G and the
//                 torso's inverse to device memory;
//   k_paper_tan : per (interval, block of 64 columns of [Phi_x | B- | B+ | S]) one
//                 wave per leg, a lane holding its column on the torso and leg
//                 rows; the stage's coefficients as vectors of 16 that enter the
//                 FMAs as DPP broadcasts; one exchange of three values between
//                 the legs per stage (the torso's system).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <type_traits>
#include <utility>

#include "../../include/cis.h"
#include "cis_debug.hpp"
#include "cis_host.hpp"
#include "cis_launch.hpp"
#include "cis_model.hpp"
#include "cis_pack.hpp"
#include "cis_paper.hpp"
#include "cis_paper_dense.hpp"
#include "cis_reduced.hpp"

namespace cis {

// Layout of an interval's record area (doubles): header [HDR]: s, h, 0 x6, the masses,
// then (k_j, d_j); stage t < 4 K, leg l at HDR + (t L + l) LEG, as vectors of 16:
//   joint of link l at JN (l - 1): arms a_p, a_c, then d by th_p, th_c, w_p, w_c (x, y
//   each), a_p . lambda, a_c . lambda
//   HI: H^-1 (lower triangle); G [D][3]; SI: the torso's inverse (upper triangle)
//   CO: the contact: force and torque by its x and theta, by the controls phi_t and
//   phi_n, d lambda_c by x, theta, w, d violation by x, y, theta, and the controls'
//   integrand partials
//   SF: forcing of S: v and v' of the torso and the links, the integrands
template <class TP>
struct PRec {
    static constexpr int D = TP::D;
    static constexpr int HDR = (8 + TP::NB + 2 * TP::NJ + 7) / 8 * 8;
    static constexpr int JN = 14, HI = JN * D, G = HI + D * (D + 1) / 2, SI = G + 3 * D;
    static constexpr int CO = SI + 6;
    enum { FXX = CO, FXT, FYX, FYT, TQX, TQT, CTX, CNX, CTY, CNY, CTT, CTN, LX, LT, LW, SX, SY, ST,
           LCT, LCG, RCN, RCT, VN, VT, VG, SF };
    static constexpr int YF = SF + 6 * (D + 1), NSC = YF + 5, NV = (NSC + 15) / 16;
    static constexpr int LEG = 16 * NV, STAGE = TP::L * LEG;
    __host__ __device__ static constexpr int hi(int i, int k) {   // i >= k
        return HI + i * (i + 1) / 2 + k;
    }
    static constexpr int64_t per_interval(int K) { return HDR + (int64_t)4 * K * STAGE; }
};

template <class TP>
struct PShared {
    enum { RX, RY, SX, SY, HD, F, AX, AY, N };   // a link's part of its leg's system
    double g[N][64];
};

// ---------------------------------------------------------------------------
// k_paper_rec: four intervals, one wave, lane & 15 the body.  Sums along a leg run
// by lane shifts (links of a leg are consecutive lanes); every lane then forms its
// leg's system from the links' parts in LDS, and the torso's from the legs' sums.
// Bound by the serial chain of a stage (two sines, nine root estimates, six divisions,
// eight shift sums), 3.4 us of it.  1,603 quad13 intervals, K = 20: 270 us; one interval
// per wave with a 24 x 24 Gauss-Jordan elimination took 1,650 us.
// ROWS: the joint rows' form too, one interval per workgroup (the grid has one for each
// of them, and the legs take the first quarter).
// ---------------------------------------------------------------------------
template <class TP, bool ROWS>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1)))
    k_paper_rec(PaperArgs a, MConst<TP::NB, TP::NJ, TP::NC> mc) {
    constexpr int NJ = TP::NJ, NC = TP::NC, NQ = TP::NQ, N6 = TP::N6;
    constexpr int NX = TP::NX, NY = TP::NY, D = TP::D;
    using R = PRec<TP>;
    using SH = PShared<TP>;
    __shared__ union {
        SH legs;
        std::conditional_t<ROWS, PDenseShared<TP>, char> rows;
    } lds;
    if (heavy_link<TP>(a.prm + 2)) {
        if constexpr (ROWS) paper_dense_rec<TP>(a, mc, lds.rows, xcd_slot(blockIdx.x, gridDim.x));
        return;
    }
    SH& sh = lds.legs;
    const int me = threadIdx.x, waves = (a.N + 3) / 4;
    if ((int)blockIdx.x >= waves) return;
    const int want = 4 * xcd_slot(blockIdx.x, waves) + (me >> 4);
    const bool on = want < a.N;   // spare rows repeat the last interval
    const int k = on ? want : a.N - 1;
    const int64_t ldn = a.ldn, ldi = a.ldi;
    double* rec = a.rec + (int64_t)k * R::per_interval(a.K);
    PackTree<double, TP> c;
    c.place(me & 15);
    const bool body = on && c.body;
    const int leg = c.joint ? c.j / D : 0, lk = c.joint ? c.j % D : 0;
    const bool first = c.joint && lk == 0;
    const int leg0 = (me & 48) + 1 + leg * D;   // lane of the leg's first link
    const double s = a.s[k], h = 1.0 / double(a.K), mu = a.prm[0];
    const double m = a.prm[2 + c.b], I = m * mc.ipm[c.b];
    double rp[2] = {0.0, 0.0}, rc[2] = {0.0, 0.0}, ks = 0.0, ds = 0.0, cr[2] = {0.0, 0.0};
    double tq[2] = {0.0, 0.0}, cu[3][2];
    if (c.joint) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            rp[e] = mc.rp[c.j][e];
            rc[e] = mc.rc[c.j][e];
            tq[e] = a.U[c.j * ldn + k + e];
        }
        ks = mc.ks[c.j];
        ds = mc.ds[c.j];
    }
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int e = 0; e < 2; ++e)
            cu[q][e] = c.contact ? a.U[(NJ + 3 * c.i + q) * ldn + k + e] : 0.0;
    if (c.contact) {
        cr[0] = mc.cr[c.i][0];
        cr[1] = mc.cr[c.i][1];
    }
    // sums over a leg: up to and with the own link from the torso, and from the tip
    auto from_torso = [&](double v) {
        double t = v;
#pragma unroll
        for (int e = 1; e < D; ++e) {
            const double q = prev_lane(t);
            t = first ? v : v + q;
        }
        return t;
    };
    auto beyond = [&](double v) {   // without the own link
        double t = 0.0;
#pragma unroll
        for (int e = 1; e < D; ++e) {
            const double q = next_lane(t + v);
            t = c.inner ? q : 0.0;
        }
        return t;
    };
    const double msub = beyond(m), mleg = msub + m;   // mleg: on first links
    const double m0 = row_lane<0>(m), I0 = row_lane<0>(I);
    if (body) {
        if (c.torso) {
            rec[0] = s;
            rec[1] = h;
        }
        rec[8 + c.b] = m;
        if (c.joint) {
            rec[8 + TP::NB + 2 * c.j] = ks;
            rec[8 + TP::NB + 2 * c.j + 1] = ds;
        }
    }
    auto row = [&](int q) { return q < 3 ? 3 * c.b + q : NQ + 3 * c.b + q - 3; };
    double xb[6], xa[6], xs[6], yb[4], ya[4], vb = 0.0, va = 0.0;
#pragma unroll
    for (int q = 0; q < 6; ++q) xs[q] = xb[q] = a.X[row(q) * ldn + k];
#pragma unroll
    for (int q = 0; q < 4; ++q) yb[q] = c.contact ? a.X[(N6 + 4 * c.i + q) * ldn + k] : 0.0;
    vb = a.X[(N6 + 4 * NC) * ldn + k];
    double* sr = rec + R::HDR;
    for (int t = 0; t < 4 * a.K; ++t, sr += R::STAGE) {
        const int st = t & 3;
        const double tau = (double(t >> 2) + (st == 0 ? 0.0 : (st == 3 ? 1.0 : 0.5))) * h;
        const double omt = 1.0 - tau;
        double* lr = sr + leg * R::LEG;
        auto put = [&](int q, double v) { lr[q] = v; };
        const double om = xs[5], omp = c.parent(om);
        double cb, sb;
        sincos_pack(xs[2], &sb, &cb);
        const double cp = c.parent(cb), sp = c.parent(sb);
        // joint: arms, torque, velocity products (zero without one)
        const double apx = cp * rp[0] - sp * rp[1], apy = sp * rp[0] + cp * rp[1];
        const double acx = cb * rc[0] - sb * rc[1], acy = sb * rc[0] + cb * rc[1];
        const double thp = c.parent(xs[2]);
        const double tt = c.joint ? (omt * tq[0] + tau * tq[1]) - ks * (xs[2] - thp) - ds * (om - omp)
                                  : 0.0;
        const double wp2 = omp * omp, wc2 = om * om;
        const double gx = c.joint ? wc2 * acx - wp2 * apx : 0.0;
        const double gy = c.joint ? wc2 * acy - wp2 * apy : 0.0;
        double Fx = 0.0, Fy = -m * mc.g, T = tt - c.children(tt);
        double io[4] = {0.0, 0.0, 0.0, 0.0}, viol = 0.0;
        if (c.contact) {
            const double ax = cb * cr[0] - sb * cr[1], ay = sb * cr[0] + cb * cr[1];
            const double Px = xs[0] + ax, Py = xs[1] + ay;
            // terrain frame (Sec. II; sd = H / ||grad H||, Sec. VI-B) and its x-derivative
            double sw, cw;
            sincos_pack(mc.kappa * Px, &sw, &cw);
            const double H = Py - mc.A * sw;
            const double Hx = -mc.A * mc.kappa * cw;
            const double Hxx = mc.A * mc.kappa * mc.kappa * sw;
            const double rG = rsqrt_t(1.0 + Hx * Hx), rG3 = rG * rG * rG;
            const double sd = H * rG;
            const double nx = Hx * rG, ny = rG;
            const double dnx = Hxx * rG3, dny = -Hx * Hxx * rG3;
            const double tx = ny, ty = -nx, dtx = dny, dty = -dnx;
            const double gsx = Hx * rG - H * Hx * Hxx * rG3, gsy = rG;
            const double pt = omt * cu[0][0] + tau * cu[0][1];
            const double pn = omt * cu[1][0] + tau * cu[1][1];
            const double gm = omt * cu[2][0] + tau * cu[2][1];
            const double cfx = tx * pt + nx * pn, cfy = ty * pt + ny * pn;
            Fx += cfx;
            Fy += cfy;
            T += ax * cfy - ay * cfx;
            const double jvx = xs[3] - om * ay, jvy = xs[4] + om * ax;
            // smooth functions and slopes (a ramp is its |.|_s, or zero)
            double vn, dn, vt, dt, v1, d1, v2, d2, v3, d3, v4, d4;
            sabs_wide(mu * pn, vn, dn);
            sabs_d(pt, vt, dt);
            const double y1 = rsqrt_t<true>(pt * pt + 1.0);
            const double lc = tx * jvx + ty * jvy + gm * dt;
            const double rr = vn - vt;
            sabs_d(-pn, v1, d1);
            sabs_d(-sd, v2, d2);
            sabs_d(-gm, v3, d3);
            sabs_d(-rr, v4, d4);
            auto ramp = [](double arg, double v) { return arg > 0.0 ? v : 0.0; };
            io[0] = pn;
            io[1] = lc;
            io[2] = gm;
            io[3] = rr;
            viol = ramp(-pn, v1) + ramp(-sd, v2) + ramp(-gm, v3) + ramp(-rr, v4);
            if (body) {
                const double fxx = dtx * pt + dnx * pn, fyx = dty * pt + dny * pn;
                const double tqx = ax * fyx - ay * fxx;
                put(R::FXX, fxx);
                put(R::FXT, -fxx * ay);
                put(R::FYX, fyx);
                put(R::FYT, -fyx * ay);
                put(R::TQX, tqx);
                put(R::TQT, -(ax * cfx + ay * cfy) - tqx * ay);
                put(R::CTX, tx);
                put(R::CNX, nx);
                put(R::CTY, ty);
                put(R::CNY, ny);
                put(R::CTT, ax * ty - ay * tx);
                put(R::CTN, ax * ny - ay * nx);
                const double lx = dtx * jvx + dty * jvy;
                put(R::LX, lx);
                put(R::LT, -lx * ay - om * (tx * ax + ty * ay));
                put(R::LW, ty * ax - tx * ay);
                const double ccs = -ramp(-sd, d2);
                put(R::SX, ccs * gsx);
                put(R::SY, ccs * gsy);
                put(R::ST, ccs * (gsy * ax - gsx * ay));
                const double rcn = mu * dn, rct = -dt, ccr = -ramp(-rr, d4);
                put(R::LCT, gm * (y1 * y1 * y1));
                put(R::LCG, dt);
                put(R::RCN, rcn);
                put(R::RCT, rct);
                put(R::VN, ccr * rcn - ramp(-pn, d1));
                put(R::VT, ccr * rct);
                put(R::VG, -ramp(-gm, d3));
#pragma unroll
                for (int q = 0; q < 4; ++q) put(R::YF + q, io[q]);
            }
        }
        viol = row_sum(c.body ? viol : 0.0);
        // the leg's system
        const double Gx = from_torso(gx), Gy = from_torso(gy);
        const double Px = Fx - m * Gx, Py = Fy - m * Gy;
        const double Qx = beyond(Px), Qy = beyond(Py);
        const double nax = next_lane(apx), nay = next_lane(apy);
        const double rx = c.inner ? nax - acx : 0.0, ry = c.inner ? nay - acy : 0.0;
        {
            const double v[SH::N] = {rx, ry, msub * rx - m * acx, msub * ry - m * acy,
                                     I + m * (acx * acx + acy * acy) + msub * (rx * rx + ry * ry),
                                     T + (acy * Px - acx * Py) + (rx * Qy - ry * Qx), apx, apy};
#pragma unroll
            for (int q = 0; q < SH::N; ++q) sh.g[q][me] = v[q];
        }
        plds_sync();
        double Hi[D][D], H0[D][3], Gm[D][3], y[D];
        const double a1x = sh.g[SH::AX][leg0], a1y = sh.g[SH::AY][leg0];
#pragma unroll
        for (int i = 0; i < D; ++i) {
            const double qx = sh.g[SH::RX][leg0 + i], qy = sh.g[SH::RY][leg0 + i];
            const double ex = sh.g[SH::SX][leg0 + i], ey = sh.g[SH::SY][leg0 + i];
            Hi[i][i] = sh.g[SH::HD][leg0 + i];
            y[i] = sh.g[SH::F][leg0 + i];
            H0[i][0] = -ey;
            H0[i][1] = ex;
            H0[i][2] = ex * a1x + ey * a1y;
#pragma unroll
            for (int l = i + 1; l < D; ++l)
                Hi[i][l] = Hi[l][i] = qx * sh.g[SH::SX][leg0 + l] + qy * sh.g[SH::SY][leg0 + l];
        }
        plds_sync();
        spd_inverse<D>(Hi);
        double f[D];
#pragma unroll
        for (int i = 0; i < D; ++i) f[i] = y[i];
#pragma unroll
        for (int i = 0; i < D; ++i) {
            double t0 = 0.0, g0 = 0.0, g1 = 0.0, g2 = 0.0;
#pragma unroll
            for (int l = 0; l < D; ++l) {
                t0 += Hi[i][l] * f[l];
                g0 += Hi[i][l] * H0[l][0];
                g1 += Hi[i][l] * H0[l][1];
                g2 += Hi[i][l] * H0[l][2];
            }
            y[i] = t0;
            Gm[i][0] = g0;
            Gm[i][1] = g1;
            Gm[i][2] = g2;
        }
        // the torso's system: first links hold their leg's part
        double S[3][3], r0[3];
        {
            const double tx1 = Px + Qx, ty1 = Py + Qy;
            double p[6] = {mleg, 0.0, -mleg * a1y, mleg, mleg * a1x, mleg * (a1x * a1x + a1y * a1y)};
            double q[3] = {tx1, ty1, a1x * ty1 - a1y * tx1};
#pragma unroll
            for (int i = 0; i < D; ++i) {
                p[0] -= H0[i][0] * Gm[i][0];
                p[1] -= H0[i][0] * Gm[i][1];
                p[2] -= H0[i][0] * Gm[i][2];
                p[3] -= H0[i][1] * Gm[i][1];
                p[4] -= H0[i][1] * Gm[i][2];
                p[5] -= H0[i][2] * Gm[i][2];
#pragma unroll
                for (int e = 0; e < 3; ++e) q[e] -= H0[i][e] * y[i];
            }
#pragma unroll
            for (int e = 0; e < 6; ++e) p[e] = c.legs(p[e]);
#pragma unroll
            for (int e = 0; e < 3; ++e) r0[e] = c.legs(q[e]);
            S[0][0] = p[0] + m0;
            S[0][1] = S[1][0] = p[1];
            S[0][2] = S[2][0] = p[2];
            S[1][1] = p[3] + m0;
            S[1][2] = S[2][1] = p[4];
            S[2][2] = p[5] + I0;
            r0[0] += row_lane<0>(Fx);
            r0[1] += row_lane<0>(Fy);
            r0[2] += row_lane<0>(T);
        }
        spd_inverse<3>(S);
        double a0[3];
#pragma unroll
        for (int e = 0; e < 3; ++e) a0[e] = S[e][0] * r0[0] + S[e][1] * r0[1] + S[e][2] * r0[2];
        // accelerations of the own body
        double w = a0[2];
#pragma unroll
        for (int i = 0; i < D; ++i) {
            const double wi = y[i] - (Gm[i][0] * a0[0] + Gm[i][1] * a0[1] + Gm[i][2] * a0[2]);
            if (c.joint && lk == i) w = wi;
        }
        const double ex = from_torso(c.joint ? -ry * w : 0.0), ey = from_torso(c.joint ? rx * w : 0.0);
        double vx = a0[0], vy = a0[1];
        if (c.joint) {   // (ex, ey without the own link)
            vx += -a0[2] * a1y + Gx + (ex + ry * w) + acy * w;
            vy += a0[2] * a1x + Gy + (ey - rx * w) - acx * w;
        }
        // joint forces
        const double qx = Fx - m * vx, qy = Fy - m * vy;
        const double lx = qx + beyond(qx), ly = qy + beyond(qy);
        // ---- stage record ----
        const double wpar = c.parent(w);   // (every lane takes part in a lane shift)
        if (body) {
            if (c.joint) {
                const double jr[R::JN] = {apx, apy, acx, acy,
                                          wp2 * apy - wpar * apx, -wp2 * apx - wpar * apy,
                                          w * acx - wc2 * acy, w * acy + wc2 * acx,
                                          -2.0 * omp * apx, -2.0 * omp * apy, 2.0 * om * acx,
                                          2.0 * om * acy, apx * lx + apy * ly, acx * lx + acy * ly};
#pragma unroll
                for (int q = 0; q < R::JN; ++q) put(R::JN * lk + q, jr[q]);
                const double sf[6] = {xs[3], xs[4], om, vx, vy, w};
#pragma unroll
                for (int q = 0; q < 6; ++q) put(R::SF + 6 * (lk + 1) + q, sf[q]);
            } else {
                const double sf[6] = {xs[3], xs[4], om, vx, vy, w};
#pragma unroll
                for (int l = 0; l < TP::L; ++l) {
#pragma unroll
                    for (int q = 0; q < 6; ++q) sr[l * R::LEG + R::SF + q] = sf[q];
                    sr[l * R::LEG + R::YF + 4] = l == 0 ? viol : 0.0;
                }
            }
            if (first) {
#pragma unroll
                for (int i = 0; i < D; ++i) {
#pragma unroll
                    for (int l = 0; l <= i; ++l) put(R::hi(i, l), Hi[i][l]);
#pragma unroll
                    for (int e = 0; e < 3; ++e) put(R::G + 3 * i + e, Gm[i][e]);
                }
                const double si[6] = {S[0][0], S[0][1], S[0][2], S[1][1], S[1][2], S[2][2]};
#pragma unroll
                for (int e = 0; e < 6; ++e) put(R::SI + e, si[e]);
            }
        }
        // ---- RK4 of the nominal ----
        const double wk = (st == 0 || st == 3) ? 1.0 : 2.0;
        const double an = (st == 2) ? h : 0.5 * h;
        const double vd[3] = {vx, vy, w};
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const double kk = s * (q < 3 ? xs[3 + q] : vd[q - 3]);
            xa[q] = st == 0 ? kk : xa[q] + wk * kk;
        }
        if (st < 3) {
            const double v0 = xs[3], v1 = xs[4], v2 = xs[5];
            xs[0] = xb[0] + an * (s * v0);
            xs[1] = xb[1] + an * (s * v1);
            xs[2] = xb[2] + an * (s * v2);
#pragma unroll
            for (int q = 0; q < 3; ++q) xs[3 + q] = xb[3 + q] + an * (s * vd[q]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) ya[q] = st == 0 ? s * io[q] : ya[q] + wk * (s * io[q]);
        va = st == 0 ? s * viol : va + wk * (s * viol);
        if (st == 3) {
#pragma unroll
            for (int q = 0; q < 6; ++q) xs[q] = xb[q] += (h / 6.0) * xa[q];
#pragma unroll
            for (int q = 0; q < 4; ++q) yb[q] += (h / 6.0) * ya[q];
            vb += (h / 6.0) * va;
        }
    }
    // ---- outputs of the nominal ----
    auto out = [&](int r, double v) {
        if (a.xprop) a.xprop[r * ldi + k] = v;
        a.defect[r * ldi + k] = v - a.X[r * ldn + k + 1];
    };
    if (body) {
#pragma unroll
        for (int q = 0; q < 6; ++q) out(row(q), xb[q]);
        if (c.contact)
#pragma unroll
            for (int q = 0; q < 4; ++q) out(N6 + 4 * c.i + q, yb[q]);
        if (c.torso) out(N6 + 4 * NC, vb);
    }
    // A[:, n:] = [0; I]: the integral states feed back into nothing
    if (on)
        for (int e = me & 15; e < NX * NY; e += 16) {
            const int r = e / NY, cc = N6 + e % NY;
            a.A[((int64_t)r * NX + cc) * ldi + k] = (r == cc) ? 1.0 : 0.0;
        }
}

// ---------------------------------------------------------------------------
// k_paper_tan: columns [64 cb, 64 cb + 64) of interval k, wave `leg`.  Local
// body 0 is the torso, 1..D the links of the leg; rows zs[3 lb + q] (pose) and
// zs[3 LB + 3 lb + q] (velocity); the leg's contact rows y[0..3] and its share of
// the violation row y[4].  Bound by FP64 issue (280 instructions of a stage, 150 of
// them with a coefficient, which issue at half rate).  1,603 quad13 intervals, K = 20:
// 0.95 ms; the product with the dense M^-1 grad h^T A^-1 of every stage, read by
// scalar loads, took 5.6 ms.
// ---------------------------------------------------------------------------
template <class TP>
struct PLane {
    static constexpr int NR = 6 * TP::LB;
    double zb[NR], za[NR], zs[NR];
    double yc[5];
};

// a += coefficient IDX of the stage's vectors times x; b += coefficient IDY times z
template <int IDX, int NV>
__device__ __forceinline__ void pfma(double& a, const double (&v)[NV], double x) {
    fma_row<IDX & 15>(a, v[IDX >> 4], x);
}
template <int IDX, int IDY, int NV>
__device__ __forceinline__ void pfma2(double& a, double& b, const double (&v)[NV], double x,
                                      double z) {
    fma_row2<IDX & 15, IDY & 15>(a, b, v[IDX >> 4], v[IDY >> 4], x, z);
}

// a += coefficient I0 times x0 + coefficient I2 times x1; b likewise by I1, I3
template <int I0, int I1, int I2, int I3, int NV>
__device__ __forceinline__ void pfma22(double& a, double& b, const double (&v)[NV], double x0,
                                       double y0, double x1, double y1) {
    fma_row_pair2<I0 & 15, I1 & 15, I2 & 15, I3 & 15>(a, b, v[I0 >> 4], v[I1 >> 4], v[I2 >> 4],
                                                      v[I3 >> 4], x0, y0, x1, y1);
}
template <int I0, int I1, int I2, int I3, int NV>
__device__ __forceinline__ void pfma4(double& a0, double& a1, double& a2, double& a3,
                                      const double (&v)[NV], double x0, double x1, double x2,
                                      double x3) {
    fma_row4<I0 & 15, I1 & 15, I2 & 15, I3 & 15>(a0, a1, a2, a3, v[I0 >> 4], v[I1 >> 4],
                                                 v[I2 >> 4], v[I3 >> 4], x0, x1, x2, x3);
}

// Whether k_paper_tan holds the joint rows' form too: with three links the two do not
// fit the registers (120 bytes of scratch: 12,800 quad13 intervals 8.1 -> 9.9 ms), and
// that form has a launch of its own, which returns at once for other masses.
template <class TP>
constexpr bool PAPER_ONE = TP::D < 3;

// What a tangent lane is: hold weights, and its control's selection on this leg.
template <class TP>
struct PColumn {
    double wbm, wbp, fsel;
    bool tq[TP::D], ct, cn, cg;
};

template <class TP, int ST>
__device__ __forceinline__ void paper_tangent_stage(PLane<TP>& z, const PColumn<TP>& col,
                                                    const double (&v)[PRec<TP>::NV],
                                                    const double (&mass)[TP::D],
                                                    const double (&kd)[2 * TP::D], double s,
                                                    double h, double tau, double* xch, int leg,
                                                    int lane) {
    constexpr int D = TP::D, L = TP::L, LB = TP::LB;
    using R = PRec<TP>;
#define ZQ(lb, q) z.zs[3 * (lb) + (q)]
#define ZV(lb, q) z.zs[3 * LB + 3 * (lb) + (q)]
    // FOH weight of a B- / B+ column (0 for the other columns)
    const double w = col.wbm * (1.0 - tau) + col.wbp * tau;
    const double wt = col.ct ? w : 0.0, wn = col.cn ? w : 0.0, wg = col.cg ? w : 0.0;
    // ---- u: torques of the bodies, force at the tip; d: joint terms, summed from
    // the torso (dx, dy: link by link) ----
    double ut[LB], dx[D], dy[D];
#pragma unroll
    for (int lb = 0; lb < LB; ++lb) ut[lb] = 0.0;
    unrolled<D>([&](auto l_c) {
        constexpr int l = decltype(l_c)::value, J = R::JN * l;
        double t = -kd[2 * l] * (ZQ(l + 1, 2) - ZQ(l, 2)) - kd[2 * l + 1] * (ZV(l + 1, 2) - ZV(l, 2));
        t += col.tq[l] ? w : 0.0;
        ut[l] -= t;
        ut[l + 1] += t;
        pfma2<J + 12, J + 13>(ut[l], ut[l + 1], v, -ZQ(l, 2), ZQ(l + 1, 2));
        dx[l] = dy[l] = 0.0;
        pfma22<J + 4, J + 5, J + 6, J + 7>(dx[l], dy[l], v, ZQ(l, 2), ZQ(l, 2), ZQ(l + 1, 2),
                                           ZQ(l + 1, 2));
        pfma22<J + 8, J + 9, J + 10, J + 11>(dx[l], dy[l], v, ZV(l, 2), ZV(l, 2), ZV(l + 1, 2),
                                             ZV(l + 1, 2));
    });
    double fx = 0.0, fy = 0.0, tc = 0.0;
    pfma22<R::FXX, R::FYX, R::FXT, R::FYT>(fx, fy, v, ZQ(D, 0), ZQ(D, 0), ZQ(D, 2), ZQ(D, 2));
    pfma22<R::CTX, R::CTY, R::CNX, R::CNY>(fx, fy, v, wt, wt, wn, wn);
    pfma22<R::TQX, R::CTT, R::TQT, R::CTN>(ut[D], tc, v, ZQ(D, 0), wt, ZQ(D, 2), wn);
    ut[D] += tc;
    // ---- generalized forces f of the leg, and its part of the torso's system ----
    double f[D], px = 0.0, py = 0.0;   // (px, py): sum of u - m Gamma beyond a link
    {
        double Gx[D], Gy[D];
#pragma unroll
        for (int l = 0; l < D; ++l) {
            Gx[l] = l ? Gx[l > 0 ? l - 1 : 0] + dx[l] : dx[l];
            Gy[l] = l ? Gy[l > 0 ? l - 1 : 0] + dy[l] : dy[l];
        }
        unrolled<D>([&](auto e_c) {
            constexpr int l = D - 1 - decltype(e_c)::value, J = R::JN * l;
            // with E a_p of the next joint on the links beyond (px, py before)
            const double qx = px, qy = py;
            if constexpr (l == D - 1) {
                px = fma(-mass[l], Gx[l], fx);
                py = fma(-mass[l], Gy[l], fy);
            } else {
                px = fma(-mass[l], Gx[l], px);
                py = fma(-mass[l], Gy[l], py);
            }
            double t = ut[l + 1], q = 0.0;
            if constexpr (l < D - 1)
                pfma22<J + 3, J + R::JN, J + 2, J + R::JN + 1>(t, q, v, px, qy, -py, -qx);
            else
                pfma2<J + 3, J + 2>(t, q, v, px, -py);
            f[l] = t + q;
        });
    }
    double r0[3] = {px, py, ut[0]}, rt = 0.0;
    pfma2<0, 1>(r0[2], rt, v, py, -px);
    r0[2] += rt;
    unrolled<D>([&](auto l_c) {
        constexpr int l = decltype(l_c)::value;
        const double n = -f[l];
        fma_row3<(R::G + 3 * l) & 15, (R::G + 3 * l + 1) & 15, (R::G + 3 * l + 2) & 15>(
            r0[0], r0[1], r0[2], v[(R::G + 3 * l) >> 4], v[(R::G + 3 * l + 1) >> 4],
            v[(R::G + 3 * l + 2) >> 4], n, n, n);
    });
    // ---- exchange: the legs' parts ----
    if constexpr (L > 1) {
#pragma unroll
        for (int e = 0; e < 3; ++e) xch[(leg * 3 + e) * 64 + lane] = r0[e];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            double acc = 0.0;
#pragma unroll
            for (int l = 0; l < L; ++l) acc += xch[(l * 3 + e) * 64 + lane];
            r0[e] = acc;
        }
    }
    double a0[3] = {0.0, 0.0, 0.0}, kv[3 * LB];
    pfma22<R::SI, R::SI + 1, R::SI + 1, R::SI + 3>(a0[0], a0[1], v, r0[0], r0[0], r0[1], r0[1]);
    fma_row3<(R::SI + 2) & 15, (R::SI + 2) & 15, (R::SI + 4) & 15>(
        a0[2], a0[0], a0[1], v[(R::SI + 2) >> 4], v[(R::SI + 2) >> 4], v[(R::SI + 4) >> 4], r0[0],
        r0[2], r0[2]);
    fma_row_chain<(R::SI + 4) & 15, (R::SI + 5) & 15>(a0[2], v[(R::SI + 4) >> 4],
                                                      v[(R::SI + 5) >> 4], r0[1], r0[2]);
    // ---- angular accelerations of the leg, then the links' translations ----
    kv[0] = a0[0];
    kv[1] = a0[1];
    kv[2] = a0[2];
    const double n0[3] = {-a0[0], -a0[1], -a0[2]};
    unrolled<D>([&](auto l_c) {
        constexpr int l = decltype(l_c)::value;
        double t = 0.0, q = 0.0;
        constexpr int h0 = R::hi(l, 0), h1 = D > 1 ? (l >= 1 ? R::hi(l, 1) : R::hi(1, l)) : h0;
        if constexpr (D > 1)
            pfma22<R::G + 3 * l, h0, R::G + 3 * l + 1, h1>(t, q, v, n0[0], f[0], n0[1],
                                                           f[D > 1 ? 1 : 0]);
        else pfma22<R::G, h0, R::G + 1, R::G + 2>(t, q, v, n0[0], f[0], n0[1], n0[2]);
        if constexpr (D == 2) pfma<R::G + 3 * l + 2>(t, v, n0[2]);
        if constexpr (D == 3) pfma2<R::G + 3 * l + 2, R::hi(2, l)>(t, q, v, n0[2], f[D - 1]);
        static_assert(D <= 3, "a row of H^-1 is written out");
        kv[3 * (l + 1) + 2] = t + q;
    });
    double ax = a0[0], ay = a0[1];
    unrolled<D>([&](auto l_c) {
        constexpr int l = decltype(l_c)::value, J = R::JN * l;
        const double wp = kv[3 * l + 2], wc = kv[3 * l + 5];
        ax += dx[l];
        ay += dy[l];
        pfma22<J + 1, J, J + 3, J + 2>(ax, ay, v, -wp, wp, wc, -wc);
        kv[3 * l + 3] = ax;
        kv[3 * l + 4] = ay;
    });
    // ---- the leg's integral rows and its share of the violation row ----
    double ky[5] = {wn, 0.0, wg, 0.0, 0.0}, rc = 0.0;
    pfma22<R::LX, R::SX, R::LT, R::SY>(ky[1], ky[4], v, ZQ(D, 0), ZQ(D, 0), ZQ(D, 2), ZQ(D, 1));
    pfma22<R::CTX, R::ST, R::CTY, R::VN>(ky[1], ky[4], v, ZV(D, 0), ZQ(D, 2), ZV(D, 1), wn);
    pfma22<R::LW, R::VT, R::LCT, R::VG>(ky[1], ky[4], v, ZV(D, 2), wt, wt, wg);
    fma_row3<R::LCG & 15, R::RCN & 15, R::RCT & 15>(ky[1], ky[3], rc, v[R::LCG >> 4],
                                                   v[R::RCN >> 4], v[R::RCT >> 4], wg, wn, wt);
    ky[3] += rc;
#pragma unroll
    for (int q = 0; q < 5; ++q) ky[q] *= s;
    pfma4<R::YF, R::YF + 1, R::YF + 2, R::YF + 3>(ky[0], ky[1], ky[2], ky[3], v, col.fsel, col.fsel,
                                                  col.fsel, col.fsel);
    pfma<R::YF + 4>(ky[4], v, col.fsel);
    // ---- classical RK4 combination ----
    constexpr double wk = (ST == 0 || ST == 3) ? 1.0 : 2.0;
    const double an = ST == 2 ? h : 0.5 * h, h6 = h / 6.0;
    auto combine = [&](int r, double k) {
        z.za[r] = ST == 0 ? k : z.za[r] + wk * k;
        if constexpr (ST < 3) z.zs[r] = z.zb[r] + an * k;
        else z.zs[r] = z.zb[r] += h6 * z.za[r];
    };
    unrolled<LB>([&](auto b_c) {
        constexpr int lb = decltype(b_c)::value, F = R::SF + 6 * lb, r = 3 * lb, p = 3 * LB + r;
        double q0 = s * z.zs[p], q1 = s * z.zs[p + 1], q2 = s * z.zs[p + 2];
        double k0 = s * kv[r], k1 = s * kv[r + 1], k2 = s * kv[r + 2];
        const double fs = col.fsel;
        fma_row3<F & 15, (F + 1) & 15, (F + 2) & 15>(q0, q1, q2, v[F >> 4], v[(F + 1) >> 4],
                                                     v[(F + 2) >> 4], fs, fs, fs);
        fma_row3<(F + 3) & 15, (F + 4) & 15, (F + 5) & 15>(
            k0, k1, k2, v[(F + 3) >> 4], v[(F + 4) >> 4], v[(F + 5) >> 4], fs, fs, fs);
        combine(r, q0);
        combine(r + 1, q1);
        combine(r + 2, q2);
        combine(p, k0);
        combine(p + 1, k1);
        combine(p + 2, k2);
    });
#pragma unroll
    for (int q = 0; q < 5; ++q) z.yc[q] += (h6 * wk) * ky[q];
#undef ZQ
#undef ZV
}

template <class TP>
__global__ void __launch_bounds__(64 * TP::L) __attribute__((amdgpu_waves_per_eu(2)))
    k_paper_tan(PaperArgs a) {
    constexpr int N6 = TP::N6, NQ = TP::NQ, M = TP::M, D = TP::D, L = TP::L, LB = TP::LB;
    constexpr int NX = TP::NX, NC = TP::NC, NJ = TP::NJ;
    using R = PRec<TP>;
    __shared__ union {
        double xch[2][3 * L * 64];   // in turn, one barrier per stage
        std::conditional_t<PAPER_ONE<TP>, PDenseTan<TP>, char> rows;
    } lds;
    int k, cb;
    unit_item(xcd_slot(blockIdx.x, gridDim.x), a.N, TP::NBLK, k, cb);
    if (heavy_link<TP>(a.prm + 2)) {
        if constexpr (PAPER_ONE<TP>) paper_dense_tan<TP>(a, lds.rows, k, cb);
        return;
    }
    auto& xch = lds.xch;
    const int tid = threadIdx.x, lane = tid & 63;
    const int leg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = cb * 64 + lane;
    const bool active = col < TP::NCOL;
    auto gb = [&](int lb) { return lb == 0 ? 0 : 1 + leg * D + lb - 1; };
    PColumn<TP> pc;
    pc.wbm = pc.wbp = pc.fsel = 0.0;
    int ctrl = -1;
    if (col >= N6 && col < N6 + M) { pc.wbm = 1.0; ctrl = col - N6; }
    else if (col >= N6 + M && col < N6 + 2 * M) { pc.wbp = 1.0; ctrl = col - N6 - M; }
    else if (col == N6 + 2 * M) pc.fsel = 1.0;
#pragma unroll
    for (int l = 0; l < D; ++l) pc.tq[l] = ctrl == leg * D + l;
    pc.ct = ctrl == NJ + 3 * leg;
    pc.cn = ctrl == NJ + 3 * leg + 1;
    pc.cg = ctrl == NJ + 3 * leg + 2;
    PLane<TP> z;
#pragma unroll
    for (int lb = 0; lb < LB; ++lb)
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int g = 3 * gb(lb) + q;
            z.zb[3 * lb + q] = (g == col) ? 1.0 : 0.0;
            z.zb[3 * LB + 3 * lb + q] = (NQ + g == col) ? 1.0 : 0.0;
        }
#pragma unroll
    for (int r = 0; r < 6 * LB; ++r) {
        z.zs[r] = z.zb[r];
        z.za[r] = 0.0;
    }
#pragma unroll
    for (int q = 0; q < 5; ++q) z.yc[q] = 0.0;
    const double* hd = a.rec + (int64_t)k * R::per_interval(a.K);
    const double h = uniform(1.0 / double(a.K)), s = hd[0];
    double mass[D], kd[2 * D];
#pragma unroll
    for (int l = 0; l < D; ++l) {
        mass[l] = hd[8 + gb(l + 1)];
        kd[2 * l] = hd[8 + TP::NB + 2 * (leg * D + l)];
        kd[2 * l + 1] = hd[8 + TP::NB + 2 * (leg * D + l) + 1];
    }
    // the stage's coefficients, element lane & 15 of each vector; a stage ahead
    const double* at = hd + R::HDR + leg * R::LEG + (lane & 15);
    const double* last = at + (int64_t)(4 * a.K - 1) * R::STAGE;
    double v[2][R::NV];
    auto load = [&](double (&to)[R::NV]) {
#pragma unroll
        for (int q = 0; q < R::NV; ++q) to[q] = at[16 * q];
        at = at < last ? at + R::STAGE : last;
    };
    load(v[0]);
    for (int j = 0; j < a.K; ++j) {
        auto stage = [&](auto st_c) {
            constexpr int ST = decltype(st_c)::value;
            load(v[(ST + 1) & 1]);
            const double tau =
                uniform((double(j) + (ST == 0 ? 0.0 : (ST == 3 ? 1.0 : 0.5))) * h);
            paper_tangent_stage<TP, ST>(z, pc, v[ST & 1], mass, kd, s, h, tau, xch[ST & 1], leg,
                                        lane);
            __builtin_amdgcn_sched_barrier(0);
        };
        stage(std::integral_constant<int, 0>{});
        stage(std::integral_constant<int, 1>{});
        stage(std::integral_constant<int, 2>{});
        stage(std::integral_constant<int, 3>{});
    }
    // violation row: the legs' shares in leg order
    double yct = z.yc[4];
    if constexpr (L > 1) {
        xch[0][leg * 64 + lane] = yct;   // (last read before the last stage's barrier)
        __syncthreads();
        yct = 0.0;
#pragma unroll
        for (int l = 0; l < L; ++l) yct += xch[0][l * 64 + lane];
    }
    if (!active) return;
    const int64_t ldi = a.ldi;
    double* out;
    int64_t cstride, c0;   // element (row, column) at out[(row * cstride + c0) * ldi + k]
    if (col < N6) { out = a.A; cstride = NX; c0 = col; }
    else if (col < N6 + M) { out = a.Bm; cstride = M; c0 = col - N6; }
    else if (col < N6 + 2 * M) { out = a.Bp; cstride = M; c0 = col - N6 - M; }
    else { out = a.S; cstride = 1; c0 = 0; }
#pragma unroll
    for (int lb = 0; lb < LB; ++lb) {
        if (lb == 0 && leg != 0) continue;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int g = 3 * gb(lb) + q;
            out[((int64_t)g * cstride + c0) * ldi + k] = z.zb[3 * lb + q];
            out[((int64_t)(NQ + g) * cstride + c0) * ldi + k] = z.zb[3 * LB + 3 * lb + q];
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) out[((int64_t)(N6 + 4 * leg + q) * cstride + c0) * ldi + k] = z.yc[q];
    if (leg == 0) out[((int64_t)(N6 + 4 * NC) * cstride + c0) * ldi + k] = yct;
}

// The joint rows' form by itself.  (The columns: one workgroup for each part of each interval:
// in a loop over them the records' reads are no longer scalar loads, 57 -> 815 ms for
// 12,800 quad13 intervals.)
template <class TP>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
    k_paper_rec_rows(PaperArgs a, MConst<TP::NB, TP::NJ, TP::NC> mc) {
    __shared__ PDenseShared<TP> lds;
    if (heavy_link<TP>(a.prm + 2))
        paper_dense_rec<TP>(a, mc, lds, xcd_slot(blockIdx.x, gridDim.x));
}

template <class TP>
__global__ void __launch_bounds__(64 * TP::L) __attribute__((amdgpu_waves_per_eu(2)))
    k_paper_tan_rows(PaperArgs a) {
    __shared__ PDenseTan<TP> lds;
    if (!heavy_link<TP>(a.prm + 2)) return;
    int k, cb;
    unit_item(xcd_slot(blockIdx.x, gridDim.x), a.N, TP::NBLK, k, cb);
    paper_dense_tan<TP>(a, lds, k, cb);
}

template <int L, int D>
static cis_status launch_paper_t(const cis_model* m, const PaperArgs& a, hipStream_t stream) {
    if constexpr (L >= 1 && D >= 1) {
        using TP = PTopo<L, D>;
        const auto mc = make_const<TP::NB, TP::NJ, TP::NC>(m);
        // The masses are on the device, so both forms are launched and one returns at once.
        // Up to one interval per SIMD the records of both take one launch (with a launch
        // each, a call of 8 hopper intervals, K = 1, took 33 us instead of 28); beyond, the
        // joint rows' form needs the second wave per SIMD that the registers of the other
        // do not leave (a heavy tip, hopper, K = 20: 1,000 intervals 353 us in one launch
        // and 355 in two, 5,000 1,452 and 1,043).
        if (a.N <= 4 * device_cus()) {
            hipLaunchKernelGGL((k_paper_rec<TP, true>), dim3(a.N), dim3(64), 0, stream, a, mc);
        } else {
            hipLaunchKernelGGL((k_paper_rec<TP, false>), dim3((a.N + 3) / 4), dim3(64), 0, stream,
                               a, mc);
            hipLaunchKernelGGL(k_paper_rec_rows<TP>, dim3(a.N), dim3(64), 0, stream, a, mc);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(CIS_ERR_HIP, "k_paper_rec launch: %s", hipGetErrorString(e));
        hipLaunchKernelGGL(k_paper_tan<TP>, dim3(a.N * TP::NBLK), dim3(64 * TP::L), 0, stream, a);
        e = hipGetLastError();
        if (e != hipSuccess) return fail(CIS_ERR_HIP, "k_paper_tan launch: %s", hipGetErrorString(e));
        if constexpr (!PAPER_ONE<TP>) {
            hipLaunchKernelGGL(k_paper_tan_rows<TP>, dim3(a.N * TP::NBLK), dim3(64 * TP::L), 0,
                               stream, a);
            e = hipGetLastError();
            if (e != hipSuccess)
                return fail(CIS_ERR_HIP, "k_paper_tan_rows launch: %s", hipGetErrorString(e));
        }
        return CIS_OK;
    } else {
        return fail(CIS_ERR_UNSUPPORTED, "the paper-dynamics form needs legs with links");
    }
}

template <int L, int D>
static int64_t paper_elems_t(int K) {
    if constexpr (L >= 1 && D >= 1)
        return std::max(PRec<PTopo<L, D>>::per_interval(K), PDenseRec<PTopo<L, D>>::per_interval(K));
    else return -1;
}

static int64_t paper_elems(const cis_model* m, int K) {
#define CIS_PAPER_SZ(LL, DD) \
    if (m->L == LL && m->D == DD) return paper_elems_t<LL, DD>(K);
    CIS_TOPOLOGIES(CIS_PAPER_SZ)
#undef CIS_PAPER_SZ
    return -1;
}

}  // namespace cis

using namespace cis;

extern "C" cis_status cis_paper_dims(const cis_model* model, int32_t* nx, int32_t* m) {
    if (!model) return fail(CIS_ERR_NULL, "cis_paper_dims: model is required");
    if (nx) *nx = 6 * model->nb + 4 * model->nc + 1;
    if (m) *m = model->nj + 3 * model->nc;
    return CIS_OK;
}

extern "C" cis_status cis_paper_workspace_size(const cis_model* m, const cis_shape* sh,
                                               size_t* bytes) {
    if (!m || !sh || !bytes) return fail(CIS_ERR_NULL, "cis_paper_workspace_size: null argument");
    if (sh->N < 1 || sh->substeps < 1 || sh->substeps > 4096)
        return fail(CIS_ERR_DIM, "cis_paper_workspace_size: N=%d, K=%d out of range", sh->N,
                    sh->substeps);
    if (sh->dtype != CIS_F64)
        return fail(CIS_ERR_DTYPE, "cis_paper_workspace_size: the paper-dynamics form is FP64 only");
    const int64_t per = paper_elems(m, sh->substeps);
    if (per < 0) return fail(CIS_ERR_UNSUPPORTED, "paper-dynamics form: the model has no legs with links");
    *bytes = (size_t)per * (size_t)sh->N * sizeof(double);
    return CIS_OK;
}

static cis_status discretize_paper_impl(const cis_model* model, const cis_shape* shape,
                                        const void* X, const void* U, const void* s,
                                        const void* params, void* A, void* Bm, void* Bp,
                                        void* S, void* defect, void* xprop, void* ws,
                                        size_t ws_bytes, void* stream) {
    cis_status st = check_common(model, shape, X, U, s, params);
    if (st != CIS_OK) return st;
    if (shape->dtype != CIS_F64)
        return fail(CIS_ERR_DTYPE, "cis_discretize_paper: FP64 only");
    if (!A || !Bm || !Bp || !S || !defect)
        return fail(CIS_ERR_NULL, "cis_discretize_paper: A, Bm, Bp, S and defect are required");
    if (!aligned(A, 8) || !aligned(S, 8) || !aligned(defect, 8) || !aligned(xprop, 8) ||
        !aligned(Bm, 8) || !aligned(Bp, 8) || !aligned(ws, 8))
        return fail(CIS_ERR_LAYOUT, "cis_discretize_paper: pointer not aligned to 8 bytes");
    size_t need = 0;
    st = cis_paper_workspace_size(model, shape, &need);
    if (st != CIS_OK) return st;
    if (!ws || ws_bytes < need)
        return fail(CIS_ERR_WORKSPACE, "cis_discretize_paper: workspace of %zu bytes needed", need);
    PaperArgs a;
    a.X = (const double*)X;
    a.U = (const double*)U;
    a.s = (const double*)s;
    a.prm = (const double*)params;
    a.A = (double*)A;
    a.Bm = (double*)Bm;
    a.Bp = (double*)Bp;
    a.S = (double*)S;
    a.defect = (double*)defect;
    a.xprop = (double*)xprop;
    a.rec = (double*)ws;
    a.ldn = shape->ld_node;
    a.ldi = shape->ld_int;
    a.N = shape->N;
    a.K = shape->substeps;
    hipStream_t hs = (hipStream_t)stream;
#define CIS_DISPATCH_PAPER(LL, DD) \
    if (model->L == LL && model->D == DD) return launch_paper_t<LL, DD>(model, a, hs);
    CIS_TOPOLOGIES(CIS_DISPATCH_PAPER)
#undef CIS_DISPATCH_PAPER
    return fail(CIS_ERR_UNSUPPORTED, "cis_discretize_paper: topology has no compiled kernel");
}

extern "C" cis_status cis_discretize_paper(const cis_model* model, const cis_shape* shape,
                                           const void* X, const void* U, const void* s,
                                           const void* params, void* A, void* Bm, void* Bp,
                                           void* S, void* defect, void* xprop, void* ws,
                                           size_t ws_bytes, void* stream) {
    cis_status st = discretize_paper_impl(model, shape, X, U, s, params, A, Bm, Bp, S, defect,
                                          xprop, ws, ws_bytes, stream);
    if (st != CIS_OK || !debug_finite_enabled()) return st;
    int32_t nx = 0, nu = 0;
    st = cis_paper_dims(model, &nx, &nu);
    if (st != CIS_OK) return st;
    return debug_scan_forward("cis_discretize_paper", model, shape, nx, nu, X, U, s, params, A,
                              Bm, Bp, S, defect, xprop, nullptr, stream);
}
