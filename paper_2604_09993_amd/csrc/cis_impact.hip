// Node-level impact map and impact conditions of the transcribed problem, with
// their Jacobians (arxiv 2604.09993, Sec. II-B eq. impulse-dynamics and the
// elimination of the joint impulse that follows it; Sec. IV-C eq. FB-relax,
// eq. cito-impulse and the constraint families Theta^delta and Psi^{delta,eps}).
//
// One wave per node.  The joint impulses are eliminated leg by leg: grad h v* = 0 gives
// every link's translation from the torso's velocity a0 = (v_0, w_0) and the angular
// velocities of its leg,
//     v_l = v_0 + w_0 E a_p1 + sum_{i<=l} w_i E r_li,  r_li = a_p,i+1 - a_c,i (i < l),
//     r_ll = -a_c,l,  E a = (-a_y, a_x),
// and the momenta along the w_i leave, per leg, H w = f - H0 a0 (as many rows as the leg
// has links) and a 3 x 3 system of the torso.  So v* = T a0 + (the leg's own response),
// with T the motion of every body row under the torso's.
// A Jacobian column of the velocity jump touches one body: its momenta m du, du = df +
// d(M^-1) grad h^T Lambda + M^-1 dgrad_h^T Lambda, and for an angle the change of grad h
// act on that body's leg, and the rest of the machine follows through T.  One lane
// forms a column: the response of one leg, the torso's, then three products a row.
// Bound by FP64 issue up to some thousand nodes (4,000 quad13 nodes: 98 -> 44 us), then
// by the stores (470 MB of 12,864 nodes: 252 -> 182 us); before, a Gauss-Jordan
// elimination of the 24 joint rows and eight products a row.  The
// impact conditions of a contact depend on 14 node variables; one lane per
// (contact, variable) evaluates them in dual numbers.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>

#include "../../include/cis.h"
#include "cis_host.hpp"
#include "cis_model.hpp"
#include "cis_reduced.hpp"

namespace cis {

template <int L_, int D_>
struct ImpTopo {
    static constexpr int L = L_, D = D_;
    static constexpr int NB = 1 + L * D, NJ = L * D, NC = L;
    static constexpr int NQ = 3 * NB, NY = NC + 1, NXT = 6 * NB + NY;
    static constexpr int NJ2 = 2 * NJ, P = NB + 2, DM = cmax(D, 1), LM = cmax(L, 1);
    static constexpr int NTV = (3 * NQ + 15) / 16;     // T in vectors of 16
    static constexpr int NQP = NQ + (NQ & 1);          // row stride of X in LDS
    static constexpr int NCV = 2 * NQ + 2 * NC + NB;   // columns of JGv
    static constexpr int NTH = 10 * NC;                // rows of Theta
    static constexpr int NCT = 14;                     // columns of JTc
    static constexpr int ADJ = L > 2 ? L : 2;          // joints at one body, at most
    static constexpr int NIN = 2 * NXT + 3 * NC;       // node inputs (x+, x-, Phi, Gamma)
    static_assert(NJ2 + NQ + 1 <= 64, "one lane per column of the augmented system");
    static_assert(NCT * NC <= 64, "one lane per (contact, variable)");
    static_assert(32 + 5 * NC <= 64, "one lane per (contact, wrench direction)");
    __host__ __device__ static constexpr int parent(int j) {
        return D == 0 ? 0 : ((j % D == 0) ? 0 : j);
    }
    __host__ __device__ static constexpr int cbody(int i) { return D * (i + 1); }
    // contact carried by body b, or -1
    __host__ __device__ static constexpr int contact_at(int b) {
        if (NC == 0) return -1;
        if (D == 0) return b == 0 ? 0 : -1;
        return (b >= 1 && (b - 1) % D == D - 1) ? (b - 1) / D : -1;
    }
    // slot s of the joints at body b: the joint index, whether b is its parent
    __host__ __device__ static constexpr int slot_joint(int b, int s, bool& b_is_parent) {
        b_is_parent = false;
        if (NJ == 0) return -1;
        if (b == 0) {
            b_is_parent = true;
            return s < L ? s * D : -1;
        }
        if (s == 0) return b - 1;                             // the joint above b
        b_is_parent = true;
        return (s == 1 && (b - 1) % D != D - 1) ? b : -1;     // the joint below b
    }
};

// ---------------------------------------------------------------------------
// Dual numbers (value, directional derivative) for the contact terms.
// ---------------------------------------------------------------------------
struct Dual {
    double v, d;
};
__device__ __forceinline__ Dual dn(double v, double d = 0.0) { return Dual{v, d}; }
__device__ __forceinline__ Dual operator+(Dual a, Dual b) { return {a.v + b.v, a.d + b.d}; }
__device__ __forceinline__ Dual operator-(Dual a, Dual b) { return {a.v - b.v, a.d - b.d}; }
__device__ __forceinline__ Dual operator-(Dual a) { return {-a.v, -a.d}; }
__device__ __forceinline__ Dual operator*(Dual a, Dual b) {
    return {a.v * b.v, fma(a.d, b.v, a.v * b.d)};
}
__device__ __forceinline__ Dual operator*(double a, Dual b) { return {a * b.v, a * b.d}; }
__device__ __forceinline__ Dual operator/(Dual a, Dual b) {   // |b.v| >= 1 wherever it is used
    // a residual that is no number: an operand is infinite, and a.v r the quotient
    const double r = 1.0 / b.v, q0 = a.v * r, e = fma(-q0, b.v, a.v);
    const double q = e == e ? fma(e, r, q0) : q0;
    return {q, (a.d - q * b.d) * r};
}
__device__ __forceinline__ Dual dsqrt(Dual a) {   // a.v > 0 wherever it is used
    // hardware estimate, two residual steps, and one on the root itself
    const double y = rsqrt_t<true>(a.v), s = a.v * y, v = fma(fma(-s, s, a.v), 0.5 * y, s);
    return {a.v < HUGE_VAL ? v : a.v, a.d * (0.5 * y)};
}
__device__ __forceinline__ void dsincos(Dual a, Dual& s, Dual& c) {
    double sv, cv;
    sincos_t(a.v, &sv, &cv);
    s = {sv, cv * a.d};
    c = {cv, -sv * a.d};
}
// pseudo-Huber absolute value sqrt(a^2+1) - 1, written a^2 / (sqrt(a^2+1) + 1)
__device__ __forceinline__ Dual dsabs(Dual a) {
    const Dual r = dsqrt(a * a + dn(1.0));
    return (a * a) / (r + dn(1.0));
}
// Fischer-Burmeister relaxation a + b - sqrt(a^2 + b^2 + delta), delta > 0
__device__ __forceinline__ Dual dfb(Dual a, Dual b, double delta) {
    return a + b - dsqrt(a * a + b * b + dn(delta));
}

// Contact frame at P (Sec. II; terrain h = P_y - A sin(kappa P_x), signed
// distance h / ||grad h|| as in Sec. VI-B): sd, normal n, tangent t = (n_y, -n_x).
template <class MC>
__device__ __forceinline__ void frame_d(const MC& mc, Dual Px, Dual Py, Dual& sd, Dual& nx,
                                        Dual& ny, Dual& tx, Dual& ty) {
    Dual sw, cw;
    dsincos(mc.kappa * Px, sw, cw);
    const Dual H = Py - mc.A * sw;
    const Dual Hx = (-mc.A * mc.kappa) * cw;
    const Dual w = dn(1.0) + Hx * Hx;
    const double y = rsqrt_t(w.v);
    const Dual rG = dn(y, -0.5 * (y * y * y) * w.d);   // 1 / ||grad h||
    sd = H * rG;
    nx = Hx * rG;
    ny = rG;
    tx = ny;
    ty = -nx;
}

// World-frame contact impulse R Phi = t Phi_t + n Phi_n at contact i of a body
// at (x, y, th), and its generalized force on that body (force, moment of the
// force about the body origin).
template <class MC>
__device__ __forceinline__ void contact_wrench(const MC& mc, int i, Dual x, Dual y, Dual th,
                                               Dual pt, Dual pn, Dual& Fx, Dual& Fy, Dual& Tq) {
    Dual s, c;
    dsincos(th, s, c);
    const double rx = mc.cr[i][0], ry = mc.cr[i][1];
    const Dual ax = rx * c - ry * s, ay = rx * s + ry * c;
    Dual sd, nx, ny, tx, ty;
    frame_d(mc, x + ax, y + ay, sd, nx, ny, tx, ty);
    Fx = tx * pt + nx * pn;
    Fy = ty * pt + ny * pn;
    Tq = ax * Fy - ay * Fx;
}

template <class TP>
struct ImpLegs {
    // links: r_li (l > i), sum_{l >= i} m_l r_li, their momenta's f, then w of the node
    double rho[cmax(TP::NJ, 1)][2], sig[cmax(TP::NJ, 1)][2], hd[cmax(TP::NJ, 1)];
    double fg[cmax(TP::NJ, 1)], w[cmax(TP::NJ, 1)];
    double Hi[TP::LM][TP::DM][TP::DM], G[TP::LM][TP::DM][3];   // H^-1, H^-1 H0
    double S[TP::LM][9];                // the legs' parts of the torso's system
    double T[16 * TP::NTV];             // [NQ][3]
};

template <class TP>
struct ImpShared {
    double z[TP::NIN];                  // x+ | x- | Phi | Gamma of the node
    double ynext[TP::NY];               // integral states of x- at the next node
    double prm[TP::P];
    double cs[TP::NB][2];               // cos, sin of the post-impact angles
    double minv[TP::NQ];                // diagonal of M^-1
    double arm[cmax(TP::NJ, 1)][4];     // world-frame joint arms a_p, a_c
    double cw[cmax(TP::NC, 1)][3];      // generalized contact force on the contact body
    double f[TP::NQ];                   // v- + M^-1 J^T R Phi
    double vs[TP::NQ];                  // v*
    double lam[cmax(TP::NJ2, 1)];       // Lambda
    union {
        ImpLegs<TP> leg;
        double X[cmax(TP::NJ2, 1)][TP::NQP];   // A^-1 grad h M^-1 (heavy bodies)
    };
    double dw[cmax(TP::NC, 1)][5][3];   // d(contact wrench)/d(x_b, y_b, th_b, Phi_t, Phi_n)
};

// value of v in lane `src` (wave-uniform), in every lane
__device__ __forceinline__ double bcast(double v, int src) {
    const int2 w = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_readlane(w.x, src),
                                                __builtin_amdgcn_readlane(w.y, src)));
}

__device__ __forceinline__ void lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

struct ImpactArgs {
    const double* Xp;      // [nx][ld]
    const double* Xm;      // [nx][ld]
    const double* Phi;     // [2 nc][ld]
    const double* Gam;     // [nc][ld]
    const double* prm;     // [P]
    double* G;             // [n][nx]
    double* Theta;         // [n][10 nc]
    double* JGv;           // [n][3 nb][NCV]
    double* JTc;           // [n][10 nc][14]
    double* Psi;           // [n-1][ny] or null
    int64_t ld;
    int n;
    double delta, eps;
};

// The joint rows' system, for models with a link much heavier than what lies between
// it and the torso, or a fixed body (heavy_link): it takes 1/m.  12,864 quad13 nodes
// with a heavy tip: 251 us (500: 29 us; with every row's reads in flight at once, which
// held 516 bytes of scratch per lane, 440 us and 54 us).
// X = A^-1 grad h M^-1, A = grad h M^-1 grad h^T, and Lambda = -A^-1 grad h f by
// Gauss-Jordan elimination of [A | grad h M^-1 | grad h f], a lane per column, the
// pivot column by lane reads; then v* = f + M^-1 grad h^T Lambda.
template <class TP>
__device__ __forceinline__ void impact_dense(ImpShared<TP>& sh, int lane) {
    constexpr int NJ = TP::NJ, NJ2 = TP::NJ2, NQ = TP::NQ, W = NJ2 + NQ + 1;
    const int l = lane < W ? lane : W - 1;   // (spare lanes repeat the last column)
    // the lane's column before grad h, entry by entry: a factor on 1/m (or on f), which
    // is +-1 or an arm's component at one or two bodies (a joint row), or 1 at one entry
    const double* base = l < NJ2 + NQ ? sh.minv : sh.f;
    const int jl = l < NJ2 ? l >> 1 : 0, cl = l & 1;
    const int pl = l < NJ2 ? TP::parent(jl) : -1, chl = l < NJ2 ? jl + 1 : -1;
    const double epl = cl == 0 ? -sh.arm[jl][1] : sh.arm[jl][0];
    const double ecl = cl == 0 ? sh.arm[jl][3] : -sh.arm[jl][2];
    auto y = [&](int r) {
        const int b = r / 3, q = r - 3 * b;
        double w = l - NJ2 == r || l == W - 1 ? 1.0 : 0.0;
        const double wp = q == 2 ? epl : (q == cl ? 1.0 : 0.0);
        const double wc = q == 2 ? ecl : (q == cl ? -1.0 : 0.0);
        if (b == pl) w = wp;
        if (b == chl) w = wc;
        return base[r] * w;
    };
    double col[NJ2];
#pragma unroll
    for (int i = 0; i < NJ2; ++i) {
        const int j = i >> 1, c = i & 1, p = TP::parent(j), ch = j + 1;
        const double ep = c == 0 ? -sh.arm[j][1] : sh.arm[j][0];
        const double ec = c == 0 ? -sh.arm[j][3] : sh.arm[j][2];
        col[i] = (y(3 * p + c) + y(3 * p + 2) * ep) - (y(3 * ch + c) + y(3 * ch + 2) * ec);
        // (a few rows at a time: the reads of all of them do not fit the registers)
        if (i % 4 == 3) {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int kk = 0; kk < NJ2; ++kk) {
        const double t = col[kk] / bcast(col[kk], kk);
#pragma unroll
        for (int i = 0; i < NJ2; ++i) col[i] = i == kk ? t : fma(-bcast(col[i], kk), t, col[i]);
    }
    if (lane >= NJ2 && lane < NJ2 + NQ)
#pragma unroll
        for (int i = 0; i < NJ2; ++i) sh.X[i][lane - NJ2] = col[i];
    if (lane == NJ2 + NQ)
#pragma unroll
        for (int i = 0; i < NJ2; ++i) sh.lam[i] = -col[i];
    lds_sync();
    if (lane < NQ) {   // (the joints at the row's body)
        const int b = lane / 3, q = lane - 3 * b;
        double jt = 0.0;
#pragma unroll
        for (int e = 0; e < TP::ADJ; ++e) {
            bool par;
            const int j = TP::slot_joint(b, e, par);
            if (j < 0) continue;
            const double lx = sh.lam[2 * j], ly = sh.lam[2 * j + 1];
            const double ax = par ? sh.arm[j][0] : sh.arm[j][2];
            const double ay = par ? sh.arm[j][1] : sh.arm[j][3];
            const double v = q == 0 ? lx : (q == 1 ? ly : ax * ly - ay * lx);
            jt += par ? v : -v;
        }
        sh.vs[lane] = sh.f[lane] + sh.minv[lane] * jt;
    }
}

template <class TP>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3)))
    k_impact(ImpactArgs a, MConst<TP::NB, TP::NJ, TP::NC> mc) {
    constexpr int NB = TP::NB, NJ = TP::NJ, NC = TP::NC, NQ = TP::NQ, NY = TP::NY;
    constexpr int NXT = TP::NXT, NCV = TP::NCV, NIN = TP::NIN;
    __shared__ ImpShared<TP> sh;
    const int lane = threadIdx.x;
    const int k = xcd_slot(blockIdx.x, gridDim.x);
    if (k >= a.n) return;   // whole wave
    const int64_t ld = a.ld;

    // ---- node inputs -------------------------------------------------------
    for (int r = lane; r < NIN; r += 64) {
        const double* src = r < NXT ? a.Xp + (int64_t)r * ld
                          : r < 2 * NXT ? a.Xm + (int64_t)(r - NXT) * ld
                          : r < 2 * NXT + 2 * NC ? a.Phi + (int64_t)(r - 2 * NXT) * ld
                                                 : a.Gam + (int64_t)(r - 2 * NXT - 2 * NC) * ld;
        sh.z[r] = src[k];
    }
    if (lane < TP::P) sh.prm[lane] = a.prm[lane];
    if (a.Psi && lane < NY && k + 1 < a.n) sh.ynext[lane] = a.Xm[(int64_t)(6 * NB + lane) * ld + k + 1];
    lds_sync();
    const double* qp = sh.z;              // post-impact pose
    const double* vp = sh.z + NQ;         // post-impact velocity
    const double* qm = sh.z + NXT;
    const double* vm = sh.z + NXT + NQ;
    const double* phi = sh.z + 2 * NXT;
    const double* gam = sh.z + 2 * NXT + 2 * NC;

    // ---- rotations, M^-1 ---------------------------------------------------
    if (lane < NB) {
        double sn, cn;
        sincos_t(qp[3 * lane + 2], &sn, &cn);
        sh.cs[lane][0] = cn;
        sh.cs[lane][1] = sn;
        const double m = sh.prm[2 + lane];
        sh.minv[3 * lane] = 1.0 / m;
        sh.minv[3 * lane + 1] = 1.0 / m;
        sh.minv[3 * lane + 2] = 1.0 / (m * mc.ipm[lane]);
    }
    lds_sync();
    // ---- joint arms, contact wrenches --------------------------------------
    if constexpr (NJ > 0) {
        if (lane < NJ) {
            const int p = TP::parent(lane), c = lane + 1;
            const double cp = sh.cs[p][0], sp = sh.cs[p][1], cc = sh.cs[c][0], sc = sh.cs[c][1];
            sh.arm[lane][0] = cp * mc.rp[lane][0] - sp * mc.rp[lane][1];
            sh.arm[lane][1] = sp * mc.rp[lane][0] + cp * mc.rp[lane][1];
            sh.arm[lane][2] = cc * mc.rc[lane][0] - sc * mc.rc[lane][1];
            sh.arm[lane][3] = sc * mc.rc[lane][0] + cc * mc.rc[lane][1];
        }
    }
    if constexpr (NC > 0) {
        // lane 32 + 5 i + d: the wrench of contact i and its derivative along
        // direction d of (x_b, y_b, th_b, Phi_t, Phi_n)
        if (lane >= 32 && lane < 32 + 5 * NC) {
            const int i = (lane - 32) / 5, d = lane - 32 - 5 * i, b = TP::cbody(i);
            Dual Fx, Fy, Tq;
            contact_wrench(mc, i, dn(qp[3 * b], d == 0), dn(qp[3 * b + 1], d == 1),
                           dn(qp[3 * b + 2], d == 2), dn(phi[2 * i], d == 3),
                           dn(phi[2 * i + 1], d == 4), Fx, Fy, Tq);
            if (d == 0) {
                sh.cw[i][0] = Fx.v;
                sh.cw[i][1] = Fy.v;
                sh.cw[i][2] = Tq.v;
            }
            sh.dw[i][d][0] = Fx.d;
            sh.dw[i][d][1] = Fy.d;
            sh.dw[i][d][2] = Tq.d;
        }
    }
    lds_sync();
    if (lane < NQ) {
        const int b = lane / 3, q = lane - 3 * b, i = TP::contact_at(b);
        const double gen = i >= 0 ? sh.cw[i < 0 ? 0 : i][q] : 0.0;
        sh.f[lane] = vm[lane] + sh.minv[lane] * gen;
    }
    lds_sync();

    // ---- v* = f + M^-1 grad h^T Lambda, grad h v* = 0 ------------------------
    const bool heavy = NJ > 0 && heavy_link<TP>(sh.prm + 2);
    double si[3][3], Z[3] = {0.0, 0.0, 0.0};   // the torso's inverse; its system by a_p1
    if constexpr (NJ > 0) {
        if (heavy) {
            impact_dense<TP>(sh, lane);
        } else {
            constexpr int D = TP::D, L = TP::L;
            const double* mass = sh.prm + 2;
            if (lane < NJ) {
                const int c = lane + 1, lk = lane % D;
                const double m = mass[c], I = m * mc.ipm[c];
                const double acx = sh.arm[lane][2], acy = sh.arm[lane][3];
                double msub = 0.0, qx = 0.0, qy = 0.0;   // links beyond: mass, momentum
#pragma unroll
                for (int e = 1; e < D; ++e)
                    if (lk + e < D) {
                        const double me = mass[c + e];
                        msub += me;
                        qx += me * sh.f[3 * (c + e)];
                        qy += me * sh.f[3 * (c + e) + 1];
                    }
                const bool inner = lk + 1 < D;
                const int nx = inner ? lane + 1 : lane;
                const double rx = inner ? sh.arm[nx][0] - acx : 0.0;
                const double ry = inner ? sh.arm[nx][1] - acy : 0.0;
                const double px = m * sh.f[3 * c], py = m * sh.f[3 * c + 1];
                sh.leg.rho[lane][0] = rx;
                sh.leg.rho[lane][1] = ry;
                sh.leg.sig[lane][0] = msub * rx - m * acx;
                sh.leg.sig[lane][1] = msub * ry - m * acy;
                sh.leg.hd[lane] = I + m * (acx * acx + acy * acy) + msub * (rx * rx + ry * ry);
                sh.leg.fg[lane] = I * sh.f[3 * c + 2] + (acy * px - acx * py) + (rx * qy - ry * qx);
            }
            lds_sync();
            if (lane < L) {   // a leg's system
                const int j0 = lane * D;
                const double a1x = sh.arm[j0][0], a1y = sh.arm[j0][1];
                double H[D][D], H0[D][3], f[D], ml = 0.0, tx = 0.0, ty = 0.0;
#pragma unroll
                for (int i = 0; i < D; ++i) {
                    const double ex = sh.leg.sig[j0 + i][0], ey = sh.leg.sig[j0 + i][1];
                    H[i][i] = sh.leg.hd[j0 + i];
                    f[i] = sh.leg.fg[j0 + i];
                    H0[i][0] = -ey;
                    H0[i][1] = ex;
                    H0[i][2] = ex * a1x + ey * a1y;
#pragma unroll
                    for (int l = i + 1; l < D; ++l)
                        H[i][l] = H[l][i] = sh.leg.rho[j0 + i][0] * sh.leg.sig[j0 + l][0] +
                                            sh.leg.rho[j0 + i][1] * sh.leg.sig[j0 + l][1];
                    const double m = mass[j0 + i + 1];
                    ml += m;
                    tx += m * sh.f[3 * (j0 + i + 1)];
                    ty += m * sh.f[3 * (j0 + i + 1) + 1];
                }
                spd_inverse<D>(H);
                double S[9] = {ml, 0.0, -ml * a1y, ml, ml * a1x, ml * (a1x * a1x + a1y * a1y),
                               tx, ty, a1x * ty - a1y * tx};
#pragma unroll
                for (int i = 0; i < D; ++i) {
                    double y = 0.0, g[3] = {0.0, 0.0, 0.0};
#pragma unroll
                    for (int l = 0; l < D; ++l) {
                        y += H[i][l] * f[l];
#pragma unroll
                        for (int e = 0; e < 3; ++e) g[e] += H[i][l] * H0[l][e];
                        sh.leg.Hi[lane][i][l] = H[i][l];
                    }
                    sh.leg.w[j0 + i] = y;
                    S[0] -= H0[i][0] * g[0];
                    S[1] -= H0[i][0] * g[1];
                    S[2] -= H0[i][0] * g[2];
                    S[3] -= H0[i][1] * g[1];
                    S[4] -= H0[i][1] * g[2];
                    S[5] -= H0[i][2] * g[2];
#pragma unroll
                    for (int e = 0; e < 3; ++e) {
                        S[6 + e] -= H0[i][e] * y;
                        sh.leg.G[lane][i][e] = g[e];
                    }
                }
#pragma unroll
                for (int e = 0; e < 9; ++e) sh.leg.S[lane][e] = S[e];
            }
            lds_sync();
            double s[9] = {mass[0], 0.0, 0.0, mass[0], 0.0, mass[0] * mc.ipm[0],
                           mass[0] * sh.f[0], mass[0] * sh.f[1], mass[0] * mc.ipm[0] * sh.f[2]};
#pragma unroll
            for (int l = 0; l < L; ++l) {
                double v[9];
#pragma unroll
                for (int e = 0; e < 9; ++e) {
                    v[e] = sh.leg.S[l][e];
                    s[e] += v[e];
                }
                const double ax = sh.arm[l * D][0], ay = sh.arm[l * D][1];
                Z[0] += v[0] * ax + v[1] * ay;
                Z[1] += v[1] * ax + v[3] * ay;
                Z[2] += v[2] * ax + v[4] * ay;
            }
            si[0][0] = s[0];
            si[1][1] = s[3];
            si[2][2] = s[5];
            si[0][1] = si[1][0] = s[1];
            si[0][2] = si[2][0] = s[2];
            si[1][2] = si[2][1] = s[4];
            spd_inverse<3>(si);
            double a0[3];
#pragma unroll
            for (int e = 0; e < 3; ++e) a0[e] = si[e][0] * s[6] + si[e][1] * s[7] + si[e][2] * s[8];
            if (lane < NQ) {
                const int b = lane / 3, q = lane - 3 * b;
                const int leg = b > 0 ? (b - 1) / D : 0, lk = b > 0 ? (b - 1) % D : 0, j0 = leg * D;
                double t[3] = {q == 0 ? 1.0 : 0.0, q == 1 ? 1.0 : 0.0, q == 2 ? 1.0 : 0.0}, own = 0.0;
                if (b > 0) {
                    t[2] = q == 0 ? -sh.arm[j0][1] : (q == 1 ? sh.arm[j0][0] : 0.0);
#pragma unroll
                    for (int i = 0; i < D; ++i) {
                        // row of E r_li (or the angle itself)
                        const double rx = i < lk ? sh.leg.rho[j0 + i][0] : -sh.arm[j0 + i][2];
                        const double ry = i < lk ? sh.leg.rho[j0 + i][1] : -sh.arm[j0 + i][3];
                        double er = q == 0 ? -ry : (q == 1 ? rx : 0.0);
                        if (i > lk) er = 0.0;
                        if (q == 2 && i == lk) er = 1.0;
                        own += er * sh.leg.w[j0 + i];
#pragma unroll
                        for (int e = 0; e < 3; ++e) t[e] -= er * sh.leg.G[leg][i][e];
                    }
                }
#pragma unroll
                for (int e = 0; e < 3; ++e) sh.leg.T[3 * lane + e] = t[e];
                sh.vs[lane] = (t[0] * a0[0] + t[1] * a0[1] + t[2] * a0[2]) + own;
            }
            lds_sync();
            if (lane < NJ) {   // joint impulses, from the tip
                double lx = 0.0, ly = 0.0;
#pragma unroll
                for (int e = D - 1; e >= 0; --e)
                    if (lane % D + e < D) {
                        const int r = 3 * (lane + 1 + e);
                        lx += mass[lane + 1 + e] * (sh.f[r] - sh.vs[r]);
                        ly += mass[lane + 1 + e] * (sh.f[r + 1] - sh.vs[r + 1]);
                    }
                sh.lam[2 * lane] = lx;
                sh.lam[2 * lane + 1] = ly;
            }
        }
    } else {
        if (lane < NQ) sh.vs[lane] = sh.f[lane];
    }
    lds_sync();
    // ---- node residual G~ ---------------------------------------------------
    {
        double* Gk = a.G + (int64_t)k * NXT;
        for (int r = lane; r < NXT; r += 64) {
            double g;
            if (r < NQ) g = qp[r] - qm[r];
            else if (r < 2 * NQ) g = vp[r - NQ] - sh.vs[r - NQ];
            else g = sh.z[r] - sh.z[NXT + r];
            Gk[r] = g;
        }
        if (a.Psi && lane < NY && k + 1 < a.n)
            a.Psi[(int64_t)k * NY + lane] =
                (sh.ynext[lane] - sh.z[6 * NB + lane]) - (lane < NC ? a.delta : a.eps);
    }

    // ---- JGv: columns of dG~_v / d(q+, v-, Phi, masses) ---------------------
    double* Jk = a.JGv + (int64_t)k * NQ * NCV;
    double tv[TP::NTV];   // T, element lane & 15 of each vector
    if constexpr (NJ > 0)
#pragma unroll
        for (int q = 0; q < TP::NTV; ++q) tv[q] = heavy ? 0.0 : sh.leg.T[16 * q + (lane & 15)];
#pragma unroll 1
    for (int c0 = 0; c0 < NCV; c0 += 64) {
        // (spare lanes repeat the last column: T's broadcasts need every lane)
        const int cj = c0 + lane < NCV ? c0 + lane : NCV - 1;
        int b, kind, comp;   // kind 0: q+, 1: v-, 2: Phi, 3: mass
        if (cj < NQ) { kind = 0; b = cj / 3; comp = cj % 3; }
        else if (cj < 2 * NQ) { kind = 1; b = (cj - NQ) / 3; comp = (cj - NQ) % 3; }
        else if (cj < 2 * NQ + 2 * NC) { kind = 2; comp = cj - 2 * NQ; b = TP::cbody(comp >> 1); }
        else { kind = 3; b = cj - 2 * NQ - 2 * NC; comp = 0; }
        double du[3] = {0.0, 0.0, 0.0};
        if constexpr (NC > 0) {
            const int i = TP::contact_at(b);
            if (i >= 0 && (kind == 0 || kind == 2)) {
                const int d = kind == 0 ? comp : 3 + (comp & 1);
#pragma unroll
                for (int q = 0; q < 3; ++q) du[q] = sh.minv[3 * b + q] * sh.dw[i][d][q];
            }
        }
        if (kind == 1) du[comp] = 1.0;
        if (kind == 3) {
            const double rm = 1.0 / sh.prm[2 + b];
#pragma unroll
            for (int q = 0; q < 3; ++q) du[q] = -(sh.vs[3 * b + q] - vm[3 * b + q]) * rm;
        }
        const bool thdir = kind == 0 && comp == 2;
        if constexpr (NJ == 0) {
#pragma unroll
            for (int r = 0; r < NQ; ++r)
                Jk[(int64_t)r * NCV + cj] = (r / 3 == b) ? -du[r % 3] : 0.0;
        } else if (heavy) {
            // joints at b: d(grad h)^T Lambda (angle direction), grad h du + d(grad h) v*
            double dtq = 0.0;
            int js[TP::ADJ];
            double sg[TP::ADJ], ax[TP::ADJ], ay[TP::ADJ];
#pragma unroll
            for (int q = 0; q < TP::ADJ; ++q) {
                bool par;
                const int j = TP::slot_joint(b, q, par);
                js[q] = j < 0 ? 0 : j;
                sg[q] = j < 0 ? 0.0 : (par ? 1.0 : -1.0);
                ax[q] = par ? sh.arm[js[q]][0] : sh.arm[js[q]][2];
                ay[q] = par ? sh.arm[js[q]][1] : sh.arm[js[q]][3];
                if (thdir)   // d(E a)/dth = -a: parent side -a_p, child side +a_c
                    dtq -= sg[q] * (ax[q] * sh.lam[2 * js[q]] + ay[q] * sh.lam[2 * js[q] + 1]);
            }
            du[2] += sh.minv[3 * b + 2] * dtq;
            const double om = thdir ? sh.vs[3 * b + 2] : 0.0;
            double bx[TP::ADJ], by[TP::ADJ];
#pragma unroll
            for (int q = 0; q < TP::ADJ; ++q) {
                bx[q] = sg[q] * ((du[0] - du[2] * ay[q]) - ax[q] * om);
                by[q] = sg[q] * ((du[1] + du[2] * ax[q]) - ay[q] * om);
            }
#pragma unroll 2
            for (int rb = 0; rb < NB; ++rb)
#pragma unroll
                for (int q3 = 0; q3 < 3; ++q3) {
                    const int r = 3 * rb + q3;
                    double acc = rb == b ? -du[q3] : 0.0;
#pragma unroll
                    for (int q = 0; q < TP::ADJ; ++q)
                        acc = fma(sh.X[2 * js[q]][r], bx[q],
                                  fma(sh.X[2 * js[q] + 1][r], by[q], acc));
                    Jk[(int64_t)r * NCV + cj] = acc;
                }
        } else {
            constexpr int D = TP::D, L = TP::L;
            // joints at b: d(grad h)^T Lambda (angle direction)
            double dtq = 0.0;
#pragma unroll
            for (int s = 0; s < TP::ADJ; ++s) {
                bool par;
                const int j = TP::slot_joint(b, s, par);
                if (j >= 0 && thdir) {
                    // d(E a)/dth = -a: parent side -a_p, child side +a_c
                    const double ax = par ? -sh.arm[j][0] : sh.arm[j][2];
                    const double ay = par ? -sh.arm[j][1] : sh.arm[j][3];
                    dtq += ax * sh.lam[2 * j] + ay * sh.lam[2 * j + 1];
                }
            }
            const double m = sh.prm[2 + b], I = m * mc.ipm[b];
            const double Fx = m * du[0], Fy = m * du[1], Tq = I * du[2] + dtq;
            // turning a link by dth moves the links from it on by -w dth r, a torso
            // the first joints by -w dth a_p
            const double w = thdir ? sh.vs[3 * b + 2] : 0.0;
            const bool link = b > 0;
            const int leg = link ? (b - 1) / D : 0, lk = link ? (b - 1) % D : 0, j0 = leg * D;
            const int jb = j0 + lk;
            const double lx = link ? Fx : 0.0, ly = link ? Fy : 0.0, lt = link ? Tq : 0.0;
            const double wl = link ? w : 0.0, w0 = link ? 0.0 : w;
            const double rbx = sh.leg.rho[jb][0], rby = sh.leg.rho[jb][1];
            const double gx = fma(wl, sh.leg.sig[jb][0], lx), gy = fma(wl, sh.leg.sig[jb][1], ly);
            const double acx = sh.arm[jb][2], acy = sh.arm[jb][3];
            const double a1x = sh.arm[j0][0], a1y = sh.arm[j0][1];
            double f[D], R[3], rx[D], ry[D], cx[D], cy[D];
#pragma unroll
            for (int i = 0; i < D; ++i) {
                rx[i] = sh.leg.rho[j0 + i][0];
                ry[i] = sh.leg.rho[j0 + i][1];
                cx[i] = sh.arm[j0 + i][2];
                cy[i] = sh.arm[j0 + i][3];
                const double ax = i < lk ? rx[i] : sh.leg.sig[j0 + i][0];
                const double ay = i < lk ? ry[i] : sh.leg.sig[j0 + i][1];
                const double bx = i < lk ? gx : wl * rbx, by = i < lk ? gy : wl * rby;
                f[i] = i == lk ? lt + (acy * lx - acx * ly) : ax * by - ay * bx;
            }
            R[0] = link ? gx : Fx + w0 * Z[0];
            R[1] = link ? gy : Fy + w0 * Z[1];
            R[2] = link ? a1x * gy - a1y * gx : Tq + w0 * Z[2];
            double y[D];
#pragma unroll
            for (int i = 0; i < D; ++i) {
                y[i] = 0.0;
#pragma unroll
                for (int l = 0; l < D; ++l) y[i] += sh.leg.Hi[leg][i][l] * f[l];
#pragma unroll
                for (int e = 0; e < 3; ++e) R[e] -= sh.leg.G[leg][i][e] * f[i];
            }
            double n0[3];   // -a0
#pragma unroll
            for (int e = 0; e < 3; ++e)
                n0[e] = -(si[e][0] * R[0] + si[e][1] * R[1] + si[e][2] * R[2]);
            // the leg's own response
            double own[3 * D], sx = 0.0, sy = 0.0;
#pragma unroll
            for (int i = 0; i < D; ++i) {
                const double mx = i == lk ? wl * acx : (i > lk ? -wl * rbx : 0.0);
                const double my = i == lk ? wl * acy : (i > lk ? -wl * rby : 0.0);
                own[3 * i] = mx + (sx + cy[i] * y[i]);
                own[3 * i + 1] = my + (sy - cx[i] * y[i]);
                own[3 * i + 2] = y[i];
                sx -= ry[i] * y[i];
                sy += rx[i] * y[i];
            }
#pragma unroll
            for (int r = 0; r < 3; ++r) Jk[(int64_t)r * NCV + cj] = n0[r];
            unrolled<L>([&](auto l_c) {
                constexpr int l = decltype(l_c)::value;
                const double on = link && leg == l ? -1.0 : 0.0;
                const double nx = fma(w0, sh.arm[l * D][0], n0[0]);
                const double ny = fma(w0, sh.arm[l * D][1], n0[1]);
                unrolled<3 * D>([&](auto q_c) {
                    constexpr int r = 3 + 3 * D * l + decltype(q_c)::value, t = 3 * r;
                    double acc = on * own[decltype(q_c)::value];
                    fma_row<t & 15>(acc, tv[t >> 4], nx);
                    fma_row<(t + 1) & 15>(acc, tv[(t + 1) >> 4], ny);
                    fma_row<(t + 2) & 15>(acc, tv[(t + 2) >> 4], n0[2]);
                    Jk[(int64_t)r * NCV + cj] = acc;
                });
            });
        }
    }

    // ---- Theta and JTc: one lane per (contact, variable) --------------------
    if constexpr (NC > 0) {
        if (lane < TP::NCT * NC) {
            const int i = lane / TP::NCT, c = lane - TP::NCT * i, b = TP::cbody(i);
            auto in = [&](double v, int idx) { return dn(v, c == idx ? 1.0 : 0.0); };
            const Dual x = in(qp[3 * b], 0), y = in(qp[3 * b + 1], 1), th = in(qp[3 * b + 2], 2);
            const Dual ux = in(vp[3 * b], 3), uy = in(vp[3 * b + 1], 4), uo = in(vp[3 * b + 2], 5);
            const Dual wx = in(vm[3 * b], 6), wy = in(vm[3 * b + 1], 7), wo = in(vm[3 * b + 2], 8);
            const Dual pt = in(phi[2 * i], 9), pn = in(phi[2 * i + 1], 10);
            const Dual g = in(gam[i], 11), mu = in(sh.prm[0], 12), e = in(sh.prm[1], 13);
            Dual s, co;
            dsincos(th, s, co);
            const double rx = mc.cr[i][0], ry = mc.cr[i][1];
            const Dual ax = rx * co - ry * s, ay = rx * s + ry * co;
            Dual sd, nx, ny, tx, ty;
            frame_d(mc, x + ax, y + ay, sd, nx, ny, tx, ty);
            // contact-point velocities J v+ and J v- (E a = (-a_y, a_x))
            const Dual px = ux - uo * ay, py = uy + uo * ax;
            const Dual mx = wx - wo * ay, my = wy + wo * ax;
            const Dual w = nx * (px + e * mx) + ny * (py + e * my);
            const Dual vt = tx * px + ty * py;
            const Dual lam = vt + g * pt / dsqrt(pt * pt + dn(1.0));
            const Dual rho = dsabs(mu * pn) - dsabs(pt);
            const double dl = a.delta;
            const Dual rows[10] = {dfb(pn, sd, dl), dfb(pn, w, dl), pn * lam - dn(dl),
                                   -(pn * lam) - dn(dl), dfb(g, rho, dl), -pn, -sd, -w, -g, -rho};
            double* Tk = a.JTc + ((int64_t)k * TP::NTH + 10 * i) * TP::NCT + c;
#pragma unroll
            for (int q = 0; q < 10; ++q) Tk[q * TP::NCT] = rows[q].d;
            if (c == 0) {
                double* th_out = a.Theta + (int64_t)k * TP::NTH + 10 * i;
#pragma unroll
                for (int q = 0; q < 10; ++q) th_out[q] = rows[q].v;
            }
        }
    }
}

template <int L, int D>
cis_status launch_impact(const cis_model* m, const ImpactArgs& args, hipStream_t stream) {
    using TP = ImpTopo<L, D>;
    const auto mc = make_const<TP::NB, TP::NJ, TP::NC>(m);
    hipLaunchKernelGGL(k_impact<TP>, dim3(args.n), dim3(64), 0, stream, args, mc);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? CIS_OK
                           : fail(CIS_ERR_HIP, "cis_impact_linearize: launch failed: %s",
                                  hipGetErrorString(e));
}

}  // namespace cis

using namespace cis;

extern "C" cis_status cis_impact_dims(const cis_model* model, int32_t* n_theta, int32_t* n_jgv_cols,
                                      int32_t* n_jtc_cols) {
    if (!model) return fail(CIS_ERR_NULL, "cis_impact_dims: model is required");
    if (n_theta) *n_theta = 10 * model->nc;
    if (n_jgv_cols) *n_jgv_cols = 6 * model->nb + 2 * model->nc + model->nb;
    if (n_jtc_cols) *n_jtc_cols = 14;
    return CIS_OK;
}

extern "C" cis_status cis_impact_linearize(const cis_model* model, int32_t n_nodes, int64_t ld_node,
                                           const double* Xp, const double* Xm, const double* Phi,
                                           const double* Gamma, const double* params, double delta,
                                           double eps, double* G, double* Theta, double* JGv,
                                           double* JTc, double* Psi, void* stream) {
    if (!model) return fail(CIS_ERR_NULL, "cis_impact_linearize: model is required");
    if (n_nodes < 0 || n_nodes > (1 << 30))
        return fail(CIS_ERR_DIM, "cis_impact_linearize: n_nodes=%d out of range", n_nodes);
    if (ld_node < n_nodes || ld_node < 1)
        return fail(CIS_ERR_DIM, "cis_impact_linearize: ld_node=%lld < max(n_nodes, 1)",
                    (long long)ld_node);
    if (!(delta > 0.0) || !std::isfinite(delta) || !std::isfinite(eps))
        return fail(CIS_ERR_DIM, "cis_impact_linearize: delta must be finite and > 0, eps finite");
    if (n_nodes == 0) return CIS_OK;
    const bool hc = model->nc > 0;
    if (!Xp || !Xm || !params || !G || !JGv || (hc && (!Phi || !Gamma || !Theta || !JTc)))
        return fail(CIS_ERR_NULL,
                    "cis_impact_linearize: Xp, Xm, params, G, JGv (and Phi, Gamma, Theta, JTc "
                    "when the model has contacts) are required");
    const void* ptrs[] = {Xp, Xm, Phi, Gamma, params, G, Theta, JGv, JTc, Psi};
    for (const void* p : ptrs)
        if (!aligned(p, 8))
            return fail(CIS_ERR_LAYOUT, "cis_impact_linearize: pointer not aligned to 8 bytes");
    ImpactArgs a;
    a.Xp = Xp;
    a.Xm = Xm;
    a.Phi = Phi;
    a.Gam = Gamma;
    a.prm = params;
    a.G = G;
    a.Theta = Theta;
    a.JGv = JGv;
    a.JTc = JTc;
    a.Psi = Psi;
    a.ld = ld_node;
    a.n = n_nodes;
    a.delta = delta;
    a.eps = eps;
    hipStream_t hs = (hipStream_t)stream;
#define CIS_DISPATCH_IMPACT(LL, DD) \
    if (model->L == LL && model->D == DD) return launch_impact<LL, DD>(model, a, hs);
    CIS_TOPOLOGIES(CIS_DISPATCH_IMPACT)
#undef CIS_DISPATCH_IMPACT
    return fail(CIS_ERR_UNSUPPORTED, "cis_impact_linearize: topology has no compiled kernel");
}
