// Gradient step of legs with links, four intervals per workgroup on rows of 16
// body lanes (cis_pack.hpp): the defects pass with its checkpoints, and the
// reverse sweep of the discrete RK4 map (same maps as cis.hip's defects and
// cis_adjoint.hip's sweep; the penalized defect merit of Sec. V is one use).
//
// Reverse sweep, one workgroup barrier per step, stages last first:
//   wave E : the four stage inputs of a substep from its start state, with their
//            rotations and accelerations (stage e at step e);
//   wave C : the Jacobian coefficients of the stages, last first, four steps on;
//   wave R : the transposed Jacobian product, a step behind C:
//            kbar_i = h/6 w_i xbar + h a_{i+1} Xbar_{i+1}, Xbar_i = s J^T kbar_i;
//   wave S : (checkpoints more than a substep apart) the substep starts of the
//            next checkpoint segment, a segment ahead of E.
// A lane's joint and contact are its own, so J^T needs only its parent's velocity
// adjoints and its children's joint terms, by DPP as in the forward sweep; no
// scatter through LDS.
//
// Bound by the serial chain of one step (E and R some 250 FP64 instructions each)
// with 6 waves per CU: at 206 to 224 registers eight waves fit a CU, and so two
// workgroups of three, which is also what their 71 to 78 KB of LDS leave room for.
// 12,800 flat quad13 intervals, K = 20: sweep 7.81 -> 0.57 ms, defects 0.93 -> 0.25 ms
// against one interval per workgroup on element lanes; 50 cheetah7 intervals,
// checkpoints 5 apart: 130 -> 82 us and 54 -> 47 us.
#include <hip/hip_runtime.h>

#include <cstring>

#include "../../include/cis.h"
#include "cis_host.hpp"
#include "cis_launch.hpp"
#include "cis_model.hpp"
#include "cis_pack.hpp"
#include "cis_reduced.hpp"

namespace cis {

// One RK4 stage's update of the nominal state of a body lane (the arithmetic of
// the record launch: increments apart, weights with s rounded once).
template <class T>
struct PackRK {
    T h, sK, s6;
    __device__ __forceinline__ PackRK(T s, T Kt)
        : h(T(1) / Kt), sK(s / Kt), s6(s / (T(6) * Kt)) {}
    template <int ST>
    __device__ __forceinline__ void step(T (&xb)[6], T (&xa)[6], T (&xs)[6],
                                         const T (&f)[3]) const {
        const T ux = ST == 0 || ST == 3 ? s6 : T(2) * s6, un = ST == 2 ? sK : T(0.5) * sK;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const T v = xs[3 + q];
            if constexpr (ST == 0) {
                xa[q] = ux * v;
                xa[3 + q] = ux * f[q];
            } else {
                xa[q] += ux * v;
                xa[3 + q] += ux * f[q];
            }
            if constexpr (ST < 3) {
                xs[q] = xb[q] + un * v;
                xs[3 + q] = xb[3 + q] + un * f[q];
            } else {
                xs[q] = xb[q] += xa[q];
                xs[3 + q] = xb[3 + q] += xa[3 + q];
            }
        }
    }
};

template <class TP>
__device__ __forceinline__ int pack_row(int b, int q) {   // state row q of body b
    return q < 3 ? 3 * b + q : TP::NQ + 3 * b + q - 3;
}

// ---------------------------------------------------------------------------
// Defects pass: wave 0 the nominal recursion with the checkpoints, wave 1 the
// integral rows a stage behind.
// ---------------------------------------------------------------------------
template <class T, class TP, bool FLAT>
__device__ __forceinline__ void defects_pack(const FwdArgs<T>& a,
                                             const MConst<TP::NB, TP::NJ, TP::NC>& mc, int k,
                                             bool on, int most, PackShared<T>& sh) {
    constexpr int NX = TP::NX, NC = TP::NC;
    const int me = threadIdx.x & 63;
    PackBody<T, TP, FLAT> c;
    c.lc = &sh.lc.v[0][me];
    c.load(a, mc, k, me & 15);   // both waves store the same constants
    const int nst = 4 * a.K;
    const T Kt = T(a.K);
    const PackRK<T> rk(c.s, Kt);
    auto put = [&](int r, T x) {
        if (a.xprop) a.xprop[r * a.ldi + k] = x;
        a.defect[r * a.ldi + k] = x - a.X[r * a.ldn + k + 1];
    };
    __syncthreads();
    if (threadIdx.x < 64) {
        T xb[6], xs[6], xa[6];
        const T zs[6] = {T(0), T(0), T(0), T(0), T(0), T(0)};
#pragma unroll
        for (int q = 0; q < 6; ++q) xs[q] = xb[q] = a.X[pack_row<TP>(c.b, q) * a.ldn + k];
        int togo = 0;   // substeps to the next checkpoint
        T* ck = a.ckpt ? a.ckpt + k : nullptr;
        auto stage = [&](auto st_c, int t) {
            constexpr int ST = decltype(st_c)::value;
            if (t < nst) {   // whole rows of 16 lanes
                if constexpr (ST == 0) {
                    if (ck && togo == 0) {
                        if (on && c.body)
#pragma unroll
                            for (int q = 0; q < 6; ++q) ck[pack_row<TP>(c.b, q) * a.ldi] = xb[q];
                        ck += (int64_t)NX * a.ldi;
                        togo = a.C;
                    }
                    --togo;
                }
                const T jt = T(t >> 2) + (ST == 0 ? T(0) : (ST == 3 ? T(1) : T(0.5)));
                T f[3], kz[3], cth, cb, sb;
                pack_state<T, TP, FLAT>(c, mc, xs, zs, quotient(jt, Kt, rk.h), f, kz, cth, cb, sb);
                sh.put(ST & 1, me, xs, cb, sb);
                rk.template step<ST>(xb, xa, xs, f);
            }
            __syncthreads();
        };
        for (int t = 0; t < 4 * most; t += 4) {
            stage(std::integral_constant<int, 0>{}, t);
            stage(std::integral_constant<int, 1>{}, t + 1);
            stage(std::integral_constant<int, 2>{}, t + 2);
            stage(std::integral_constant<int, 3>{}, t + 3);
        }
        if (on && c.body)
#pragma unroll
            for (int q = 0; q < 6; ++q) put(pack_row<TP>(c.b, q), xb[q]);
    } else {
        T ycc = c.contact ? a.X[(NX + c.i) * a.ldn + k] : T(0);
        T yct = c.torso && c.body ? a.X[(NX + NC) * a.ldn + k] : T(0);
        T yca = T(0), yta = T(0);
        PackSums<T, TP, FLAT> sm;
        for (int t = 0; t < 4 * most; ++t) {
            __syncthreads();   // the state wave has left stage t
            if (t >= nst) continue;
            const int st = t & 3;
            T cc, ct;
            pack_coef<T, TP, FLAT, false>(c, mc, sh, t & 1, StageHold<T>{}, cc, ct, sm,
                                          (T*)nullptr, false);
            const T w = st == 0 || st == 3 ? rk.s6 : T(2) * rk.s6;
            yca += w * cc;
            yta += w * ct;
            if (st == 3) {
                ycc += yca;
                yct += yta;
                yca = yta = T(0);
            }
        }
        yct = row_sum(yct);
        if (on) {
            if (c.contact) put(NX + c.i, ycc);
            if (c.torso && c.body) put(NX + NC, yct);
        }
    }
}

// Workgroup's four intervals of an item list, or none: item index of the lane,
// whether it repeats another's, and the largest substep count of the four.
struct PackRow {
    int item;
    bool on;
};
__device__ __forceinline__ PackRow pack_row_item(int n) {
    const int want = 4 * xcd_slot(blockIdx.x, gridDim.x) + (((int)threadIdx.x & 63) >> 4);
    return PackRow{want < n ? want : n - 1, want < n};
}
__device__ __forceinline__ int pack_most(int K) {
    int most = K;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int v = __builtin_amdgcn_readlane(K, 16 * q);
        most = v > most ? v : most;
    }
    return most;
}

// FP64: three waves per SIMD on flat ground (60 bytes of scratch; at two and none 253
// us instead of 250 for 12,800 quad13 intervals), two on the sinusoid (188 bytes at
// three; gradient step of biped5 batches of 300, 3,000 and 12,800 intervals: 195,
// 355 and 1,137 us at three, 171, 329 and 1,080 at two).
template <class T, class TP, bool FLAT>
__global__ void __launch_bounds__(128)
    __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? (FLAT ? 3 : 2) : 4)))
    k_defects_pack(ItemList<T> l, MConst<TP::NB, TP::NJ, TP::NC> mc) {
    __shared__ PackShared<T> sh;
    const PackRow r = pack_row_item(l.n);
    const FwdArgs<T> a = l.args(r.item);
    defects_pack<T, TP, FLAT>(a, mc, l.interval(r.item), r.on, pack_most(a.K), sh);
}

// ---------------------------------------------------------------------------
// Reverse sweep
// ---------------------------------------------------------------------------
// stage values of wave E, and coefficients of wave C, per lane
enum { H_X = 0, H_Y, H_VX, H_VY, H_OM, H_C, H_S, H_F0, H_F1, H_F2, H_CTH, H_N };
enum { G_CTH = 0, G_CVX, G_CVY, G_CVT, G_APX, G_APY, G_ACX, G_ACY, G_VX, G_VY, G_OM, G_F0, G_F1,
       G_F2, G_CC, G_CT, G_CY, G_CVXD, G_COM, G_CTHC, G_AX, G_AY, G_G0, G_G1, G_G2, G_JMU, G_NFLAT,
       // sinusoid: contact force along the surface, frame, remaining cc terms
       G_FXX = G_NFLAT, G_FYX, G_FTX, G_CX, G_CVYD, G_NX, G_NY, G_NALL };

template <bool FLAT, int NSEG>
struct AdjPack {
    using T = double;
    static constexpr int NG = FLAT ? (int)G_NFLAT : (int)G_NALL;
    PackConst<T> lc;
    T hist[5][H_N][64];               // E to C: five slots, see adj_slot
    T cf[2][NG][64];                  // C to R
    T start[NSEG + 1][6][64];         // S to E: substep starts of a segment
};

// Slot of element i (of n, plus a spare) of group g, where group g + 1 is written
// forward while group g is read backward at the same pace.
__device__ __forceinline__ int adj_slot(int g, int i, int n) { return (g & 1) ? n - i : i; }

// Wave C: coefficients of one stage (unweighted: the adjoint carries the weights).
template <class TP, bool FLAT, int NSEG>
__device__ __forceinline__ void adj_coef(const PackBody<double, TP, FLAT>& c,
                                         const MConst<TP::NB, TP::NJ, TP::NC>& mc,
                                         AdjPack<FLAT, NSEG>& sh, int slot, double tau,
                                         double (*out)[64]) {
    using T = double;
    using C = PackConst<T>;
    asm volatile("" ::: "memory");
    const int me = threadIdx.x & 63, up = (me & 48) + c.p;
    const T(*h)[64] = sh.hist[slot];
    const T xb = h[H_X][me], yb = h[H_Y][me], vx = h[H_VX][me], vy = h[H_VY][me], om = h[H_OM][me];
    const T cb = h[H_C][me], sb = h[H_S][me];
    const T cp = h[H_C][up], sp = h[H_S][up], xp = h[H_X][up], yp = h[H_Y][up];
    const auto cr = c.get(C::RX), jp = c.get(C::RP), jc = c.get(C::RC);
    const auto lb = c.get(C::LB), ls = c.get(C::LS);   // (lnb, ltpb), (ltmb, slack)
    const T ax = cb * cr.a - sb * cr.b, ay = sb * cr.a + cb * cr.b;
    const Frame<T> f = FLAT ? Frame<T>{yb + ay, T(0), T(1), T(1), T(0), T(0), T(1), T(0), T(0)}
                            : terrain<T>(mc, xb + ax, yb + ay);
    const T Pdx = vx - om * ay, Pdy = vy + om * ax;
    const T apx = cp * jp.a - sp * jp.b, apy = sp * jp.a + cp * jp.b;
    const T acx = cb * jc.a - sb * jc.b, acy = sb * jc.a + cb * jc.b;
    const T vt = FLAT ? Pdx + T(0) * Pdy : f.tx * Pdx + f.ty * Pdy;
    T v0, d0, v1, d1, av, dav, v3, d3;
    sabs_d(xp + apx - xb - acx, v0, d0);
    sabs_d(yp + apy - yb - acy, v1, d1);
    sabs_d(vt, av, dav);
    sabs_d(-f.sd, v3, d3);
    const T rp = vt > T(0) ? av : T(0), rm = vt < T(0) ? av : T(0);
    const bool pen = c.contact && -f.sd > T(0);
    const T s = c.s;
    const T gv = lb.b * (vt > T(0) ? dav : T(0)) + ls.a * (vt < T(0) ? dav : T(0)) + ls.b * dav;
    if (!c.joint) d0 = d1 = T(0);
    const T Dg = pen ? -d3 : T(0);
    T zpx = T(0), zpy = Dg;
    T cx = T(0), cy = s * lb.a, cvx = s * gv, cvy = T(0);
    T com = -(s * gv) * ay, cth = -(s * gv) * om * ax;
    auto put = [&](int q, T v) { out[q][me] = v; };
    if constexpr (!FLAT) {
        zpx = c.contact ? Dg * f.dsd_px : T(0);
        zpy = c.contact ? Dg * f.dsd_py : T(0);
        const T omt = T(1) - tau;
        const auto l0 = c.get(C::LN), l1 = c.get(C::FT);
        const T ln = omt * l0.a + tau * l0.b, ft = omt * l1.a + tau * l1.b;
        const T dfx = f.dny * ft + f.dnx * ln, dfy = -f.dnx * ft + f.dny * ln;
        cx = s * (lb.a * f.dsd_px + gv * (f.dny * Pdx - f.dnx * Pdy));
        // (by itself in the y row: no 0 x NaN of the frame's x without a contact)
        cy = c.contact ? s * (lb.a * f.dsd_py) : T(0);
        cvx = s * (gv * f.tx);
        cvy = s * (gv * f.ty);
        com = s * (gv * (f.ty * ax - f.tx * ay));
        cth = s * (-gv * om * (f.tx * ax + f.ty * ay));
        put(G_FXX, dfx * (s * c.mi));
        put(G_FYX, dfy * (s * c.mi));
        put(G_FTX, (ax * dfy - ay * dfx) * (s * c.ii));
        put(G_CX, cx);
        put(G_CVYD, cvy);
        put(G_NX, f.nx);
        put(G_NY, f.ny);
    }
    put(G_CVX, s * (c.children(d0) - d0 + zpx));
    put(G_CVY, s * (c.children(d1) - d1 + zpy));
    put(G_CVT, s * (c.children(d1 * apx - d0 * apy) + (d0 * acy - d1 * acx) +
                    (zpy * ax - zpx * ay)));
    put(G_CY, cy);
    put(G_CVXD, cvx);
    put(G_COM, com);
    put(G_CTHC, cth + (cy * ax - cx * ay));
    put(G_APX, apx);
    put(G_APY, apy);
    put(G_ACX, acx);
    put(G_ACY, acy);
    put(G_AX, ax);
    put(G_AY, ay);
    put(G_CC, lb.a * f.sd + lb.b * rp + ls.a * rm + ls.b * av);
    put(G_CT, (c.joint ? v0 + v1 : T(0)) + (pen ? v3 : T(0)));
    put(G_G0, (T(0.5) * s) * (f.sd + c.mu * av));
    put(G_G1, (T(0.5) * s) * (rp - av));
    put(G_G2, (T(0.5) * s) * (rm - av));
    put(G_JMU, s * (lb.a * av));
    put(G_VX, vx);
    put(G_VY, vy);
    put(G_OM, om);
    put(G_F0, h[H_F0][me]);
    put(G_F1, h[H_F1][me]);
    put(G_F2, h[H_F2][me]);
    put(G_CTH, h[H_CTH][me]);
}

template <class TP, bool FLAT, int NSEG>
__device__ __forceinline__ void adjoint_pack(const AdjArgs<double>& aa,
                                             const MConst<TP::NB, TP::NJ, TP::NC>& mc, int k,
                                             bool on, int most, AdjPack<FLAT, NSEG>& sh) {
    using T = double;
    using C = PackConst<T>;
    constexpr int NX = TP::NX, NC = TP::NC, NJ = TP::NJ;
    const FwdArgs<T>& a = aa.f;
    const int me = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    PackBody<T, TP, FLAT> c;
    c.lc = &sh.lc.v[0][me];
    c.load(a, mc, k, me & 15);   // every wave stores the same constants
    const int K = a.K, nst = 4 * K;
    const int Cs = NSEG ? __builtin_amdgcn_readfirstlane(a.C) : 1;
    const int d0 = NSEG ? 4 * Cs : 0;             // steps before E starts
    const int nsteps = d0 + 4 * most + 5;
    const T Kt = T(K);
    const PackRK<T> rk(c.s, Kt);
    const T zs[6] = {T(0), T(0), T(0), T(0), T(0), T(0)};
    auto tau_of = [&](int j, int st) {
        return quotient(T(j) + (st == 0 ? T(0) : (st == 3 ? T(1) : T(0.5))), Kt, rk.h);
    };
    // state at a checkpoint of the lane's body
    auto load_state = [&](int slot, T (&x)[6]) {
        const T* ck = a.ckpt + (int64_t)slot * NX * a.ldi + k;
#pragma unroll
        for (int q = 0; q < 6; ++q) x[q] = ck[pack_row<TP>(c.b, q) * a.ldi];
    };
    __syncthreads();
    if (wave == 0) {
        // ---- E: stage e - 4 J of the J-th substep from the end ----
        T xb[6], xs[6], xa[6], nx[6];
        if constexpr (!NSEG) load_state(K - 1, nx);
        auto stage = [&](auto st_c, int e) {
            constexpr int ST = decltype(st_c)::value;
            if (e >= 0 && e < nst) {
                const int J = e >> 2, j = K - 1 - J;
                if constexpr (ST == 0) {
                    if constexpr (NSEG) {
                        const int u = J / Cs, i = Cs - 1 - (J - u * Cs);
#pragma unroll
                        for (int q = 0; q < 6; ++q) xb[q] = sh.start[adj_slot(u, i, Cs)][q][me];
                    } else {
                        // (the next substep's start is on its way meanwhile)
#pragma unroll
                        for (int q = 0; q < 6; ++q) xb[q] = nx[q];
                        load_state(j > 0 ? j - 1 : 0, nx);
                    }
#pragma unroll
                    for (int q = 0; q < 6; ++q) xs[q] = xb[q];
                }
                T f[3], kz[3], cth, cb, sb;
                pack_state<T, TP, FLAT>(c, mc, xs, zs, tau_of(j, ST), f, kz, cth, cb, sb);
                T(*h)[64] = sh.hist[adj_slot(J, ST, 4)];
                h[H_X][me] = xs[0];
                h[H_Y][me] = xs[1];
                h[H_VX][me] = xs[3];
                h[H_VY][me] = xs[4];
                h[H_OM][me] = xs[5];
                h[H_C][me] = cb;
                h[H_S][me] = sb;
                h[H_F0][me] = f[0];
                h[H_F1][me] = f[1];
                h[H_F2][me] = f[2];
                h[H_CTH][me] = cth;
                if constexpr (ST < 3) rk.template step<ST>(xb, xa, xs, f);
            }
            __syncthreads();
        };
        for (int p = 0; p < d0; ++p) __syncthreads();
        for (int e = 0; e < 4 * most; e += 4) {
            stage(std::integral_constant<int, 0>{}, e);
            stage(std::integral_constant<int, 1>{}, e + 1);
            stage(std::integral_constant<int, 2>{}, e + 2);
            stage(std::integral_constant<int, 3>{}, e + 3);
        }
        for (int p = 0; p < 5; ++p) __syncthreads();
    } else if (wave == 1) {
        // ---- C: stage r from the end at step d0 + 4 + r ----
        for (int p = 0; p < nsteps; ++p) {
            const int r = p - d0 - 4;
            if (r >= 0 && r < nst) {
                const int J = r >> 2, st = 3 - (r & 3);
                adj_coef<TP, FLAT, NSEG>(c, mc, sh, adj_slot(J, st, 4), tau_of(K - 1 - J, st),
                                         sh.cf[r & 1]);
            }
            __syncthreads();
        }
    } else if (wave == 2) {
        // ---- R: stage r from the end at step d0 + 5 + r ----
        T xb[6], xp[6], xsum[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            xb[q] = aa.seed[pack_row<TP>(c.b, q) * a.ldi + k];
            xp[q] = xsum[q] = T(0);
        }
        const T scc = c.contact ? aa.seed[(NX + c.i) * a.ldi + k] : T(0);
        const T sct = aa.seed[(NX + NC) * a.ldi + k];
        const T h6 = T(1) / (T(6) * Kt);
        const T si = c.s * c.ii, sm = c.s * c.mi;
        const auto kd = c.get(C::KD);
        T sacc = T(0), muacc = T(0), macc = T(0), ju[3][2], cu[3][2];
#pragma unroll
        for (int q = 0; q < 3; ++q) ju[q][0] = ju[q][1] = cu[q][0] = cu[q][1] = T(0);
        auto stage = [&](auto rr_c, int r) {
            constexpr int ST = 3 - decltype(rr_c)::value;   // RK stage
            if (r >= 0 && r < nst) {
                const T(*g)[64] = sh.cf[ST & 1 ? 0 : 1];    // r & 1
                auto at = [&](int q) { return g[q][me]; };
                const T tau = tau_of(K - 1 - (r >> 2), ST), omt = T(1) - tau;
                const T w = ST == 0 || ST == 3 ? h6 : T(2) * h6;
                const T an = ST == 2 ? rk.h : T(0.5) * rk.h;
                T kb[6];
#pragma unroll
                for (int q = 0; q < 6; ++q) kb[q] = w * xb[q] + (ST < 3 ? an * xp[q] : T(0));
                const T kcc = w * scc, lc = w * sct;
                const T wi = si * kb[5], mx = sm * kb[3], my = sm * kb[4];
                const T wip = c.parent(wi), mxp = c.parent(mx), myp = c.parent(my);
                const T de = wip - wi;                      // zero without a joint
                const T t1 = kd.a * de, t2 = kd.b * de;
                T X[6];
                X[0] = at(G_CVX) * lc;
                X[1] = at(G_CVY) * lc;
                X[2] = at(G_CTH) * kb[5] + at(G_CVT) * lc + (t1 - c.children(t1));
                X[3] = c.s * kb[0];
                X[4] = c.s * kb[1];
                X[5] = c.s * kb[2] + (t2 - c.children(t2));
                // contact (kcc = 0 and no force without one)
                const T ax = at(G_AX), ay = at(G_AY);
                X[1] += at(G_CY) * kcc;
                X[2] += at(G_CTHC) * kcc;
                X[3] += at(G_CVXD) * kcc;
                X[5] += at(G_COM) * kcc;
                T in, it;   // unit normal and tangent force on (mx, my, wi)
                if constexpr (FLAT) {
                    in = my + ax * wi;
                    it = mx - ay * wi;
                } else {
                    const T nx = at(G_NX), ny = at(G_NY);
                    const T q = at(G_FXX) * kb[3] + at(G_FYX) * kb[4], qt = at(G_FTX) * kb[5];
                    if (c.contact) {
                        X[0] += q + qt + at(G_CX) * kcc;
                        X[2] -= ay * q;                      // (G_CTH holds its torque part)
                        X[4] += at(G_CVYD) * kcc;
                    }
                    in = nx * mx + ny * my + (ax * ny - ay * nx) * wi;
                    it = ny * mx - nx * my - (ax * nx + ay * ny) * wi;
                }
                // controls
                const T fx = (mxp - mx) - at(G_APY) * wip + at(G_ACY) * wi;
                const T fy = (myp - my) + at(G_APX) * wip - at(G_ACX) * wi;
                ju[0][0] -= omt * de;
                ju[0][1] -= tau * de;
                ju[1][0] += omt * fx;
                ju[1][1] += tau * fx;
                ju[2][0] += omt * fy;
                ju[2][1] += tau * fy;
                const T b0 = at(G_G0) * kcc, b1 = at(G_G1) * kcc, b2 = at(G_G2) * kcc;
                cu[0][0] += omt * in + b0;
                cu[0][1] += tau * in + b0;
                cu[1][0] += omt * it + b1;
                cu[1][1] += tau * it + b1;
                cu[2][0] += b2 - omt * it;
                cu[2][1] += b2 - tau * it;
                // dilation, masses, friction coefficient
                const T f0 = at(G_F0), f1 = at(G_F1), f2 = at(G_F2);
                sacc += at(G_VX) * kb[0] + at(G_VY) * kb[1] + at(G_OM) * kb[2] + f0 * kb[3] +
                        f1 * kb[4] + f2 * kb[5] + at(G_CC) * kcc + at(G_CT) * lc;
                macc -= sm * (f0 * kb[3] + (f1 + T(mc.g)) * kb[4] + f2 * kb[5]);
                muacc += at(G_JMU) * kcc;
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    xp[q] = X[q];
                    xsum[q] += X[q];
                    if constexpr (ST == 0) {
                        xb[q] += xsum[q];
                        xsum[q] = T(0);
                    }
                }
            }
            __syncthreads();
        };
        for (int p = 0; p < d0 + 5; ++p) __syncthreads();
        for (int r = 0; r < 4 * most; r += 4) {
            stage(std::integral_constant<int, 0>{}, r);
            stage(std::integral_constant<int, 1>{}, r + 1);
            stage(std::integral_constant<int, 2>{}, r + 2);
            stage(std::integral_constant<int, 3>{}, r + 3);
        }
        sacc = row_sum(c.body ? sacc : T(0));
        muacc = row_sum(c.contact ? muacc : T(0));
        if (on && c.body) {
            const int64_t N = a.N;
#pragma unroll
            for (int q = 0; q < 6; ++q) aa.gX[pack_row<TP>(c.b, q) * a.ldn + k] = xb[q];
            if (c.contact) aa.gX[(NX + c.i) * a.ldn + k] = scc;
            if (c.torso) {
                aa.gX[(NX + NC) * a.ldn + k] = sct;
                aa.gs[k] = sacc;
                aa.ws_p[k] = muacc;
                aa.ws_p[N + k] = T(0);   // restitution: no dependence on this path
            }
            aa.ws_p[(2 + c.b) * N + k] = macc;
            auto control = [&](int u, const T (&v)[2]) {
                aa.ws_uk[u * N + k] = v[0];
                aa.ws_uk1[u * N + k] = v[1];
            };
            if (c.joint) {
                control(c.j, ju[0]);
                control(NJ + 2 * c.j, ju[1]);
                control(NJ + 2 * c.j + 1, ju[2]);
            }
            if (c.contact)
#pragma unroll
                for (int q = 0; q < 3; ++q) control(3 * NJ + 3 * c.i + q, cu[q]);
        }
    } else if constexpr (NSEG) {
        // ---- S: substep starts of segment u (from the end), forward, at steps
        // 4 Cs u .. ----
        T xb[6], xs[6], xa[6];
        for (int p = 0; p < nsteps; p += 4) {
            const int t = p >> 2, u = t / Cs, i = t - u * Cs;
            const bool live = (u + 1) * Cs <= K;
            const int g = live ? K / Cs - 1 - u : 0;
            if (live) {
                if (i == 0) load_state(g, xb);
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    sh.start[adj_slot(u, i, Cs)][q][me] = xb[q];
                    xs[q] = xb[q];
                }
            }
            const bool run = live && i < Cs - 1;   // the last start ends the segment
            auto stage = [&](auto st_c) {
                constexpr int ST = decltype(st_c)::value;
                if (run) {
                    T f[3], kz[3], cth, cb, sb;
                    pack_state<T, TP, FLAT>(c, mc, xs, zs, tau_of(g * Cs + i, ST), f, kz, cth, cb,
                                            sb);
                    rk.template step<ST>(xb, xa, xs, f);
                }
                if (p + ST < nsteps) __syncthreads();
            };
            stage(std::integral_constant<int, 0>{});
            stage(std::integral_constant<int, 1>{});
            stage(std::integral_constant<int, 2>{});
            stage(std::integral_constant<int, 3>{});
        }
    }
}

struct AdjList {
    const AdjArgs<double>* descs;   // NULL: one trajectory, `one`
    const int2* items;
    int n;
    AdjArgs<double> one;
};

template <class TP, bool FLAT, int NSEG>
__global__ void __launch_bounds__(NSEG ? 256 : 192) __attribute__((amdgpu_waves_per_eu(2)))
    k_adjoint_pack(AdjList l, MConst<TP::NB, TP::NJ, TP::NC> mc) {
    __shared__ AdjPack<FLAT, NSEG> sh;
    const PackRow r = pack_row_item(l.n);
    AdjArgs<double> a = l.one;
    if (l.descs) a = l.descs[l.items[r.item].x];
    adjoint_pack<TP, FLAT, NSEG>(a, mc, l.descs ? l.items[r.item].y : r.item, r.on,
                                 pack_most(a.f.K), sh);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
constexpr int SEG_MAX = 16;   // largest checkpoint spacing whose starts fit the LDS

bool gradient_pack_supported(const cis_model* m) { return m->L >= 1 && m->D >= 1; }
int gradient_pack_max_ckpt() { return SEG_MAX; }

template <class T, class TP, bool FLAT>
static void defects_launch(const cis_model* m, const ItemList<T>& l, KLaunch* out) {
    out->arg(l);
    out->arg(make_const<TP::NB, TP::NJ, TP::NC>(m));
    out->func = (const void*)&k_defects_pack<T, TP, FLAT>;
    out->grid = dim3((l.n + 3) / 4);
    out->block = dim3(128);
}

template <class T, int L, int D>
static cis_status defects_pack_t(const cis_model* m, const FwdArgs<T>* one, const BatchGroupDev* g,
                                 KLaunch* out) {
    if constexpr (L >= 1 && D >= 1) {
        ItemList<T> l;
        std::memset(&l, 0, sizeof(l));
        if (one) {
            l.one = *one;
            l.n = one->N;
        } else {
            l.descs = (const FwdArgs<T>*)g->fdesc;
            l.items = g->items;
            l.n = g->n_items;
        }
        if (m->A == 0.0) defects_launch<T, Topo<L, D>, true>(m, l, out);
        else defects_launch<T, Topo<L, D>, false>(m, l, out);
        return out->ok() ? CIS_OK : fail(CIS_ERR_DIM, "k_defects_pack: launch record refused");
    } else {
        return fail(CIS_ERR_UNSUPPORTED, "the packed gradient step needs legs with links");
    }
}

cis_status prep_defects_pack(const cis_model* m, int32_t dtype, const void* one,
                             const BatchGroupDev* g, KLaunch* out) {
#define CIS_DEF_PACK(LL, DD)                                                               \
    if (m->L == LL && m->D == DD)                                                          \
        return dtype == CIS_F64                                                            \
                   ? defects_pack_t<double, LL, DD>(m, (const FwdArgs<double>*)one, g, out) \
                   : defects_pack_t<float, LL, DD>(m, (const FwdArgs<float>*)one, g, out);
    CIS_TOPOLOGIES(CIS_DEF_PACK)
#undef CIS_DEF_PACK
    return fail(CIS_ERR_UNSUPPORTED, "k_defects_pack: topology has no compiled kernel");
}

template <class TP, bool FLAT>
static void adjoint_launch(const cis_model* m, const AdjList& l, int C, KLaunch* out) {
    out->arg(l);
    out->arg(make_const<TP::NB, TP::NJ, TP::NC>(m));
    out->func = C == 1   ? (const void*)&k_adjoint_pack<TP, FLAT, 0>
                : C <= 8 ? (const void*)&k_adjoint_pack<TP, FLAT, 8>
                         : (const void*)&k_adjoint_pack<TP, FLAT, SEG_MAX>;
    out->grid = dim3((l.n + 3) / 4);
    out->block = dim3(C == 1 ? 192 : 256);
}

template <int L, int D>
static cis_status adjoint_pack_t(const cis_model* m, const AdjArgs<double>* one,
                                 const BatchGroupDev* g, int C, KLaunch* out) {
    if constexpr (L >= 1 && D >= 1) {
        AdjList l;
        std::memset(&l, 0, sizeof(l));
        if (one) {
            l.one = *one;
            l.n = one->f.N;
        } else {
            l.descs = (const AdjArgs<double>*)g->adesc;
            l.items = g->items;
            l.n = g->n_items;
        }
        if (m->A == 0.0) adjoint_launch<Topo<L, D>, true>(m, l, C, out);
        else adjoint_launch<Topo<L, D>, false>(m, l, C, out);
        return out->ok() ? CIS_OK : fail(CIS_ERR_DIM, "k_adjoint_pack: launch record refused");
    } else {
        return fail(CIS_ERR_UNSUPPORTED, "the packed gradient step needs legs with links");
    }
}

cis_status prep_adjoint_pack(const cis_model* m, const void* one, const BatchGroupDev* g, int C,
                             KLaunch* out) {
    if (C < 1 || C > SEG_MAX)
        return fail(CIS_ERR_DIM, "k_adjoint_pack: checkpoint spacing %d beyond %d", C, SEG_MAX);
#define CIS_ADJ_PACK(LL, DD)      \
    if (m->L == LL && m->D == DD) \
        return adjoint_pack_t<LL, DD>(m, (const AdjArgs<double>*)one, g, C, out);
    CIS_TOPOLOGIES(CIS_ADJ_PACK)
#undef CIS_ADJ_PACK
    return fail(CIS_ERR_UNSUPPORTED, "k_adjoint_pack: topology has no compiled kernel");
}

}  // namespace cis
