// Runge-Kutta-Fehlberg form of the discretize step (arxiv 2604.09993, Sec. VI:
// the transcription integrates every interval with a Runge-Kutta-Fehlberg
// method and a fixed number of steps, and differentiates it internally).
//
// The integrator is Fehlberg's 4(5) pair: six stages per step; the fourth-order
// solution is propagated (its weight on the sixth stage is zero, so the
// sensitivities need only the first five stages), and the fifth-order one
// gives the embedded error estimate
//     e_j = h sum_i (bh_i - b_i) K_i,
// reported per interval as the largest |e_j| over its steps and all augmented
// rows.  The stage times tau = (j + c_i) / K feed the FOH controls.
//
// Two kernels in the split layout (cis_pack.hpp, cis_reduced.hpp):
//   k_rkf_rec : four intervals per workgroup of two waves, the nominal steps with
//               the S column (and the sixth stage for the estimate) and the
//               coefficients of the five propagated stages;
//   k_rkf_tan : the coupled columns of [Phi_x | B- | B+], one per lane, with the
//               stage derivatives of a step kept (the tableau is not diagonal,
//               unlike classical RK4), and the late closed-form entries.
#include <hip/hip_runtime.h>

#include <cstring>
#include <utility>

#include "../../include/cis.h"
#include "cis_body.hpp"
#include "cis_debug.hpp"
#include "cis_host.hpp"
#include "cis_launch.hpp"
#include "cis_model.hpp"
#include "cis_pack.hpp"
#include "cis_reduced.hpp"

namespace cis {

// Fehlberg (1969) 4(5) tableau: nodes c, coefficients a, fourth-order weights
// b, and e = (fifth-order weights) - b.
struct Fehlberg45 {
    static constexpr int S = 6;   // stages
    static constexpr int R = 5;   // stages of the propagated solution
    __host__ __device__ static constexpr double c(int i) {
        constexpr double v[6] = {0.0, 1.0 / 4.0, 3.0 / 8.0, 12.0 / 13.0, 1.0, 1.0 / 2.0};
        return v[i];
    }
    __host__ __device__ static constexpr double a(int i, int l) {
        constexpr double v[6][5] = {
            {0, 0, 0, 0, 0},
            {1.0 / 4.0, 0, 0, 0, 0},
            {3.0 / 32.0, 9.0 / 32.0, 0, 0, 0},
            {1932.0 / 2197.0, -7200.0 / 2197.0, 7296.0 / 2197.0, 0, 0},
            {439.0 / 216.0, -8.0, 3680.0 / 513.0, -845.0 / 4104.0, 0},
            {-8.0 / 27.0, 2.0, -3544.0 / 2565.0, 1859.0 / 4104.0, -11.0 / 40.0}};
        return v[i][l];
    }
    __host__ __device__ static constexpr double b(int i) {
        constexpr double v[6] = {25.0 / 216.0, 0.0, 1408.0 / 2565.0, 2197.0 / 4104.0, -1.0 / 5.0,
                                 0.0};
        return v[i];
    }
    __host__ __device__ static constexpr double bh(int i) {
        constexpr double v[6] = {16.0 / 135.0, 0.0, 6656.0 / 12825.0, 28561.0 / 56430.0,
                                 -9.0 / 50.0, 2.0 / 55.0};
        return v[i];
    }
    __host__ __device__ static constexpr double e(int i) { return bh(i) - b(i); }
    // products of the tableau: (A c)_i and (A A c)_i, the responses of a stage to a
    // force growing with time; (A A)_il and (b A)_l, those of a position to the
    // velocity derivatives of earlier stages
    __host__ __device__ static constexpr double ac(int i) {
        double v = 0;
        for (int l = 0; l < i; ++l) v += a(i, l) * c(l);
        return v;
    }
    __host__ __device__ static constexpr double aac(int i) {
        double v = 0;
        for (int l = 0; l < i; ++l) v += a(i, l) * ac(l);
        return v;
    }
    __host__ __device__ static constexpr double aa(int i, int l) {
        double v = 0;
        for (int m = l + 1; m < i; ++m) v += a(i, m) * a(m, l);
        return v;
    }
    __host__ __device__ static constexpr double ba(int l) {
        double v = 0;
        for (int m = l + 1; m < R; ++m) v += b(m) * a(m, l);
        return v;
    }
};
using RKF = Fehlberg45;

// What the coefficient wave needs of stage i: c, b, e, A c, A A c.  Its loop runs
// stage by stage (unrolled over the five, the compiler moves work across them and
// holds over 500 registers).
struct RkfStage {
    double c, b, e, ac, aac;
};
constexpr RkfStage rkf_stage(int i) {
    return {RKF::c(i), RKF::b(i), RKF::e(i), RKF::ac(i), RKF::aac(i)};
}
__constant__ const RkfStage RKF_STAGES[6] = {rkf_stage(0), rkf_stage(1), rkf_stage(2),
                                             rkf_stage(3), rkf_stage(4), rkf_stage(5)};

// A tableau coefficient formed where it is used (FP64: in scalar registers; kept
// in vector registers across the step, 25 of them spill others).
#define CIS_TAB(V) tableau<T, __builtin_bit_cast(uint64_t, (double)(V))>()
template <class T, uint64_t BITS>
__device__ __forceinline__ T tableau() {
    if constexpr (sizeof(T) == 8) return scalar_const<BITS>();
    else return (T)__builtin_bit_cast(double, BITS);
}

// out = base + h sum_{l <= I} a(I + 1, l) kd[l] (zero coefficients skipped)
template <int I, class T, int NR>
__device__ __forceinline__ void next_input(const T (&kd)[RKF::R][NR], const T (&base)[NR], T h,
                                           T (&out)[NR]) {
    T acc[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) acc[q] = T(0);
    unrolled<I + 1>([&](auto l_c) {
        constexpr int l = decltype(l_c)::value;
        if constexpr (RKF::a(I + 1, l) != 0.0) {
            const T w = CIS_TAB(RKF::a(I + 1, l));
#pragma unroll
            for (int q = 0; q < NR; ++q) acc[q] += w * kd[l][q];
        }
    });
#pragma unroll
    for (int q = 0; q < NR; ++q) out[q] = base[q] + h * acc[q];
}

// ---------------------------------------------------------------------------
// k_rkf_rec: four intervals by two waves, one workgroup barrier per record stage
// (five per step), the roles of cis_split.hip's record launch: wave 0 the nominal
// steps and S (at the fifth stage also the sixth, and the step's end), wave 1 the
// coefficients, sums and integral rows a stage behind, with their estimate.
// ---------------------------------------------------------------------------
template <class T, class TP, bool FLAT>
__device__ __forceinline__ void rkf_rec_item(const FwdArgs<T>& a,
                                             const MConst<TP::NB, TP::NJ, TP::NC>& mc, int k,
                                             T* __restrict__ rec, T* __restrict__ sums, int64_t n,
                                             T* __restrict__ err, bool on, PackShared<T, 3>& sh) {
    constexpr int NQ = TP::NQ, NX = TP::NX, NC = TP::NC, NR = RKF::R;
    using R = PackRec<TP, FLAT>;
    const int me = threadIdx.x & 63;
    PackBody<T, TP, FLAT> c;
    c.lc = &sh.lc.v[0][me];
    c.template load<true>(a, mc, k, me & 15);   // both waves store the same constants
    const T s = c.s, Kt = T(a.K), h = T(1) / Kt, sK = s / Kt;
    T* sr = rec + R::HDR;
    __syncthreads();
    if (threadIdx.x < 64) {
        if (on) pack_header(c, h, rec);
        T xb[6], xs[6], kd[NR][6], zb[6], zs[6], zd[NR][6], emax = T(0);
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            xb[q] = a.X[(q < 3 ? 3 * c.b + q : NQ + 3 * c.b + q - 3) * a.ldn + k];
            xs[q] = xb[q];
            zb[q] = zs[q] = T(0);
        }
        for (int j = 0; j < a.K; ++j) {
            const T jt = T(j);
            unrolled<NR>([&](auto i_c) {
                constexpr int I = decltype(i_c)::value;
                const int slot = (NR * j + I) & 1;
                T f[3], kz[3], cth, cb, sb;
                pack_accel<T, TP, FLAT>(c, mc, xs, zs, quotient(jt + CIS_TAB(RKF::c(I)), Kt, h), f, kz,
                                        cth, cb, sb);
                sh.put(slot, me, xs, cb, sb);
#pragma unroll
                for (int q = 0; q < 6; ++q) sh.z[slot][q][me] = zs[q];
                if (on && c.body) sr[R::CTH + c.b] = cth;
                sr += R::STAGE;
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    kd[I][q] = s * xs[3 + q];
                    kd[I][3 + q] = s * f[q];
                    zd[I][q] = s * zs[3 + q] + xs[3 + q];
                    zd[I][3 + q] = kz[q];
                }
                if constexpr (I < NR - 1) {
                    next_input<I>(kd, xb, h, xs);
                    next_input<I>(zd, zb, h, zs);
                } else {
                    // sixth stage (estimate only), then the step's end
                    T x6[6], f6[3], kz6[3], cth6, c6, s6;
                    next_input<I>(kd, xb, h, x6);
                    pack_accel<T, TP, FLAT>(c, mc, x6, zs, quotient(jt + CIS_TAB(RKF::c(5)), Kt, h), f6,
                                            kz6, cth6, c6, s6);
                    sh.put(2, me, x6, c6, s6);
                    T ev[6], xn[6], zn[6];
                    const T e6 = CIS_TAB(RKF::e(5));
#pragma unroll
                    for (int q = 0; q < 6; ++q) {
                        ev[q] = e6 * (s * (q < 3 ? x6[q < 3 ? 3 + q : 0] : f6[q < 3 ? 0 : q - 3]));
                        xn[q] = zn[q] = T(0);
                    }
                    unrolled<NR>([&](auto l_c) {
                        constexpr int l = decltype(l_c)::value;
                        if constexpr (RKF::e(l) != 0.0) {
                            const T e = CIS_TAB(RKF::e(l));
#pragma unroll
                            for (int q = 0; q < 6; ++q) ev[q] += e * kd[l][q];
                        }
                        if constexpr (RKF::b(l) != 0.0) {
                            const T b = CIS_TAB(RKF::b(l));
#pragma unroll
                            for (int q = 0; q < 6; ++q) {
                                xn[q] += b * kd[l][q];
                                zn[q] += b * zd[l][q];
                            }
                        }
                    });
#pragma unroll
                    for (int q = 0; q < 6; ++q) {
                        emax = fmax(emax, fabs(h * ev[q]));
                        xs[q] = xb[q] += h * xn[q];
                        zs[q] = zb[q] += h * zn[q];
                    }
                }
                __syncthreads();
            });
        }
        sh.fin[me] = xb[2] + xb[5];
        sh.err[me] = emax;
        // a foot's translation takes 0 x the slope of its contact force on flat
        // ground: nothing, or a NaN of its angle
        if (FLAT && c.contact)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                zb[q] += T(0) * zb[2];
                zb[3 + q] += T(0) * zb[2];
            }
        __syncthreads();
        if (on && c.body)
#pragma unroll
            for (int q = 0; q < 6; ++q)
                pack_output(a, k, q < 3 ? 3 * c.b + q : NQ + 3 * c.b + q - 3, xb[q], zb[q]);
    } else {
        T ycc = c.contact ? a.X[(NX + c.i) * a.ldn + k] : T(0);
        T yct = c.torso && c.body ? a.X[(NX + NC) * a.ldn + k] : T(0);
        T emax = T(0);
        PackSums<T, TP, FLAT> sm;
        sm.clear();
        for (int j = 0; j < a.K; ++j) {
            const T jt = T(j), t0 = quotient(jt, Kt, h);
            const T hh = h * h;
            T vm0, vp0, xm0, xp0;
            hold_nodes(t0, vm0, vp0, xm0, xp0);
            T yac = T(0), yat = T(0), yec = T(0), yet = T(0);
#pragma unroll 1
            for (int i = 0; i < NR; ++i) {
                __syncthreads();   // the state wave has left this stage
                const RkfStage st = RKF_STAGES[i];
                const T sb = T(st.b), se = T(st.e);
                // response of a unit mass to the hold weights at the stage input
                StageHold<T> hd;
                hd.tau = quotient(jt + T(st.c), Kt, h);
                hd.w = h * sb;
                hd.sw = sK * sb;
                const T h1 = h * T(st.c), h2 = hh * T(st.ac), h3 = hh * (h * T(st.aac));
                hd.vm = vm0 + (h1 * (T(1) - t0) - h2);
                hd.vp = vp0 + (h1 * t0 + h2);
                hd.xm = xm0 + (h1 * vm0 + h2 * (T(1) - t0) - h3);
                hd.xp = xp0 + (h1 * vp0 + h2 * t0 + h3);
                T cc, ct;
                pack_coef<T, TP, FLAT, true>(c, mc, sh, (NR * j + i) & 1, hd, cc, ct, sm, sr, on);
                sr += R::STAGE;
                yac += sb * s * cc;
                yat += sb * s * ct;
                yec += se * s * cc;
                yet += se * s * ct;
            }
            const T e6 = T(RKF_STAGES[5].e);
            T c6, t6;
            pack_coef<T, TP, FLAT, false>(c, mc, sh, 2, StageHold<T>{}, c6, t6, sm, sr, false);
            yec += e6 * s * c6;
            yet += e6 * s * t6;
            ycc += h * yac;
            yct += h * yat;
            // estimate: the cross-complementarity rows on their lanes, the
            // violation row from the body lanes' parts
            if (c.contact) emax = fmax(emax, fabs(h * yec));
            emax = fmax(emax, fabs(h * row_sum_first<TP::NB>(yet)));
        }
        __syncthreads();
        const T angles = row_sum(sh.fin[me]);
        yct = row_sum(yct);
        const T zct = row_sum(c.body ? sm.zct : T(0));
        T m = fmax(emax, sh.err[me]);
        m = fmax(m, row_ror<8>(m));
        m = fmax(m, row_ror<4>(m));
        m = fmax(m, row_ror<2>(m));
        m = fmax(m, row_ror<1>(m));
        if (on) {
            pack_sums(c, sm, angles, zct, sums, n);
            if (c.contact) pack_output(a, k, NX + c.i, ycc, sm.zcc);
            if (c.torso && c.body) {
                pack_output(a, k, NX + NC, yct, zct);
                if (err) err[k] = m;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// k_rkf_tan: one step of a column.  Velocity rows keep their stage derivatives
// k_l; the pose rows follow from them through the products of the tableau (pose
// rate s v): theta_i = theta + c_i h s w + h^2 s sum (A A)_il k_l.
// ---------------------------------------------------------------------------
template <class T, class TP, bool FLAT>
__device__ __forceinline__ void rkf_tangent_item(const T* __restrict__ rec, T* lds,
                                                 const RedCol& col, int K,
                                                 T (&pb)[RedTopo<TP, FLAT>::NP],
                                                 T (&vb)[RedTopo<TP, FLAT>::NP], T (&ycc)[TP::NC],
                                                 T& yct) {
    using RT = RedTopo<TP, FLAT>;
    using R = PackRec<TP, FLAT>;
    using LN = RedLane<T, TP, FLAT>;
    constexpr int NP = RT::NP, NR = RKF::R;
    const int lane = threadIdx.x & 63;
    LN ln;
    ln.init(rec, lds, col, lane);
    const T s = rec[0], Kt = uniform(T(K)), h = uniform(T(1) / Kt);
    const T hs = uniform(s / Kt), hhs = uniform(s / (Kt * Kt));
    const T* rs = rec + R::HDR;
    const T* last = rs + (int64_t)(NR * K - 1) * R::STAGE;
    T ps[NP], vs[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        pb[p] = p < RT::NU && col.col == p ? T(1) : T(0);
        vb[p] = p < RT::NU && col.col == RT::NU + p ? T(1) : T(0);
        ps[p] = pb[p];
        vs[p] = vb[p];
    }
#pragma unroll
    for (int i = 0; i < TP::NC; ++i) ycc[i] = T(0);
    T kc[R::NVK], cv[2][R::NV], f[2][LN::NFL];
    T yt[4] = {T(0), T(0), T(0), T(0)};
    ln.vectors(rec + R::KC, kc);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        ln.vectors(rs + q * R::STAGE, cv[q]);
        ln.fetch(rs + q * R::STAGE, f[q]);
    }
    ln.place(f[0]);
    // steps in pairs: the coefficient slots alternate over an odd number of stages
    auto step = [&](auto par_c, int j) {
        constexpr int PAR = decltype(par_c)::value;
        const T jt = T(j);
        T kd[NR - 1][NP];
        unrolled<NR>([&](auto i_c) {
            constexpr int I = decltype(i_c)::value, SL = (PAR + I) & 1;
            T k[NP];
            red_rates<T, TP, FLAT>(ln, kc, cv[SL], uniform(quotient(jt + T(RKF::c(I)), Kt, h)), ps,
                                   vs, k, ycc, yt, f[SL ^ 1]);
            const T* ahead = rs + 2 * R::STAGE;
            ahead = ahead < last ? ahead : last;
            ln.vectors(ahead, cv[SL]);
            ln.fetch(ahead, f[SL]);
            // weights of the next stage input (I + 1), or of the step
            if constexpr (I < NR - 1) {
                const T hc = uniform(T(RKF::c(I + 1)) * hs);
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    kd[I][p] = k[p];
                    T v = T(0), x = hc * vb[p];
#pragma unroll
                    for (int l = 0; l <= I; ++l) {
                        v += uniform(h * T(RKF::a(I + 1, l))) * kd[l][p];
                        if (l < I) x += uniform(hhs * T(RKF::aa(I + 1, l))) * kd[l][p];
                    }
                    ps[p] = pb[p] + x;
                    vs[p] = vb[p] + v;
                }
            }
            if constexpr (I == NR - 2) {
                // the step's end but for the last derivative, which the pose does
                // not see (the kept derivatives are not needed beyond)
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    T v = T(0), x = hs * vb[p];
#pragma unroll
                    for (int l = 0; l < NR - 1; ++l) {
                        if (RKF::b(l) != 0.0) v += uniform(h * T(RKF::b(l))) * kd[l][p];
                        if (RKF::ba(l) != 0.0) x += uniform(hhs * T(RKF::ba(l))) * kd[l][p];
                    }
                    kd[0][p] = v;
                    pb[p] += x;
                }
            }
            if constexpr (I == NR - 1) {
                const T w = uniform(h * T(RKF::b(NR - 1)));
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    vs[p] = vb[p] += kd[0][p] + w * k[p];
                    ps[p] = pb[p];
                }
            }
            rs += R::STAGE;
            if constexpr (sizeof(T) == 8) __builtin_amdgcn_sched_barrier(0);
        });
    };
    static_assert(RKF::b(1) == 0.0 && RKF::b(5) == 0.0 && RKF::ba(NR - 1) == 0.0,
                  "the last derivative enters the velocity only");
    for (int j = 0; j < K; j += 2) {
        step(std::integral_constant<int, 0>{}, j);
        if (j + 1 < K) step(std::integral_constant<int, 1>{}, j + 1);
    }
    yct = (yt[0] + yt[1]) + (yt[2] + yt[3]);
}

// Two waves per SIMD on flat ground (quad13, 3,201 intervals, K = 20: 250 us with 68
// bytes of scratch per lane, 280 us at one; one interval per workgroup 1,130 us).
// The sinusoid's frame holds more: one (biped5 on it, up to 400 intervals: 240 us
// against 345 with 272 bytes of scratch).
template <class T, class TP, bool FLAT>
__global__ void __launch_bounds__(128)
    __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? (FLAT ? 2 : 1) : 3)))
    k_rkf_rec(ItemList<T> l, MConst<TP::NB, TP::NJ, TP::NC> mc, T* __restrict__ err) {
    __shared__ PackShared<T, 3> sh;
    red_record_block<T, TP, FLAT>(l, [&](const FwdArgs<T>& a, int item, bool on, int) {
        rkf_rec_item<T, TP, FLAT>(a, mc, l.interval(item), l.records(item), l.sums + item, l.n,
                                  err, on, sh);
    });
}

// Eight values per pair and lane at the fourth stage: FP64 takes one wave per SIMD
// (346 registers for quad13).  3,201 intervals, K = 20: 610 us (two waves per SIMD
// spill 270 bytes per lane and take 1,060 us; one wave per leg and every row and
// column of Z took 4,180 us).
template <class T, class TP, bool FLAT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 1 : 2)))
    k_rkf_tan(ItemList<T> l, const T* __restrict__ recs, const T* __restrict__ sums) {
    __shared__ T lds[RedTopo<TP, FLAT>::LDS];
    red_tangent_block<T, TP, FLAT>(
        l, recs, sums, lds,
        [](const T* rec, T* g, const RedCol& col, int K, auto& pb, auto& vb, auto& ycc, T& yct) {
            rkf_tangent_item<T, TP, FLAT>(rec, g, col, K, pb, vb, ycc, yct);
        });
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
template <int L, int D>
static int64_t rkf_elems_t(const cis_model* m, int K) {
    if constexpr (L >= 1 && D >= 1)
        return m->A == 0.0 ? PackRec<Topo<L, D>, true>::per_interval(K, RKF::R)
                           : PackRec<Topo<L, D>, false>::per_interval(K, RKF::R);
    else return -1;
}

static int64_t rkf_elems_per_interval(const cis_model* m, int K) {
#define CIS_RKF_SZ(LL, DD) \
    if (m->L == LL && m->D == DD) return rkf_elems_t<LL, DD>(m, K);
    CIS_TOPOLOGIES(CIS_RKF_SZ)
#undef CIS_RKF_SZ
    return -1;
}

template <class T, class TP, bool FLAT>
static cis_status rkf_launches(const cis_model* m, ItemList<T>& l, T* err, hipStream_t stream) {
    l.per = PackRec<TP, FLAT>::records(l.one.K, RKF::R);
    l.sums = l.rec + (int64_t)l.n * l.per;
    KLaunch ka, kb;
    ka.arg(l);
    ka.arg(make_const<TP::NB, TP::NJ, TP::NC>(m));
    ka.arg(err);
    ka.func = (const void*)&k_rkf_rec<T, TP, FLAT>;
    ka.grid = dim3(RedGrid<TP, FLAT>::rec_blocks(l.n));
    ka.block = dim3(128);
    hipError_t st = ka.launch(stream);
    if (st != hipSuccess) return fail(CIS_ERR_HIP, "k_rkf_rec launch: %s", hipGetErrorString(st));
    kb.arg(l);
    kb.arg((const T*)l.rec);
    kb.arg((const T*)l.sums);
    kb.func = (const void*)&k_rkf_tan<T, TP, FLAT>;
    kb.grid = dim3(RedGrid<TP, FLAT>::blocks(l.n));
    kb.block = dim3(64 * RedTopo<TP, FLAT>::IPW);
    st = kb.launch(stream);
    if (st != hipSuccess) return fail(CIS_ERR_HIP, "k_rkf_tan launch: %s", hipGetErrorString(st));
    return CIS_OK;
}

template <class T, int L, int D>
static cis_status launch_rkf_t(const cis_model* m, const cis_shape* sh, const void* X,
                               const void* U, const void* s, const void* prm, void* A, void* Bm,
                               void* Bp, void* S, void* defect, void* xprop, void* err, void* ws,
                               hipStream_t stream) {
    if constexpr (L >= 1 && D >= 1) {
        ItemList<T> l;
        std::memset(&l, 0, sizeof(l));
        FwdArgs<T>& a = l.one;
        a.X = (const T*)X;
        a.U = (const T*)U;
        a.s = (const T*)s;
        a.prm = (const T*)prm;
        a.A = (T*)A;
        a.Bm = (T*)Bm;
        a.Bp = (T*)Bp;
        a.S = (T*)S;
        a.defect = (T*)defect;
        a.xprop = (T*)xprop;
        a.ldn = sh->ld_node;
        a.ldi = sh->ld_int;
        a.N = sh->N;
        a.K = sh->substeps;
        a.C = 1;
        l.n = sh->N;
        l.rec = (T*)ws;
        return m->A == 0.0 ? rkf_launches<T, Topo<L, D>, true>(m, l, (T*)err, stream)
                           : rkf_launches<T, Topo<L, D>, false>(m, l, (T*)err, stream);
    } else {
        return fail(CIS_ERR_UNSUPPORTED, "the RKF form needs legs with links");
    }
}

}  // namespace cis

using namespace cis;

static cis_status rkf_ws_bytes(const cis_model* m, const cis_shape* sh, size_t* bytes) {
    const int64_t per = rkf_elems_per_interval(m, sh->substeps);
    if (per < 0) return fail(CIS_ERR_UNSUPPORTED, "RKF form: the model has no legs with links");
    *bytes = (size_t)per * (size_t)sh->N * elem_size(sh->dtype);
    return CIS_OK;
}

extern "C" cis_status cis_rkf_workspace_size(const cis_model* m, const cis_shape* sh,
                                             size_t* bytes) {
    if (!m || !sh || !bytes) return fail(CIS_ERR_NULL, "cis_rkf_workspace_size: null argument");
    if (sh->N < 1 || sh->substeps < 1 || sh->substeps > 4096)
        return fail(CIS_ERR_DIM, "cis_rkf_workspace_size: N=%d, K=%d out of range", sh->N,
                    sh->substeps);
    if (sh->dtype != CIS_F64 && sh->dtype != CIS_F32)
        return fail(CIS_ERR_DTYPE, "cis_rkf_workspace_size: unknown dtype %d", sh->dtype);
    return rkf_ws_bytes(m, sh, bytes);
}

static cis_status discretize_rkf_impl(const cis_model* model, const cis_shape* shape,
                                      const void* X, const void* U, const void* s,
                                      const void* params, int32_t waves, void* A, void* Bm,
                                      void* Bp, void* S, void* defect, void* xprop, void* err,
                                      void* ws, size_t ws_bytes, void* stream) {
    cis_status st = check_common(model, shape, X, U, s, params);
    if (st != CIS_OK) return st;
    if (waves != 1 && waves != 2)
        return fail(CIS_ERR_DIM, "cis_discretize_rkf: waves=%d must be 1 or 2", waves);
    const bool hasm = model->m > 0;
    if (!A || !S || !defect || (hasm && (!Bm || !Bp)))
        return fail(CIS_ERR_NULL, "cis_discretize_rkf: A, S, defect (and Bm, Bp when m > 0) are required");
    const size_t es = elem_size(shape->dtype);
    if (!aligned(A, es) || !aligned(S, es) || !aligned(defect, es) || !aligned(xprop, es) ||
        !aligned(Bm, es) || !aligned(Bp, es) || !aligned(err, es) || !aligned(ws, 8))
        return fail(CIS_ERR_LAYOUT, "cis_discretize_rkf: pointer not aligned to %zu bytes", es);
    size_t need = 0;
    st = rkf_ws_bytes(model, shape, &need);
    if (st != CIS_OK) return st;
    if (!ws || ws_bytes < need)
        return fail(CIS_ERR_WORKSPACE, "cis_discretize_rkf: workspace of %zu bytes needed", need);
    hipStream_t hs = (hipStream_t)stream;
#define CIS_DISPATCH_RKF(LL, DD)                                                               \
    if (model->L == LL && model->D == DD)                                                      \
        return shape->dtype == CIS_F64                                                         \
                   ? launch_rkf_t<double, LL, DD>(model, shape, X, U, s, params, A, Bm, Bp, S, \
                                                  defect, xprop, err, ws, hs)           \
                   : launch_rkf_t<float, LL, DD>(model, shape, X, U, s, params, A, Bm, Bp, S,  \
                                                 defect, xprop, err, ws, hs);
    CIS_TOPOLOGIES(CIS_DISPATCH_RKF)
#undef CIS_DISPATCH_RKF
    return fail(CIS_ERR_UNSUPPORTED, "cis_discretize_rkf: topology has no compiled kernel");
}

extern "C" cis_status cis_discretize_rkf(const cis_model* model, const cis_shape* shape,
                                         const void* X, const void* U, const void* s,
                                         const void* params, int32_t waves, void* A, void* Bm,
                                         void* Bp, void* S, void* defect, void* xprop, void* err,
                                         void* ws, size_t ws_bytes, void* stream) {
    const cis_status st = discretize_rkf_impl(model, shape, X, U, s, params, waves, A, Bm, Bp, S,
                                              defect, xprop, err, ws, ws_bytes, stream);
    if (st != CIS_OK || !debug_finite_enabled()) return st;
    return debug_scan_forward("cis_discretize_rkf", model, shape, model->nx, model->m, X, U, s,
                              params, A, Bm, Bp, S, defect, xprop, err, stream);
}
