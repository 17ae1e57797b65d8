// Split form of the discretize step for many intervals (arxiv 2604.09993,
// Sec. IV-B eq. intg-aug-sys-param; sensitivities by internal numerical
// differentiation, Sec. VI).  Two kernels per batch of intervals:
//
//   k_coefrec : the nominal RK4 recursion with the dilation column S, and the
//               coefficients of every stage (compact records and sums,
//               cis_pack.hpp), four intervals per workgroup of two waves; writes
//               F~, the defect and S.
//   k_tangent : the coupled columns of Z = [Phi_x | B- | B+], one per lane
//               (cis_reduced.hpp), and the closed-form entries of A, B-, B+.
#include <hip/hip_runtime.h>

#include <cstring>

#include "../../include/cis.h"
#include "cis_debug.hpp"
#include "cis_host.hpp"
#include "cis_launch.hpp"
#include "cis_model.hpp"
#include "cis_pack.hpp"
#include "cis_reduced.hpp"

namespace cis {

// Four intervals by two waves, one workgroup barrier per stage: wave 0 the
// nominal recursion and the S column (stage t at step t), wave 1 the
// coefficients, sums and integral rows (stage t - 1 at step t), both on rows of
// 16 body lanes.  k, a: the lane's interval; item: its index in the launch (of
// n); on: not a repeat; most: the largest substep count of the four.
//
// Bound by the length of the two chains (VALU busy 41 % for 12,800 quad13
// intervals), so they are shared between two waves, four intervals fill a wave
// that one would leave three quarters idle, and the constants of the bodies stay
// in LDS.  quad13, K = 20: 200 intervals 70 us, 12,800 370 us (with the
// closed-form rows 560 us); one wave doing both chains held 330 registers and took
// 127 and 540 us; one interval per workgroup of two waves 145 and 1,810 us.
template <class T, class TP, bool FLAT>
__device__ __forceinline__ void coefrec_item(const FwdArgs<T>& a,
                                             const MConst<TP::NB, TP::NJ, TP::NC>& mc, int k,
                                             T* __restrict__ rec, T* __restrict__ sums, int64_t n,
                                             bool on, int most, PackShared<T>& sh) {
    constexpr int NQ = TP::NQ, NX = TP::NX, NC = TP::NC;
    using R = PackRec<TP, FLAT>;
    const int me = threadIdx.x & 63;
    PackBody<T, TP, FLAT> c;
    c.lc = &sh.lc.v[0][me];
    c.load(a, mc, k, me & 15);   // both waves store the same constants
    const int nst = 4 * a.K;
    const T s = c.s, Kt = T(a.K), h = T(1) / Kt, h6 = T(1) / (T(6) * Kt);
    const T sK = s / Kt, s6 = s / (T(6) * Kt);   // the weights with s (one rounding each)
    T* sr = rec + R::HDR;
    __syncthreads();
    if (threadIdx.x < 64) {
        if (on) pack_header(c, h, rec);
        T xb[6], xs[6], xa[6], zb[6], zs[6], za[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            xb[q] = a.X[(q < 3 ? 3 * c.b + q : NQ + 3 * c.b + q - 3) * a.ldn + k];
            xs[q] = xb[q];
            zb[q] = zs[q] = T(0);
        }
        auto stage = [&](auto st_c, int t) {
            constexpr int ST = decltype(st_c)::value;
            if (t < nst) {   // whole rows of 16 lanes
                const T jt = T(t >> 2) + (ST == 0 ? T(0) : (ST == 3 ? T(1) : T(0.5)));
                T f[3], kz[3], cth, cb, sb;
                pack_state<T, TP, FLAT>(c, mc, xs, zs, quotient(jt, Kt, h), f, kz, cth, cb, sb);
                constexpr int sl = ST & 1;
                sh.put(sl, me, xs, cb, sb);
#pragma unroll
                for (int q = 0; q < 6; ++q) sh.z[sl][q][me] = zs[q];
                if (on && c.body) sr[R::CTH + c.b] = cth;
                sr += R::STAGE;
                // pose rows s v (and + v of the nominal state in the S column),
                // velocity rows s f
                constexpr bool outer = ST == 0 || ST == 3;
                const T wx = outer ? h6 : T(2) * h6, ux = outer ? s6 : T(2) * s6;
                const T an = ST == 2 ? h : T(0.5) * h, un = ST == 2 ? sK : T(0.5) * sK;
                T kp[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    kp[q] = s * zs[3 + q] + xs[3 + q];
                    // the substep's increments apart: one rounding of the running
                    // value per substep
                    if constexpr (ST == 0) {
                        xa[q] = ux * xs[3 + q];
                        xa[3 + q] = ux * f[q];
                        za[q] = wx * kp[q];
                        za[3 + q] = wx * kz[q];
                    } else {
                        xa[q] += ux * xs[3 + q];
                        xa[3 + q] += ux * f[q];
                        za[q] += wx * kp[q];
                        za[3 + q] += wx * kz[q];
                    }
                }
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    if constexpr (ST < 3) {
                        xs[q] = xb[q] + un * xs[3 + q];
                        xs[3 + q] = xb[3 + q] + un * f[q];
                        zs[q] = zb[q] + an * kp[q];
                        zs[3 + q] = zb[3 + q] + an * kz[q];
                    } else {
                        xs[q] = xb[q] += xa[q];
                        xs[3 + q] = xb[3 + q] += xa[3 + q];
                        zs[q] = zb[q] += za[q];
                        zs[3 + q] = zb[3 + q] += za[3 + q];
                    }
                }
            }
            __syncthreads();
        };
        for (int t = 0; t < 4 * most; t += 4) {
            stage(std::integral_constant<int, 0>{}, t);
            stage(std::integral_constant<int, 1>{}, t + 1);
            stage(std::integral_constant<int, 2>{}, t + 2);
            stage(std::integral_constant<int, 3>{}, t + 3);
        }
        sh.fin[me] = xb[2] + xb[5];
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
        PackSums<T, TP, FLAT> sm;
        sm.clear();
        StageHold<T> hd;
        T vm0 = T(0), vp0 = T(0), xm0 = T(0), xp0 = T(0), yca = T(0), yta = T(0);
        auto stage = [&](auto st_c, int t) {
            constexpr int ST = decltype(st_c)::value;
            __syncthreads();   // the state wave has left stage t
            if (t >= nst) return;
            const T jt = T(t >> 2) + (ST == 0 ? T(0) : (ST == 3 ? T(1) : T(0.5)));
            // response of a unit mass to the hold weights at the stage input
            const T tp = hd.tau, vmp = hd.vm, vpp = hd.vp;
            hd.tau = quotient(jt, Kt, h);
            constexpr bool outer = ST == 0 || ST == 3;
            hd.w = outer ? h6 : T(2) * h6;
            hd.sw = outer ? s6 : T(2) * s6;
            if constexpr (ST == 0) {
                hold_nodes(hd.tau, vm0, vp0, xm0, xp0);
                hd.vm = vm0;
                hd.vp = vp0;
                hd.xm = xm0;
                hd.xp = xp0;
            } else {
                const T hh = ST == 3 ? h : T(0.5) * h;
                hd.vm = vm0 + hh * (T(1) - tp);
                hd.vp = vp0 + hh * tp;
                hd.xm = xm0 + hh * vmp;
                hd.xp = xp0 + hh * vpp;
            }
            T cc, ct;
            if constexpr (ST == 0) yca = yta = T(0);
            pack_coef<T, TP, FLAT, true>(c, mc, sh, ST & 1, hd, cc, ct, sm, sr, on);
            sr += R::STAGE;
            yca += hd.sw * cc;
            yta += hd.sw * ct;
            if constexpr (ST == 3) {
                ycc += yca;
                yct += yta;
            }
        };
        hd.tau = hd.vm = hd.vp = T(0);
        for (int t = 0; t < 4 * most; t += 4) {
            stage(std::integral_constant<int, 0>{}, t);
            stage(std::integral_constant<int, 1>{}, t + 1);
            stage(std::integral_constant<int, 2>{}, t + 2);
            stage(std::integral_constant<int, 3>{}, t + 3);
        }
        __syncthreads();
        const T angles = row_sum(sh.fin[me]);
        yct = row_sum(yct);
        const T zct = row_sum(c.body ? sm.zct : T(0));
        if (on) {
            pack_sums(c, sm, angles, zct, sums, n);
            if (c.contact) pack_output(a, k, NX + c.i, ycc, sm.zcc);
            if (c.torso && c.body) pack_output(a, k, NX + NC, yct, zct);
        }
    }
}

// RK4 over one interval's coupled columns (one per lane).
template <class T, class TP, bool FLAT>
__device__ __forceinline__ void tangent_item(const T* __restrict__ rec, T* lds,
                                             const RedCol& col, int K,
                                             T (&pb)[RedTopo<TP, FLAT>::NP],
                                             T (&vb)[RedTopo<TP, FLAT>::NP], T (&ycc)[TP::NC],
                                             T& yct) {
    using RT = RedTopo<TP, FLAT>;
    using R = PackRec<TP, FLAT>;
    using LN = RedLane<T, TP, FLAT>;
    constexpr int NP = RT::NP;
    const int lane = threadIdx.x & 63;
    LN ln;
    ln.init(rec, lds, col, lane);
    // step weights in scalar registers: h / 2 and h, h / 6 and h / 3, and times s
    // (one division each: their rounding is the same in every stage)
    const T s = rec[0], Kt = uniform(T(K)), rK = uniform(T(1) / Kt);
    const T h6 = T(1) / (T(6) * Kt), sK = s / Kt, s6 = s / (T(6) * Kt);
    const T hh[2] = {uniform(T(0.5) * rK), rK}, hw[2] = {uniform(h6), uniform(T(2) * h6)};
    const T sh[2] = {uniform(T(0.5) * sK), uniform(sK)}, sw[2] = {uniform(s6), uniform(T(2) * s6)};
    const T* rs = rec + R::HDR;
    const T* last = rs + (int64_t)(4 * K - 1) * R::STAGE;
    T ps[NP], vs[NP], pa[NP], va[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        pb[p] = p < RT::NU && col.col == p ? T(1) : T(0);
        vb[p] = p < RT::NU && col.col == RT::NU + p ? T(1) : T(0);
        ps[p] = pb[p];
        vs[p] = vb[p];
    }
#pragma unroll
    for (int i = 0; i < TP::NC; ++i) ycc[i] = T(0);
    T kc[R::NVK];
    ln.vectors(rec + R::KC, kc);
    // coefficient vectors and forcing entries of stages t and t + 1 (slot t & 1;
    // a third set in flight spilled 90 bytes per lane, and a reload from scratch
    // waits for every load issued before it)
    T cv[2][R::NV], f[2][LN::NFL];
    T yt[4] = {T(0), T(0), T(0), T(0)};
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        ln.vectors(rs + q * R::STAGE, cv[q]);
        ln.fetch(rs + q * R::STAGE, f[q]);
    }
    ln.place(f[0]);
    for (int j = 0; j < K; ++j) {
        const T jt = T(j);
        const T tau0 = uniform(quotient(jt, Kt, rK)), tauh = uniform(quotient(jt + T(0.5), Kt, rK));
        const T tau1 = uniform(quotient(jt + T(1), Kt, rK));
        auto stage = [&](auto st_c, T tau) {
            constexpr int ST = decltype(st_c)::value;
            constexpr int W = (ST == 0 || ST == 3) ? 0 : 1, H = ST == 2 ? 1 : 0;
            T k[NP];
            red_rates<T, TP, FLAT>(ln, kc, cv[ST & 1], tau, ps, vs, k, ycc, yt, f[(ST + 1) & 1]);
            const T* ahead = rs + 2 * R::STAGE;
            ahead = ahead < last ? ahead : last;
            ln.vectors(ahead, cv[ST & 1]);
            ln.fetch(ahead, f[ST & 1]);
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const T v = vs[p];
                // the substep's increments apart: one rounding of the running
                // value per substep
                if constexpr (ST == 0) {
                    pa[p] = sw[W] * v;
                    va[p] = hw[W] * k[p];
                } else {
                    pa[p] += sw[W] * v;
                    va[p] += hw[W] * k[p];
                }
                if constexpr (ST < 3) {
                    ps[p] = pb[p] + sh[H] * v;
                    vs[p] = vb[p] + hh[H] * k[p];
                } else {
                    ps[p] = pb[p] += pa[p];
                    vs[p] = vb[p] += va[p];
                }
            }
            rs += R::STAGE;
            // FP64 fills the registers: work moved across stages spills
            if constexpr (sizeof(T) == 8) __builtin_amdgcn_sched_barrier(0);
        };
        stage(std::integral_constant<int, 0>{}, tau0);
        stage(std::integral_constant<int, 1>{}, tauh);
        stage(std::integral_constant<int, 2>{}, tauh);
        stage(std::integral_constant<int, 3>{}, tau1);
    }
    yct = (yt[0] + yt[1]) + (yt[2] + yt[3]);
}

template <class T, class TP, bool FLAT>
__device__ __forceinline__ void coefrec_block(const ItemList<T>& l,
                                              const MConst<TP::NB, TP::NJ, TP::NC>& mc) {
    __shared__ PackShared<T> sh;
    red_record_block<T, TP, FLAT>(l, [&](const FwdArgs<T>& a, int item, bool on, int most) {
        coefrec_item<T, TP, FLAT>(a, mc, l.interval(item), l.records(item), l.sums + item, l.n, on,
                                  most, sh);
    });
}

template <class T, class TP, bool FLAT>
__global__ void __launch_bounds__(128)
    __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 3)))
    k_coefrec(ItemList<T> l, MConst<TP::NB, TP::NJ, TP::NC> mc) {
    coefrec_block<T, TP, FLAT>(l, mc);
}

// The same with all the registers: FP64 on a sinusoid holds 68 bytes of scratch per
// lane at two waves per SIMD.
template <class T, class TP>
__global__ void __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(1)))
    k_coefrec_sinus(ItemList<T> l, MConst<TP::NB, TP::NJ, TP::NC> mc) {
    coefrec_block<T, TP, false>(l, mc);
}

template <class T, class TP, bool FLAT>
__device__ __forceinline__ void tangent_block(const ItemList<T>& l, const T* __restrict__ recs,
                                              const T* __restrict__ sums) {
    __shared__ T lds[RedTopo<TP, FLAT>::LDS];
    red_tangent_block<T, TP, FLAT>(
        l, recs, sums, lds,
        [](const T* rec, T* g, const RedCol& col, int K, auto& pb, auto& vb, auto& ycc, T& yct) {
            tangent_item<T, TP, FLAT>(rec, g, col, K, pb, vb, ycc, yct);
        });
}

// Registers: six values per pair and lane, so FP64 holds two waves per SIMD up to
// 13 pairs (256 registers, none spilled) and one beyond.  FP32 takes three and two,
// though three cost 336 bytes of scratch per lane for quad13 and 172 for cheetah7, beside
// the stage loop (both launches of 12,800 intervals, K = 20: 960 us and 404 us; at two
// waves and none 1,050 and 463).  quad13, 12,800 intervals, K = 20: 1,010 us (VALU busy 69 %; 5,600 us
// with one wave per leg and every row and column of Z), FP32 700 us (3,000 us).
template <class T, class TP, bool FLAT>
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu((RedTopo<TP, FLAT>::NP > 14 ? 1 : 2) +
                                       (sizeof(T) == 4 ? 1 : 0))))
    k_tangent(ItemList<T> l, const T* __restrict__ recs, const T* __restrict__ sums) {
    tangent_block<T, TP, FLAT>(l, recs, sums);
}

// FP32 at the budget of FP64.
template <class TP, bool FLAT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
    k_tangent_few(ItemList<float> l, const float* __restrict__ recs,
                  const float* __restrict__ sums) {
    tangent_block<float, TP, FLAT>(l, recs, sums);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
static bool split_supported(const cis_model* m) { return m->L >= 1 && m->D >= 1; }

template <int L, int D>
static int64_t split_elems_t(const cis_model* m, int K) {
    if constexpr (L >= 1 && D >= 1)
        return m->A == 0.0 ? PackRec<Topo<L, D>, true>::per_interval(K, 4)
                           : PackRec<Topo<L, D>, false>::per_interval(K, 4);
    else return -1;
}

int64_t split_elems_per_interval(const cis_model* m, int K) {
#define CIS_SPLIT_SZ(LL, DD) \
    if (m->L == LL && m->D == DD) return split_elems_t<LL, DD>(m, K);
    CIS_TOPOLOGIES(CIS_SPLIT_SZ)
#undef CIS_SPLIT_SZ
    return -1;
}

template <int L, int D>
static int64_t split_records_t(const cis_model* m, int K) {
    if constexpr (L >= 1 && D >= 1)
        return m->A == 0.0 ? PackRec<Topo<L, D>, true>::records(K, 4)
                           : PackRec<Topo<L, D>, false>::records(K, 4);
    else return -1;
}

int64_t split_record_elems(const cis_model* m, int K) {
#define CIS_SPLIT_REC(LL, DD) \
    if (m->L == LL && m->D == DD) return split_records_t<LL, DD>(m, K);
    CIS_TOPOLOGIES(CIS_SPLIT_REC)
#undef CIS_SPLIT_REC
    return -1;
}

// The two launches over an item list (FLAT: the model's terrain is flat).
template <class T, class TP, bool FLAT>
static void split_launches(const cis_model* m, const ItemList<T>& l, KLaunch* ka, KLaunch* kb) {
    ka->arg(l);
    ka->arg(make_const<TP::NB, TP::NJ, TP::NC>(m));
    ka->func = (const void*)&k_coefrec<T, TP, FLAT>;
    // Up to about three workgroups per CU (with those of the closed-form rows) a second
    // wave per SIMD only slows the chain (both launches for biped5, K = 20: 333
    // intervals 142 us at two waves and 141 at one, 1,000 185 and 144, 1,500 196 and 157,
    // 2,000 202 and 250).
    if constexpr (!FLAT && sizeof(T) == 8)
        if (l.n <= 6 * device_cus()) ka->func = (const void*)&k_coefrec_sinus<T, TP>;
    ka->grid = dim3(RedGrid<TP, FLAT>::rec_blocks(l.n));
    ka->block = dim3(128);
    kb->arg(l);
    kb->arg((const T*)l.rec);
    kb->arg((const T*)l.sums);
    kb->func = (const void*)&k_tangent<T, TP, FLAT>;
    // FP32 with 13 pairs: while a third wave per SIMD has nothing to hide, its scratch
    // only costs (both launches for quad13, K = 1 / 20: 100 intervals 35 and 96 us at
    // three waves, 29 and 95 at two, 600 46 and 119, 34 and 119, 1,200 51 and 146,
    // 43 and 158; with 7 pairs the two are equal up to 1,200).
    if constexpr (sizeof(T) == 4 && RedTopo<TP, FLAT>::NP > 12 && RedTopo<TP, FLAT>::NP <= 14)
        if (2 * (int64_t)l.n <= 5 * device_cus()) kb->func = (const void*)&k_tangent_few<TP, FLAT>;
    kb->grid = dim3(RedGrid<TP, FLAT>::blocks(l.n));
    kb->block = dim3(64 * RedTopo<TP, FLAT>::IPW);
}

template <class T, int L, int D>
static cis_status launch_split_t(const cis_model* m, const cis_shape* sh, const void* X,
                                 const void* U, const void* s, const void* prm, void* A, void* Bm,
                                 void* Bp, void* S, void* defect, void* xprop, void* ws,
                                 hipStream_t stream) {
    if constexpr (L >= 1 && D >= 1) {
        using TP = Topo<L, D>;
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
        const bool flat = m->A == 0.0;
        l.per = flat ? PackRec<TP, true>::records(a.K, 4) : PackRec<TP, false>::records(a.K, 4);
        l.sums = l.rec + (int64_t)l.n * l.per;
        KLaunch ka, kb;
        if (flat) split_launches<T, TP, true>(m, l, &ka, &kb);
        else split_launches<T, TP, false>(m, l, &ka, &kb);
        hipError_t e = ka.launch(stream);
        if (e != hipSuccess) return fail(CIS_ERR_HIP, "k_coefrec launch: %s", hipGetErrorString(e));
        e = kb.launch(stream);
        if (e != hipSuccess) return fail(CIS_ERR_HIP, "k_tangent launch: %s", hipGetErrorString(e));
        return CIS_OK;
    } else {
        return fail(CIS_ERR_UNSUPPORTED, "split form needs legs with links");
    }
}

template <class T, int L, int D>
static cis_status prep_split_t(const cis_model* m, const BatchGroupDev& g, KLaunch* ka,
                               KLaunch* kb) {
    if constexpr (L >= 1 && D >= 1) {
        using TP = Topo<L, D>;
        ItemList<T> l;
        std::memset(&l, 0, sizeof(l));
        l.descs = (const FwdArgs<T>*)g.fdesc;
        l.items = g.items;
        l.rec_off = g.rec_off;
        l.rec = (T*)g.rec;
        l.sums = (T*)g.sums;
        l.n = g.n_items;
        if (m->A == 0.0) split_launches<T, TP, true>(m, l, ka, kb);
        else split_launches<T, TP, false>(m, l, ka, kb);
        return ka->ok() && kb->ok() ? CIS_OK
                                    : fail(CIS_ERR_DIM, "prep_split_batch: launch record refused");
    } else {
        return fail(CIS_ERR_UNSUPPORTED, "split form needs legs with links");
    }
}

cis_status prep_split_batch(const cis_model* m, int32_t dtype, const BatchGroupDev& g,
                            KLaunch* ka, KLaunch* kb) {
#define CIS_PREP_SPLIT(LL, DD)                                                        \
    if (m->L == LL && m->D == DD)                                                     \
        return dtype == CIS_F64 ? prep_split_t<double, LL, DD>(m, g, ka, kb)          \
                                : prep_split_t<float, LL, DD>(m, g, ka, kb);
    CIS_TOPOLOGIES(CIS_PREP_SPLIT)
#undef CIS_PREP_SPLIT
    return fail(CIS_ERR_UNSUPPORTED, "prep_split_batch: topology has no compiled kernel");
}

bool split_form_supported(const cis_model* m) { return split_supported(m); }

}  // namespace cis

using namespace cis;

static cis_status split_ws_bytes(const cis_model* m, const cis_shape* sh, size_t* bytes) {
    const int64_t per = split_elems_per_interval(m, sh->substeps);
    if (per < 0)
        return fail(CIS_ERR_UNSUPPORTED, "split form: the model has no legs with links");
    *bytes = (size_t)per * (size_t)sh->N * elem_size(sh->dtype);
    return CIS_OK;
}

extern "C" cis_status cis_split_workspace_size(const cis_model* m, const cis_shape* sh,
                                               size_t* bytes) {
    if (!m || !sh || !bytes) return fail(CIS_ERR_NULL, "cis_split_workspace_size: null argument");
    if (sh->N < 1 || sh->substeps < 1 || sh->substeps > 4096)
        return fail(CIS_ERR_DIM, "cis_split_workspace_size: N=%d, K=%d out of range", sh->N,
                    sh->substeps);
    if (sh->dtype != CIS_F64 && sh->dtype != CIS_F32)
        return fail(CIS_ERR_DTYPE, "cis_split_workspace_size: unknown dtype %d", sh->dtype);
    return split_ws_bytes(m, sh, bytes);
}

static cis_status discretize_split_impl(const cis_model* model, const cis_shape* shape,
                                        const void* X, const void* U, const void* s,
                                        const void* params, int32_t waves, void* A, void* Bm,
                                        void* Bp, void* S, void* defect, void* xprop, void* ws,
                                        size_t ws_bytes, void* stream) {
    cis_status st = check_common(model, shape, X, U, s, params);
    if (st != CIS_OK) return st;
    if (waves != 1 && waves != 2)
        return fail(CIS_ERR_DIM, "cis_discretize_split: waves=%d must be 1 or 2", waves);
    const bool hasm = model->m > 0;
    if (!A || !S || !defect || (hasm && (!Bm || !Bp)))
        return fail(CIS_ERR_NULL, "cis_discretize_split: A, S, defect (and Bm, Bp when m > 0) are required");
    const size_t es = elem_size(shape->dtype);
    if (!aligned(A, es) || !aligned(S, es) || !aligned(defect, es) || !aligned(xprop, es) ||
        !aligned(Bm, es) || !aligned(Bp, es) || !aligned(ws, 8))
        return fail(CIS_ERR_LAYOUT, "cis_discretize_split: pointer not aligned to %zu bytes", es);
    size_t need = 0;
    st = split_ws_bytes(model, shape, &need);
    if (st != CIS_OK) return st;
    if (!ws || ws_bytes < need)
        return fail(CIS_ERR_WORKSPACE, "cis_discretize_split: workspace of %zu bytes needed", need);
    hipStream_t hs = (hipStream_t)stream;
#define CIS_DISPATCH_SPLIT(LL, DD)                                                             \
    if (model->L == LL && model->D == DD)                                                      \
        return shape->dtype == CIS_F64                                                         \
                   ? launch_split_t<double, LL, DD>(model, shape, X, U, s, params, A, Bm, Bp, \
                                                    S, defect, xprop, ws, hs)           \
                   : launch_split_t<float, LL, DD>(model, shape, X, U, s, params, A, Bm, Bp,  \
                                                   S, defect, xprop, ws, hs);
    CIS_TOPOLOGIES(CIS_DISPATCH_SPLIT)
#undef CIS_DISPATCH_SPLIT
    return fail(CIS_ERR_UNSUPPORTED, "cis_discretize_split: topology has no compiled kernel");
}

extern "C" cis_status cis_discretize_split(const cis_model* model, const cis_shape* shape,
                                           const void* X, const void* U, const void* s,
                                           const void* params, int32_t waves, void* A, void* Bm,
                                           void* Bp, void* S, void* defect, void* xprop, void* ws,
                                           size_t ws_bytes, void* stream) {
    const cis_status st = discretize_split_impl(model, shape, X, U, s, params, waves, A, Bm, Bp,
                                                S, defect, xprop, ws, ws_bytes, stream);
    if (st != CIS_OK || !debug_finite_enabled()) return st;
    return debug_scan_forward("cis_discretize_split", model, shape, model->nx, model->m, X, U,
                              s, params, A, Bm, Bp, S, defect, xprop, nullptr, stream);
}
