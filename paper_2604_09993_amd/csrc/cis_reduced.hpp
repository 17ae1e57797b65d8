// Tangent launch of the two-launch discretize forms: the coupled columns of
// Z = [Phi_x | B- | B+], one per lane with all its rows in that lane, and the
// entries that have a closed form (arxiv 2604.09993, Sec. IV-B eq.
// intg-aug-sys-param; the structure is stated in cis_pack.hpp).
//
// What bounds it: FP64 issue of the coupled columns.  A lane holds every
// coupled row of its column, so a stage has no exchange between lanes and no
// workgroup barrier, and every coefficient is the same for the whole wave.
// Vectors of 16 coefficients are loaded ahead, element l & 15 in lane l, and
// enter the FMAs as DPP broadcasts (as scalar loads they missed the scalar cache
// in every stage: 1,900 us against 1,100 us for the columns of 12,800 quad13
// intervals, K = 20).  The forcing entries of B-/B+ columns differ by lane; each wave
// keeps them as a dense matrix [row][control] in LDS (zero except the entries
// of the stage, which the wave writes itself), so lane c reads row r at a fixed
// distance and consecutive lanes read consecutive words.
// Four waves of a workgroup take the same 64 columns of four consecutive
// intervals and store through LDS with the interval index fastest: one store
// instruction covers 32-byte runs instead of 64 separate elements.
// The closed-form entries (three quarters of the output bytes for quad13) are
// written with one interval per lane, 512 contiguous bytes per store
// instruction, by further workgroups of the record launch, whose serial chains
// leave the memory idle: 190 us of 12,800 quad13 intervals there, 380 us here,
// where they took waves from the columns (1.1 GB, 300 us by themselves).
#pragma once
#include <hip/hip_runtime.h>

#include <utility>

#include "cis_pack.hpp"

namespace cis {

// Rows and columns of the reduced system: "pairs" are (position, velocity) rows
// that are integrated per column: the body angles, then on a sinusoid the x
// and then the y of every foot.
template <class TP, bool FLAT>
struct RedTopo {
    static constexpr int NB = TP::NB, NC = TP::NC, M = TP::M;
    static constexpr int NP = NB + (FLAT ? 0 : 2 * NC);
    static constexpr int NU = NB + (FLAT ? 0 : NC);    // pairs with columns of their own
    static constexpr int NCOL = 2 * NU + 2 * M;        // [positions | velocities | B- | B+]
    static constexpr int NBLK = (NCOL + 63) / 64;
    static constexpr int NROW = 2 * NP + NC + 1;
    static constexpr int GM = M + 1;                   // forcing matrix row (last: zero)
    static constexpr int GSZ = NP * GM;
    static constexpr int IPW = 4;                      // intervals (waves) per workgroup
    static constexpr int CHUNK = 8;                    // output rows staged at a time
    static constexpr int LDS = cmax(IPW * GSZ, CHUNK * 64 * IPW);
    // row of A of pair p's position
    __host__ __device__ static constexpr int qrow(int p) {
        return p < NB ? 3 * p + 2
                      : (p < NB + NC ? 3 * TP::cbody(p - NB) : 3 * TP::cbody(p - NB - NC) + 1);
    }
    // closed-form rows: x or y (axis 0 / 1) of a body
    __host__ __device__ static constexpr bool closed(int body) {
        return FLAT || body == 0 || body % TP::D != 0;
    }
    // workgroups (two waves) of the record launch writing the closed-form rows of
    // 64 intervals, a row per wave, beside the 16 that integrate them
    static constexpr int NFILL = (TP::NX + 1) / 2, RECU = 16 + NFILL;
    static_assert(RECU % 16 != 0, "xcd_slot hands out runs of 16: some XCDs would only fill");
};

// The lane's column: index in the block layout, hold weights, control.
struct RedCol {
    int col, ctrl;        // ctrl = M: none
    bool plus;
};

template <class TP, bool FLAT>
__device__ __forceinline__ RedCol red_column(int cb, int lane) {
    using RT = RedTopo<TP, FLAT>;
    RedCol c;
    c.col = cb * 64 + lane;
    const int u = c.col - 2 * RT::NU;
    c.plus = u >= TP::M;
    c.ctrl = (u < 0 || u >= 2 * TP::M) ? TP::M : (c.plus ? u - TP::M : u);
    return c;
}

// Where stage-record forcing element e (0 <= e < NF) goes in the forcing matrix.
template <class TP, bool FLAT>
__device__ __forceinline__ int force_slot(int e) {
    using RT = RedTopo<TP, FLAT>;
    using R = PackRec<TP, FLAT>;
    constexpr int NJ = TP::NJ, NC = TP::NC;
    if (e < 4 * NJ) {
        const int f = e / NJ, j = e - f * NJ;
        const int row = f < 2 ? (j % TP::D == 0 ? 0 : j) : j + 1;
        return row * RT::GM + NJ + 2 * j + (f & 1);
    }
    const int f = (e - 4 * NJ) / NC, i = (e - 4 * NJ) - f * NC, body = TP::D * (i + 1);
    const int q = FLAT ? f : f % 3, r = FLAT ? 2 : f / 3;
    const int row = r == 2 ? body : TP::NB + r * NC + i;
    (void)R::NF;
    return row * RT::GM + 3 * NJ + 3 * i + q;
}

// The wave's view of one interval.
template <class T, class TP, bool FLAT>
struct RedLane {
    using RT = RedTopo<TP, FLAT>;
    using R = PackRec<TP, FLAT>;
    static constexpr int NF = R::NF, NFL = (NF + 63) / 64;
    T* g;              // LDS: the wave's forcing matrix
    const T* gl;       // LDS: row 0 of the lane's control
    int slot[NFL];     // where the lane's forcing elements go
    int src[NFL];      // and where they sit in a stage record
    int row;           // lane within its row of 16
    T wm, wp;          // hold weights of the column

    __device__ __forceinline__ void init(const T* cr, T* gbuf, const RedCol& c, int lane) {
        row = lane & 15;
        g = gbuf;
        gl = gbuf + c.ctrl;
        wm = (c.ctrl < TP::M && !c.plus) ? T(1) : T(0);
        wp = (c.ctrl < TP::M && c.plus) ? T(1) : T(0);
#pragma unroll
        for (int q = 0; q < NFL; ++q) {
            const int e = q * 64 + lane < NF ? q * 64 + lane : 0;   // spare lanes repeat element 0
            src[q] = R::FORCE + e;
            slot[q] = force_slot<TP, FLAT>(e);
        }
        for (int e = lane; e < RT::GSZ; e += 64) g[e] = T(0);
        order();
        // constant entries: torques on both bodies, and on a sinusoid the joint
        // force on the foot it carries
        const T s = cr[0];
        for (int j = lane; j < TP::NJ; j += 64) {
            const int p = j % TP::D == 0 ? 0 : j, b = j + 1;
            g[p * RT::GM + j] = -s * cr[R::IINV + p];
            g[b * RT::GM + j] = s * cr[R::IINV + b];
            if constexpr (!FLAT) {
                if (b % TP::D == 0) {
                    const int i = b / TP::D - 1;
                    const T sm = -s * cr[R::MINV + b];
                    g[(TP::NB + i) * RT::GM + TP::NJ + 2 * j] = sm;
                    g[(TP::NB + TP::NC + i) * RT::GM + TP::NJ + 2 * j + 1] = sm;
                }
            }
        }
        order();
    }
    // the wave's LDS operations execute in order; keep the compiler's too
    __device__ __forceinline__ void order() const {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    __device__ __forceinline__ void fetch(const T* rs, T (&v)[NFL]) const {
#pragma unroll
        for (int q = 0; q < NFL; ++q) v[q] = rs[src[q]];
    }
    template <int NV>
    __device__ __forceinline__ void vectors(const T* at, T (&v)[NV]) const {
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] = at[16 * q + row];
    }
    __device__ __forceinline__ void place(const T (&v)[NFL]) const {
        order();
#pragma unroll
        for (int q = 0; q < NFL; ++q) g[slot[q]] = v[q];
        order();
    }
};

// a_q += (element N_q of the 16-element vector c_q, held by lane N_q of every
// row of 16 lanes) * x_q.  The DPP form of the FMA reads its first factor from
// lane N of the row, so a wave-uniform coefficient costs no instruction and no
// scalar register of its own.  A DPP operand must have been written two wait
// states earlier: s_nop 1.
#define CIS_FMA_ROW4(TYPE, INS)                                                             \
    template <int N0, int N1, int N2, int N3>                                               \
    __device__ __forceinline__ void fma_row4(TYPE& a0, TYPE& a1, TYPE& a2, TYPE& a3,        \
                                             TYPE c0, TYPE c1, TYPE c2, TYPE c3, TYPE x0,   \
                                             TYPE x1, TYPE x2, TYPE x3) {                   \
        asm("s_nop 1\n\t" INS "_dpp %0, %4, %8 row_newbcast:%12 row_mask:0xf bank_mask:0xf\n\t" \
            INS "_dpp %1, %5, %9 row_newbcast:%13 row_mask:0xf bank_mask:0xf\n\t"           \
            INS "_dpp %2, %6, %10 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"          \
            INS "_dpp %3, %7, %11 row_newbcast:%15 row_mask:0xf bank_mask:0xf"              \
            : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3)                                        \
            : "v"(c0), "v"(c1), "v"(c2), "v"(c3), "v"(x0), "v"(x1), "v"(x2), "v"(x3),       \
              "n"(N0), "n"(N1), "n"(N2), "n"(N3));                                          \
    }                                                                                       \
    template <int N0, int N1>                                                               \
    __device__ __forceinline__ void fma_row2(TYPE& a0, TYPE& a1, TYPE c0, TYPE c1, TYPE x0, \
                                             TYPE x1) {                                     \
        asm("s_nop 1\n\t" INS "_dpp %0, %2, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t" \
            INS "_dpp %1, %3, %5 row_newbcast:%7 row_mask:0xf bank_mask:0xf"                \
            : "+v"(a0), "+v"(a1)                                                            \
            : "v"(c0), "v"(c1), "v"(x0), "v"(x1), "n"(N0), "n"(N1));                        \
    }                                                                                       \
    template <int N0>                                                                       \
    __device__ __forceinline__ void fma_row(TYPE& a0, TYPE c0, TYPE x0) {                   \
        asm("s_nop 1\n\t" INS "_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" \
            : "+v"(a0)                                                                      \
            : "v"(c0), "v"(x0), "n"(N0));                                                   \
    }                                                                                       \
    /* a += c0[N0] x0; a += c1[N1] x1 */                                                    \
    template <int N0, int N1>                                                               \
    __device__ __forceinline__ void fma_row_chain(TYPE& a, TYPE c0, TYPE c1, TYPE x0,       \
                                                  TYPE x1) {                                \
        asm("s_nop 1\n\t" INS "_dpp %0, %1, %3 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t" \
            INS "_dpp %0, %2, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf"                \
            : "+v"(a)                                                                       \
            : "v"(c0), "v"(c1), "v"(x0), "v"(x1), "n"(N0), "n"(N1));                        \
    }                                                                                       \
    template <int N0, int N1, int N2>                                                       \
    __device__ __forceinline__ void fma_row3(TYPE& a0, TYPE& a1, TYPE& a2, TYPE c0, TYPE c1, \
                                             TYPE c2, TYPE x0, TYPE x1, TYPE x2) {          \
        asm("s_nop 1\n\t" INS "_dpp %0, %3, %6 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t" \
            INS "_dpp %1, %4, %7 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"           \
            INS "_dpp %2, %5, %8 row_newbcast:%11 row_mask:0xf bank_mask:0xf"               \
            : "+v"(a0), "+v"(a1), "+v"(a2)                                                  \
            : "v"(c0), "v"(c1), "v"(c2), "v"(x0), "v"(x1), "v"(x2), "n"(N0), "n"(N1),       \
              "n"(N2));                                                                     \
    }                                                                                       \
    /* a += c0[N0] x0; b += c1[N1] y0; a += c2[N2] x1; b += c3[N3] y1 */                    \
    template <int N0, int N1, int N2, int N3>                                               \
    __device__ __forceinline__ void fma_row_pair2(TYPE& a, TYPE& b, TYPE c0, TYPE c1,       \
                                                  TYPE c2, TYPE c3, TYPE x0, TYPE y0,       \
                                                  TYPE x1, TYPE y1) {                       \
        asm("s_nop 1\n\t" INS "_dpp %0, %2, %6 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t" \
            INS "_dpp %1, %3, %7 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n\t"           \
            INS "_dpp %0, %4, %8 row_newbcast:%12 row_mask:0xf bank_mask:0xf\n\t"           \
            INS "_dpp %1, %5, %9 row_newbcast:%13 row_mask:0xf bank_mask:0xf"               \
            : "+v"(a), "+v"(b)                                                              \
            : "v"(c0), "v"(c1), "v"(c2), "v"(c3), "v"(x0), "v"(y0), "v"(x1), "v"(y1),       \
              "n"(N0), "n"(N1), "n"(N2), "n"(N3));                                          \
    }                                                                                       \
    /* a chain on two accumulators: a += c[N] x; b += c[N+2] x; a += c[N+1] y; b += c[N+3] y */ \
    template <int N>                                                                        \
    __device__ __forceinline__ void fma_row_joint(TYPE& a, TYPE& b, TYPE c, TYPE x, TYPE y) { \
        asm("s_nop 1\n\t" INS "_dpp %0, %2, %3 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t" \
            INS "_dpp %1, %2, %3 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"            \
            INS "_dpp %0, %2, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"            \
            INS "_dpp %1, %2, %4 row_newbcast:%8 row_mask:0xf bank_mask:0xf"                \
            : "+v"(a), "+v"(b)                                                              \
            : "v"(c), "v"(x), "v"(y), "n"(N), "n"(N + 1), "n"(N + 2), "n"(N + 3));          \
    }
CIS_FMA_ROW4(double, "v_fmac_f64")
CIS_FMA_ROW4(float, "v_fmac_f32")
#undef CIS_FMA_ROW4

// A wave-uniform value in scalar registers.
__device__ __forceinline__ float uniform(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double uniform(double v) {
    const int2 w = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_readfirstlane(w.x),
                                                __builtin_amdgcn_readfirstlane(w.y)));
}

// Compile-time loop: f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>).
template <int N, class F>
__device__ __forceinline__ void unrolled(F&& f) {
    [&]<int... Is>(std::integer_sequence<int, Is...>) {
        (f(std::integral_constant<int, Is>{}), ...);
    }(std::make_integer_sequence<int, N>{});
}

// Derivative of the velocity rows (k) at the stage input (pos, vel), and the
// stage's contribution to the integral rows.  cv: the stage record's
// coefficient vectors, kc: the joints' constants; next: the forcing entries of
// the next stage, put in place once this stage's have been read.
template <class T, class TP, bool FLAT>
__device__ __forceinline__ void red_rates(const RedLane<T, TP, FLAT>& ln,
                                          const T (&kc)[PackRec<TP, FLAT>::NVK],
                                          const T (&cv)[PackRec<TP, FLAT>::NV], T tau,
                                          const T (&pos)[RedTopo<TP, FLAT>::NP],
                                          const T (&vel)[RedTopo<TP, FLAT>::NP],
                                          T (&k)[RedTopo<TP, FLAT>::NP], T (&ycc)[TP::NC],
                                          T (&yct)[4],
                                          const T (&next)[RedLane<T, TP, FLAT>::NFL]) {
    using RT = RedTopo<TP, FLAT>;
    using R = PackRec<TP, FLAT>;
    constexpr int NB = TP::NB, NC = TP::NC;
    // the forcing entries are asked for first and used after the integral rows
    T g[RT::NP];
#pragma unroll
    for (int p = 0; p < RT::NP; ++p) g[p] = ln.gl[p * RT::GM];
    unrolled<NB / 4>([&](auto b_c) {
        constexpr int b = 4 * decltype(b_c)::value, v = R::CV + b;
        fma_row4<v % 16, (v + 1) % 16, (v + 2) % 16, (v + 3) % 16>(
            yct[0], yct[1], yct[2], yct[3], cv[v / 16], cv[(v + 1) / 16], cv[(v + 2) / 16],
            cv[(v + 3) / 16], pos[b], pos[b + 1], pos[b + 2], pos[b + 3]);
    });
    unrolled<NB % 4>([&](auto b_c) {
        constexpr int b = NB - NB % 4 + decltype(b_c)::value, v = R::CV + b;
        fma_row<v % 16>(yct[decltype(b_c)::value], cv[v / 16], pos[b]);
    });
    unrolled<NC>([&](auto i_c) {
        constexpr int i = decltype(i_c)::value, b = TP::cbody(i);
        constexpr int e0 = R::FT + R::NFOOT * i + R::F_CTH, e1 = e0 + 1;
        static_assert(R::F_COM == R::F_CTH + 1, "");
        fma_row_chain<e0 % 16, e1 % 16>(ycc[i], cv[e0 / 16], cv[e1 / 16], pos[b], vel[b]);
    });
    const T wB = ln.wm * (T(1) - tau) + ln.wp * tau;
#pragma unroll
    for (int p = 0; p < RT::NP; ++p) k[p] = wB * g[p];
    ln.place(next);   // every lane has its entries of this stage
    unrolled<NB / 4>([&](auto b_c) {
        constexpr int b = 4 * decltype(b_c)::value, v = R::CTH + b;
        fma_row4<v % 16, (v + 1) % 16, (v + 2) % 16, (v + 3) % 16>(
            k[b], k[b + 1], k[b + 2], k[b + 3], cv[v / 16], cv[(v + 1) / 16], cv[(v + 2) / 16],
            cv[(v + 3) / 16], pos[b], pos[b + 1], pos[b + 2], pos[b + 3]);
    });
    unrolled<NB % 4>([&](auto b_c) {
        constexpr int b = NB - NB % 4 + decltype(b_c)::value, v = R::CTH + b;
        fma_row<v % 16>(k[b], cv[v / 16], pos[b]);
    });
    unrolled<TP::NJ>([&](auto j_c) {
        constexpr int j = decltype(j_c)::value, p = TP::parent(j), c = j + 1;
        fma_row_joint<4 * j % 16>(k[p], k[c], kc[4 * j / 16], pos[c] - pos[p], vel[c] - vel[p]);
    });
    unrolled<NC>([&](auto i_c) {
        constexpr int i = decltype(i_c)::value, b = TP::cbody(i), f = R::FT + R::NFOOT * i;
        auto at = [&](auto q_c, T& acc, T x) {
            constexpr int e = f + decltype(q_c)::value;
            fma_row<e % 16>(acc, cv[e / 16], x);
        };
        if constexpr (!FLAT) {
#define CIS_AT(F, ACC, X) at(std::integral_constant<int, R::F>{}, ACC, X)
            constexpr int px = NB + i, py = NB + NC + i;
            CIS_AT(F_XX, k[px], pos[px]);
            CIS_AT(F_YX, k[py], pos[px]);
            CIS_AT(F_TX, k[b], pos[px]);
            CIS_AT(F_ZX, yct[0], pos[px]);
            CIS_AT(F_XT, k[px], pos[b]);
            CIS_AT(F_YT, k[py], pos[b]);
            CIS_AT(F_ZY, yct[1], pos[py]);
            CIS_AT(F_CX, ycc[i], pos[px]);
            CIS_AT(F_CY, ycc[i], pos[py]);
            CIS_AT(F_CVX, ycc[i], vel[px]);
            CIS_AT(F_CVY, ycc[i], vel[py]);
#undef CIS_AT
        }
    });
}

// Integral rows of a B-/B+ column: the share of the translations with a closed
// form (and of the contact force itself), from the interval's sums.
template <class T, class TP, bool FLAT>
__device__ __forceinline__ void red_integrals(const RedCol& c, const T* __restrict__ cr,
                                              const T* __restrict__ sums, int64_t n,
                                              T (&ycc)[TP::NC], T& yct) {
    using RT = RedTopo<TP, FLAT>;
    using R = PackRec<TP, FLAT>;
    constexpr int NB = TP::NB, NC = TP::NC, NJ = TP::NJ, D = TP::D;
    if (c.ctrl >= TP::M || c.ctrl < NJ) return;
    const T s = cr[0];
    const int q = c.plus ? 3 : 2;
    auto body = [&](int b, int ax, T f) {   // f: force per unit control (+-1) over the mass
        if (!RT::closed(b)) return;
        yct += (s * f) * sums[((ax ? R::RY : R::RX) + q * NB + b) * n];
        if (b > 0 && b % D == 0) {   // flat ground: the foot's own integral row
            const int i = b / D - 1;
            const T v = ax ? (s * f) * sums[(R::EY + q * NC + i) * n]
                           : f * sums[(R::EX + (q - 1) * NC + i) * n];
#pragma unroll
            for (int e = 0; e < NC; ++e) ycc[e] += e == i ? v : T(0);
        }
    };
    if (c.ctrl < 3 * NJ) {
        const int j = (c.ctrl - NJ) >> 1, ax = (c.ctrl - NJ) & 1;
        const int p = j % D == 0 ? 0 : j, b = j + 1;
        body(p, ax, s * cr[R::MINV + p]);
        body(b, ax, -(s * cr[R::MINV + b]));
    } else {
        const int i = (c.ctrl - 3 * NJ) / 3, f = (c.ctrl - 3 * NJ) % 3, b = D * (i + 1);
        const T sm = s * cr[R::MINV + b];
        body(b, f == 0 ? 1 : 0, f == 2 ? -sm : sm);
        const T v = sums[(R::GC + f * NC + i) * n];
#pragma unroll
        for (int e = 0; e < NC; ++e) ycc[e] += e == i ? v : T(0);
    }
}

// Where a workgroup's intervals live: trajectory arguments and interval index.
template <class T>
struct RedDst {
    T* A;
    T* Bm;
    T* Bp;
    int64_t ldi;
    int k;
};
template <class T>
__device__ __forceinline__ RedDst<T> red_dst(const FwdArgs<T>& a, int k) {
    return RedDst<T>{a.A, a.Bm, a.Bp, a.ldi, k};
}

// Store of a workgroup's columns: wave w holds interval w's pos/vel/ycc/yct of
// 64 columns; through LDS so that thread (column, interval) has the interval
// fastest.  dst(e): destination of the workgroup's interval e; valid(e).
template <class T, class TP, bool FLAT, class DST>
__device__ __forceinline__ void red_store(T* lds, int cb, const T (&pos)[RedTopo<TP, FLAT>::NP],
                                          const T (&vel)[RedTopo<TP, FLAT>::NP],
                                          const T (&ycc)[TP::NC], T yct, int n_valid, DST&& dst) {
    using RT = RedTopo<TP, FLAT>;
    constexpr int NP = RT::NP, NC = TP::NC, NX = TP::NX, NXT = TP::NXT, NQ = TP::NQ, M = TP::M;
    constexpr int IPW = RT::IPW, CHUNK = RT::CHUNK, NROW = RT::NROW;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int e = tid & (IPW - 1), cl = tid / IPW;   // interval and column of the thread's stores
    const RedCol c = red_column<TP, FLAT>(cb, cl);
    const bool on = e < n_valid && c.col < RT::NCOL;
    const RedDst<T> d = dst(e < n_valid ? e : 0);
    T* out;
    int64_t rs;   // elements from a row to the next
    if (c.ctrl == M) {
        const int u = c.col < RT::NU ? c.col : c.col - RT::NU;
        const int q = u < TP::NB ? 3 * u + 2 : 3 * (TP::D * (u - TP::NB + 1));
        out = d.A + (int64_t)(c.col < RT::NU ? q : NQ + q) * d.ldi;
        rs = (int64_t)NXT * d.ldi;
    } else {
        out = (c.plus ? d.Bp : d.Bm) + (int64_t)c.ctrl * d.ldi;
        rs = (int64_t)M * d.ldi;
    }
    out += d.k;
#pragma unroll
    for (int r0 = 0; r0 < NROW; r0 += CHUNK) {
        __syncthreads();
#pragma unroll
        for (int r = r0; r < r0 + CHUNK && r < NROW; ++r) {
            const T v = r < NP ? pos[r < NP ? r : 0]
                               : (r < 2 * NP ? vel[r >= NP && r < 2 * NP ? r - NP : 0]
                                             : (r < 2 * NP + NC
                                                    ? ycc[r >= 2 * NP && r < 2 * NP + NC ? r - 2 * NP : 0]
                                                    : yct));
            lds[((r - r0) * 64 + lane) * IPW + wave] = v;
        }
        __syncthreads();
#pragma unroll
        for (int r = r0; r < r0 + CHUNK && r < NROW; ++r) {
            const T v = lds[(r - r0) * 64 * IPW + tid];
            const int row = r < NP ? RT::qrow(r)
                                   : (r < 2 * NP ? NQ + RT::qrow(r - NP) : NX + r - 2 * NP);
            if (on) out[row * rs] = v;
        }
    }
}

// Closed-form entries of 64 intervals (one per lane), row r of A, B- and B+.
// pz: 0, or NaN where a coefficient of the row is not finite.  The pose and
// velocity rows need nothing of the recursion (s, sm = s / m of the row's body
// and pz = 0), except that NaN: the tangent launch writes them again for such
// intervals.
template <class T, class TP, bool FLAT>
__device__ __forceinline__ void red_fill_row(int r, const RedDst<T>& d, T s, T sm, T pz,
                                             const T* __restrict__ sums, int64_t n, bool on) {
    using RT = RedTopo<TP, FLAT>;
    using R = PackRec<TP, FLAT>;
    constexpr int NB = TP::NB, NC = TP::NC, NJ = TP::NJ, NQ = TP::NQ, NX = TP::NX, NXT = TP::NXT;
    constexpr int M = TP::M, D = TP::D;
    (void)NXT;
    const bool qr = r < NQ, vr = r >= NQ && r < NX;
    const int b = qr ? r / 3 : (vr ? (r - NQ) / 3 : 0);
    const int ax = qr ? r % 3 : (vr ? (r - NQ) % 3 : 0);
    const bool angle = (qr || vr) && ax == 2;
    const bool foot = b > 0 && b % D == 0;
    // zero entries: 0, or what 0 x (non-finite coefficients) leaves in such rows
    T zero = T(0);
    if (angle || foot || r >= NX) zero += pz;
    if (qr) zero += T(0) * s;
    T* out = d.A + ((int64_t)r * NXT) * d.ldi + d.k;
    const bool pairs = (qr || vr) && !angle && !FLAT && foot;   // rows integrated per column
    const bool coupled_row = angle || pairs || r >= NX;
    const int64_t ldi = d.ldi;
    // pose and velocity columns, body by body
#pragma unroll
    for (int cv = 0; cv < 2; ++cv) {
        for (int cb = 0; cb < NB; ++cb) {
            const bool cfoot = cb > 0 && cb % D == 0;
#pragma unroll
            for (int ca = 0; ca < 3; ++ca, out += ldi) {
                // columns integrated per lane cover the coupled rows only
                const bool coupled = ca == 2 || (!FLAT && cfoot && ca == 0);
                if (coupled && coupled_row) continue;
                const int c = cv * NQ + 3 * cb + ca;
                T v = zero;
                if (!coupled) {
                    if (r < NX) {
                        if (c == r) v += T(1);
                        else if (qr && c == r + NQ) v += s;
                    } else if (r == NX + NC) {
                        const T w = sums[((ca ? R::RY : R::RX) + (cv ? NB : 0) + cb) * n];
                        v += cv ? s * w : w;
                    } else if (cfoot && D * (r - NX + 1) == cb) {
                        const int i = r - NX;
                        if (ca == 1)
                            v += cv ? s * sums[(R::EY + NC + i) * n] + sums[(R::EV + i) * n]
                                    : sums[(R::EY + i) * n];
                        else if (cv) v += sums[(R::EX + i) * n];
                    }
                }
                if (on) *out = v;
            }
        }
    }
    // integral-state columns
    for (int c = NX; c < NXT; ++c, out += ldi)
        if (on) *out = c == r ? T(1) : T(0);
    // B-/B+ of the translations with a closed form
    if (!(qr || vr) || angle || pairs) return;
    const T full = qr ? s * sm : sm;
    const T um = qr ? full / T(3) : T(0.5) * full, up = qr ? full / T(6) : um;
    T* bm = d.Bm + ((int64_t)r * M) * ldi + d.k;
    T* bp = d.Bp + ((int64_t)r * M) * ldi + d.k;
    auto put = [&](T sg) {
        T vm = zero, vp = zero;
        if (sg != T(0)) {
            vm += sg * um;
            vp += sg * up;
        }
        if (on) {
            *bm = vm;
            *bp = vp;
        }
        bm += ldi;
        bp += ldi;
    };
    for (int c = 0; c < NJ; ++c) put(T(0));
    for (int j = 0; j < NJ; ++j) {
        const T sg = j + 1 == b ? T(-1) : ((j % D == 0 ? 0 : j) == b ? T(1) : T(0));
        put(ax == 0 ? sg : T(0));
        put(ax == 1 ? sg : T(0));
    }
    for (int i = 0; i < NC; ++i) {
        const bool own = D * (i + 1) == b;
        put(own && ax == 1 ? T(1) : T(0));
        put(own && ax == 0 ? T(1) : T(0));
        put(own && ax == 0 ? T(-1) : T(0));
    }
}

// Grid of the tangent launch: blocks of 64 intervals with 16 NBLK column
// workgroups each (the intervals of a column block consecutive), then one
// workgroup per 64 intervals for the closed-form entries of the integral rows.
template <class TP, bool FLAT>
struct RedGrid {
    using RT = RedTopo<TP, FLAT>;
    static constexpr int GI = 64 / RT::IPW;            // interval groups per block
    static constexpr int UNITS = GI * RT::NBLK;
    __host__ __device__ static constexpr int blocks(int n) { return (n + 63) / 64 * (UNITS + 1); }
    __host__ __device__ static constexpr int rec_blocks(int n) { return (n + 63) / 64 * RT::RECU; }
};

// Row r's closed-form entries before the recursion: inputs straight from the
// caller's arrays (record launch).
template <class T, class TP, bool FLAT>
__device__ __forceinline__ void red_fill_early(int r, const FwdArgs<T>& a, int k, bool on) {
    const int b = (r < TP::NQ ? r : r - TP::NQ) / 3;
    const T s = a.s[k], sm = s * (T(1) / a.prm[2 + b]);
    red_fill_row<T, TP, FLAT>(r, red_dst(a, k), s, sm, T(0), (const T*)nullptr, 0, on);
}

// The integral rows' closed-form entries of 64 intervals, and every row again
// where the interval is not finite (tangent launch).
template <class T, class TP, bool FLAT>
__device__ __forceinline__ void red_fill_late(int wave, int waves, const RedDst<T>& d,
                                              const T* __restrict__ cr,
                                              const T* __restrict__ sums, int64_t n, bool on) {
    using R = PackRec<TP, FLAT>;
    const T s = cr[0], pz = sums[R::PZ * n];
    for (int r = TP::NX + wave; r < TP::NXT; r += waves) {
        const int q = r == TP::NX + TP::NC ? 1 : 2 + r - TP::NX;
        red_fill_row<T, TP, FLAT>(r, d, s, T(0), sums[(R::PZ + q) * n], sums, n, on);
    }
    const bool bad = on && !(pz == T(0));
    if (!__any(bad)) return;
    for (int r = wave; r < TP::NX; r += waves) {
        const int b = (r < TP::NQ ? r : r - TP::NQ) / 3;
        red_fill_row<T, TP, FLAT>(r, d, s, s * cr[R::MINV + b], pz, sums, n, bad);
    }
}

// Single trajectory: items are its intervals; batch: the work list's.
template <class T>
struct ItemList {
    const FwdArgs<T>* descs;   // NULL: one trajectory, `one`
    const int2* items;
    const int64_t* rec_off;    // batch: element offset of an item's records
    T* rec;
    T* sums;                   // [SUM][n]
    int n;
    FwdArgs<T> one;
    int64_t per;               // one trajectory: elements of an interval's records

    __device__ __forceinline__ int interval(int item) const {
        return descs ? items[item].y : item;
    }
    __device__ __forceinline__ FwdArgs<T> args(int item) const {
        FwdArgs<T> a = one;
        if (descs) a = descs[items[item].x];
        return a;
    }
    __device__ __forceinline__ T* records(int item) const {
        return rec + (descs ? rec_off[item] : (int64_t)item * per);
    }
};

// Workgroup of the record launch: closed-form rows, or four intervals of
// integrate(args, item, not a repeat, largest substep count of the four).
template <class T, class TP, bool FLAT, class F>
__device__ __forceinline__ void red_record_block(const ItemList<T>& l, F&& integrate) {
    using RT = RedTopo<TP, FLAT>;
    const int u = xcd_slot(blockIdx.x, gridDim.x);
    const int blk = u / RT::RECU, w = u - blk * RT::RECU, lane = (int)threadIdx.x & 63;
    if (w >= 16) {
        const int want = blk * 64 + lane, item = want < l.n ? want : l.n - 1;
        const FwdArgs<T> a = l.args(item);
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        const int r = 2 * (w - 16) + wave;
        if (r < TP::NX) red_fill_early<T, TP, FLAT>(r, a, l.interval(item), want == item);
        return;
    }
    const int want = blk * 64 + 4 * w + (lane >> 4);
    if (blk * 64 + 4 * w >= l.n) return;
    const int item = want < l.n ? want : l.n - 1;
    const FwdArgs<T> a = l.args(item);
    int most = a.K;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int v = __builtin_amdgcn_readlane(a.K, 16 * q);
        most = v > most ? v : most;
    }
    integrate(a, item, want == item, most);
}

// Workgroup of the tangent launch: four intervals of 64 columns, or the late
// closed-form entries.  integrate(records, LDS, column, substeps, positions,
// velocities, ycc, yct).
template <class T, class TP, bool FLAT, class F>
__device__ __forceinline__ void red_tangent_block(const ItemList<T>& l, const T* __restrict__ recs,
                                                  const T* __restrict__ sums, T* lds,
                                                  F&& integrate) {
    using RT = RedTopo<TP, FLAT>;
    using RG = RedGrid<TP, FLAT>;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int u = xcd_slot(blockIdx.x, gridDim.x);
    const int nblk = (l.n + 63) / 64;
    if (u >= nblk * RG::UNITS) {
        const int want = (u - nblk * RG::UNITS) * 64 + lane, item = want < l.n ? want : l.n - 1;
        red_fill_late<T, TP, FLAT>(wave, RT::IPW, red_dst(l.args(item), l.interval(item)),
                                   recs + (l.records(item) - l.rec), sums + item, l.n,
                                   want == item);
        return;
    }
    const int blk = u / RG::UNITS, w = u - blk * RG::UNITS;
    const int cb = w / RG::GI, first = blk * 64 + (w - cb * RG::GI) * RT::IPW;
    if (first >= l.n) return;
    const int item = first + wave < l.n ? first + wave : l.n - 1;
    const T* rec = recs + (l.records(item) - l.rec);
    const RedCol col = red_column<TP, FLAT>(cb, lane);
    T pb[RT::NP], vb[RT::NP], ycc[TP::NC], yct;
    integrate(rec, lds + wave * RT::GSZ, col, l.args(item).K, pb, vb, ycc, yct);
    red_integrals<T, TP, FLAT>(col, rec, sums + item, l.n, ycc, yct);
    red_store<T, TP, FLAT>(lds, cb, pb, vb, ycc, yct, l.n - first < RT::IPW ? l.n - first : RT::IPW,
                           [&](int e) { return red_dst(l.args(first + e), l.interval(first + e)); });
}

}  // namespace cis
