// What the two forms of the paper-faithful dynamics (cis_paper.hip: legs,
// cis_paper_dense.hpp: joint rows) share.
#pragma once
#include <hip/hip_runtime.h>

#include "../../include/cis.h"
#include "cis_model.hpp"
#include "cis_pack.hpp"

namespace cis {

template <int L_, int D_>
struct PTopo {
    static constexpr int L = L_, D = D_;
    static constexpr int NB = 1 + L * D, NJ = L * D, NC = L;
    static constexpr int NQ = 3 * NB, N6 = 6 * NB;
    static constexpr int NY = 4 * NC + 1, NX = N6 + NY;   // augmented state
    static constexpr int M = NJ + 3 * NC, P = NB + 2;
    static constexpr int NJ2 = 2 * NJ, LB = D + 1;
    static constexpr int NCOL = N6 + 2 * M + 1;            // [Phi_x | B- | B+ | S]
    static constexpr int NBLK = (NCOL + 63) / 64;
    static_assert(NB <= 16, "the bodies fit one DPP row");
    static_assert(NJ2 + NQ + 1 <= 64, "one lane per column of the augmented system");
    __host__ __device__ static constexpr int parent(int j) { return (j % D == 0) ? 0 : j; }
    __host__ __device__ static constexpr int cbody(int i) { return D * (i + 1); }
};

struct PaperArgs {
    const double* X;    // [NX][ldn]
    const double* U;    // [M][ldn]
    const double* s;    // [N]
    const double* prm;  // [P]
    double* A;          // [NX][NX][ldi]
    double* Bm;         // [NX][M][ldi]
    double* Bp;
    double* S;          // [NX][ldi]
    double* defect;
    double* xprop;
    double* rec;        // records of every interval
    int64_t ldn, ldi;
    int N, K;
};

__device__ __forceinline__ void plds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

}  // namespace cis
