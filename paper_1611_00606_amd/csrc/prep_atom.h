// The Cholesky of T^AA_a with failure detection (Alg. 1, the try step of the
// second loop; Sec. 2 explains that T^AA_a is HPD in theory but the
// factorization may fail numerically) as a block-level device routine, run by
// extra blocks of the per-atom product launches (k_atom, k_batch) and by
// k_chol. It reports info[a] only: the products use T^AA_a itself, on both
// branches, so nothing waits for the factorization.
//
// The lower triangle of T^AA_a is spread over the block's registers (entry
// e = i(i+1)/2 + k of the packed triangle, k <= i, in slot e / NT of thread
// e % NT; for N_L = 128, 17 entries per thread of a 512-thread block); only
// the current column passes through LDS. The factorization (chol_atom) is
// right-looking with one barrier per column; a pivot that is not > 0 (NaN
// included) stops it and sets info = j+1, the LAPACK zpotrf convention.
#pragma once

#include "hs_internal.h"
#include "../../include/hs_build.h"

namespace hs {

constexpr int PACKED_MAX = HS_MAX_NL * (HS_MAX_NL + 1) / 2;
// LDS the routine needs: two column buffers of HS_MAX_NL complex values
constexpr int CHOL_LDS_BYTES = 2 * HS_MAX_NL * 16;
constexpr int CHOL_THREADS = 512;

// Right-looking Cholesky of the n x n Hermitian block t (row-major; its lower
// triangle is read) by one block of NT threads (every thread calls it), the
// triangle held in registers as described above. Before step j every entry
// (i, k), k >= j, holds L_ik = t_ik - sum_{m<j} C_im conj(C_km), and column j
// (rows i >= j) is also in the LDS buffer col[j & 1]. Step j tests the pivot
// L_jj, turns column j into C_ij = L_ij / sqrt(L_jj), subtracts
// C_ij conj(C_kj) from every entry (i, k) with k > j, and writes the updated
// column j + 1 into col[(j + 1) & 1] for the next step. Returns 0 or the
// 1-based index of the first pivot that is not > 0 (NaN included), at which
// the factorization stopped.
template <int NT>
__device__ __forceinline__ int chol_atom(const double2 *__restrict__ t, int n, double2 *col) {
    constexpr int NS = (PACKED_MAX + NT - 1) / NT;
    int tid = threadIdx.x;
    // opaque to the compiler, so that the slot decoding below is not hoisted
    // out of a caller's loop (where it would hold registers throughout)
    asm volatile("" : "+v"(tid));
    const int ntri = n * (n + 1) / 2;
    double2 v[NS];
    int ik[NS];   // i << 8 | k of each slot's entry, -1 for none
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int e = s * NT + tid;
        int i = (int)((sqrt(8.0 * e + 1.0) - 1.0) * 0.5);
        if (i * (i + 1) / 2 > e) --i;
        if ((i + 1) * (i + 2) / 2 <= e) ++i;
        ik[s] = e < ntri ? i << 8 | (e - i * (i + 1) / 2) : -1;
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int i = ik[s] >> 8, k = ik[s] & 255;
        v[s] = ik[s] < 0 ? double2{0.0, 0.0} : t[i * n + k];
        if (ik[s] >= 0 && k == 0) col[i] = v[s];
    }
    __syncthreads();
    for (int j = 0; j < n; ++j) {
        const double2 *cj = col + (j & 1) * HS_MAX_NL;
        double2 *cn = col + ((j + 1) & 1) * HS_MAX_NL;
        const double ljj = cj[j].x;
        if (!(ljj > 0.0)) return j + 1;   // the same value in every thread
        const double rs = 1.0 / sqrt(ljj);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            // decoded anew each step rather than kept decoded in registers
            asm volatile("" : "+v"(ik[s]));
            const int i = ik[s] >> 8, k = ik[s] & 255;
            if (ik[s] < 0 || k <= j) continue;
            const double2 a = cj[i], b = cj[k];
            const double ax = a.x * rs, ay = a.y * rs, bx = b.x * rs, by = b.y * rs;
            // v -= C_ij conj(C_kj)
            v[s].x -= ax * bx + ay * by;
            v[s].y -= ay * bx - ax * by;
            if (k == j + 1) cn[i] = v[s];
        }
        __syncthreads();
    }
    return 0;
}

// info[a] of atom a by one block of CHOL_THREADS threads (every thread calls
// it). lds: CHOL_LDS_BYTES of LDS, free for the caller when it returns.
__device__ __forceinline__ void chol_info(const Atoms &at, int a, const double2 *__restrict__ T_AA,
                                          int *__restrict__ info, char *lds) {
    const int n = at.row_off[a + 1] - at.row_off[a];
    const int f = chol_atom<CHOL_THREADS>(T_AA + at.t_off[a], n, reinterpret_cast<double2 *>(lds));
    if (threadIdx.x == 0) info[a] = f;
    __syncthreads();
}

}  // namespace hs
