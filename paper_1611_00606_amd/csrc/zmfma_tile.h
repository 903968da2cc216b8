// Shared definitions of the complex-double MFMA tile engines for gfx950
// (zmfma_direct.h, zmfma_atom.h): operand segments, tile shapes,
// accumulators and the accumulator layout.
//
// An engine computes one BM x BN tile of   C = sum_s P_s^H Q_s   where every
// operand is a row-major complex matrix whose rows are the contraction index
// and whose columns are the output index (this is how the stacked operands
// are laid out: A, B, X, Y are [K][N_G], and the T blocks [N_L][N_L]).
// Segments (P_s, Q_s) of equal length are concatenated along the contraction
// index, so one K-loop covers e.g. A^H X + B^H Y of the H reduction.
//
// One complex multiply-add conj(p) q is 4 real FP64 MFMA products:
//   Re += p.re q.re + p.im q.im,   Im += p.re q.im - p.im q.re
// issued as V_MFMA_F64_16X16X4_F64 on 16x16 output blocks with a K step of 4.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hs {

typedef double v4d __attribute__((ext_vector_type(4)));

// NSEG segments of `len` rows each (nseg <= NSEG of them active), forming
// the contraction index kk = s * len + r. Row r of segment s contributes
// conj(P_s[r][m]) * w * Q_s[r][n] to C[m][n] with w = qscale[kk] (SCALE;
// qscale covers the whole contraction index, nseg * len entries), else 1.
template <int NSEG, bool SCALE>
struct Segs {
    const double2 *P[NSEG];
    const double2 *Q[NSEG];
    int nseg;
    int len;
    long long ldp, ldq;   // row strides, in complex elements
    const double *qscale;
};

template <class C>
struct Acc {
    v4d re[C::TM][C::TN];
    v4d im[C::TM][C::TN];
};

// v[seg], formed arithmetically: a chain of selects between pointers read
// from the table is turned into one load at a selected address, which moves
// the whole table into scratch memory.
template <int NSEG>
__device__ __forceinline__ const double2 *pick(const double2 *const (&v)[NSEG], int seg) {
    const uintptr_t base = reinterpret_cast<uintptr_t>(v[0]);
    uintptr_t p = base;
#pragma unroll
    for (int i = 1; i < NSEG; ++i) p += (seg == i) ? reinterpret_cast<uintptr_t>(v[i]) - base : 0;
    return reinterpret_cast<const double2 *>(p);
}

// Output coordinates of accumulator element v of block (i, j) for this lane.
// Operand layouts of V_MFMA_F64_16X16X4_F64: lane l holds A[l % 16][l / 16]
// and B[l / 16][l % 16]; result element v of lane l is D[4 v + l / 16][l % 16]
// (measured on gfx950 with a one-wave probe of known integer operands).
template <class C>
__device__ __forceinline__ int acc_row(int i, int v) {
    const int wave = threadIdx.x >> 6;
    return (wave % C::WM) * C::WTM + i * 16 + 4 * v + ((threadIdx.x & 63) >> 4);
}
template <class C>
__device__ __forceinline__ int acc_col(int j) {
    const int wave = threadIdx.x >> 6;
    return (wave / C::WM) * C::WTN + j * 16 + (threadIdx.x & 15);
}

}  // namespace hs
