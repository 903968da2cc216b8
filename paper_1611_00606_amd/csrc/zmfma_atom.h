// Complex-double MFMA tile engine of the per-atom products (k_atom, k_batch):
// one tile of C = sum_s P_s^H Q_s with the operands moved global -> LDS by
// 16-byte direct loads (global_load_lds_dwordx4; lane l lands at base + 16 l),
// as in zmfma_direct.h, but shaped for the per-atom operands:
//
// * the tile's rows are the atom's N_L output rows (up to 128, in blocks of
//   16) and its columns 128 or 256 plane-wave columns, so one tile usually
//   covers every row of an atom: the A and B columns of a tile are read once
//   instead of once per 32-row tile;
// * the P rows (the atom's N_L x N_L blocks) are N_L entries long: a P row is
//   loaded as 64-column pieces with the columns past N_L clamped to the last
//   one (they only feed output rows past N_L, which are not stored);
// * a P of the first segment given transposed (X_a's T^AB_a, whose rows are
//   X_a's rows): lane m of a load reads element (m, k) at its own stride and
//   the fragment's imaginary part changes sign in registers, so no
//   conjugate-transposed copy of T^AB_a is made. Its 16-byte loads gather one
//   cache line each, but eight contraction rows share a line and the P rows
//   are a small part of a tile's loads;
// * a last stage whose second half holds no contraction rows skips it.
//
// Waves: 2 x 4; wave w takes block row w / 4 and block column w % 4, so each
// SIMD (waves w and w + 4) holds one wave of each block row.
#pragma once

#include "zmfma_tile.h"

namespace hs {

template <int TM_, int TN_, int BK_>
struct AtomCfg {
    static constexpr int WM = 2, WN = 4;
    static constexpr int NT = 64 * WM * WN;
    static constexpr int TM = TM_, TN = TN_, BK = BK_;
    static constexpr int WTM = 16 * TM, WTN = 16 * TN;   // wave tile
    static constexpr int BM = WM * WTM, BN = WN * WTN;   // tile
    static constexpr int BMS = (BM + 63) / 64 * 64;      // LDS row width of P
    static constexpr int BNS = BN;                       // LDS row width of Q
    static constexpr int PH = BMS / 64, QH = BNS / 64;   // 64-column loads per row
    static constexpr int STAGE = BK * (BMS + BNS);       // complex elements per stage
    static constexpr int LDS_ELEMS = 2 * STAGE;
    static_assert(BN % 64 == 0, "64-column loads of Q");
    static_assert(BK == 8 || BK == 16, "each wave loads BK / 8 rows of a stage");
    static_assert(BK % 8 == 0 && (BK / 4) % 2 == 0, "K steps per stage must be even");
};

// Output coordinates of accumulator element v of block (i, j) for this lane
// (V_MFMA_F64_16X16X4_F64: result element v of lane l is D[4 v + l / 16][l % 16]).
template <class C>
__device__ __forceinline__ int atom_row(int i, int v) {
    const int wave = threadIdx.x >> 6;
    return (wave / C::WN) * C::WTM + i * 16 + 4 * v + ((threadIdx.x & 63) >> 4);
}
template <class C>
__device__ __forceinline__ int atom_col(int j) {
    const int wave = threadIdx.x >> 6;
    return (wave % C::WN) * C::WTN + j * 16 + (threadIdx.x & 15);
}

// tr: segment 0's contribution is sum_k P_0[m][k] Q_0[k][n] (P_0 row-major
// with row stride ldp, not conjugated) instead of P_0^H Q_0.
template <class C>
__device__ __forceinline__ void ztile_atom(const Segs<2, false> &t, int m0, int mlim, int n0,
                                           int nlim, bool tr, Acc<C> &acc, double2 *lds) {
    static_assert(C::NT == 512, "8 waves");
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / C::WN;
    const int wn = wave % C::WN;

#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j) {
            acc.re[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
            acc.im[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
        }

    const int ktot = t.nseg * t.len;
    const int nst = (ktot + C::BK - 1) / C::BK;
    if (nst == 0) return;
    const int ntr = tr ? t.len : 0;   // transposed rows of P

    // per-lane byte offsets of the loaded columns (clamped at the edge);
    // pvt: of the loaded rows of a transposed P
    unsigned pvo[C::PH], pvt[C::PH], qvo[C::QH];
#pragma unroll
    for (int h = 0; h < C::PH; ++h) {
        const int c = m0 + 64 * h + lane;
        pvo[h] = (unsigned)(c < mlim ? c : mlim - 1) * 16u;
        pvt[h] = pvo[h] * (unsigned)t.ldp;
    }
#pragma unroll
    for (int h = 0; h < C::QH; ++h) {
        const int c = n0 + 64 * h + lane;
        qvo[h] = (unsigned)(c < nlim ? c : nlim - 1) * 16u;
    }
    auto at = [](const double2 *row, unsigned vo) __attribute__((always_inline)) {
        return reinterpret_cast<const double2 *>(reinterpret_cast<const char *>(row) + vo);
    };
    // rows w (and w + 8) of stage st into buf
    auto issue = [&](double2 *buf, int st) __attribute__((always_inline)) {
        double2 *lp = buf;
        double2 *lq = buf + C::BK * C::BMS;
#pragma unroll
        for (int k = 0; k < C::BK / 8; ++k) {
            const int r = wave + 8 * k;
            const int kk = st * C::BK + r;
            if (kk < ktot) {
                const int s = kk >= t.len ? 1 : 0;
                const long long row = kk - s * t.len;
                const bool gather = kk < ntr;
                const double2 *prow = pick<2>(t.P, s) + (gather ? row : row * t.ldp);
                const double2 *qrow = pick<2>(t.Q, s) + row * t.ldq;
#pragma unroll
                for (int h = 0; h < C::PH; ++h)
                    __builtin_amdgcn_global_load_lds(at(prow, gather ? pvt[h] : pvo[h]),
                                                     lp + r * C::BMS + 64 * h, 16, 0, 0);
#pragma unroll
                for (int h = 0; h < C::QH; ++h)
                    __builtin_amdgcn_global_load_lds(at(qrow, qvo[h]), lq + r * C::BNS + 64 * h, 16, 0, 0);
            } else {
#pragma unroll
                for (int h = 0; h < C::PH; ++h) lp[r * C::BMS + 64 * h + lane] = double2{0.0, 0.0};
#pragma unroll
                for (int h = 0; h < C::QH; ++h) lq[r * C::BNS + 64 * h + lane] = double2{0.0, 0.0};
            }
        }
    };

    const int lr = lane >> 4;   // contraction row within a K step of 4
    const int lc = lane & 15;   // column within a 16-wide block
    auto ldfrag = [&](const double2 *lp, const double2 *lq, int st, int k4, double2 (&a)[C::TM],
                      double2 (&b)[C::TN]) __attribute__((always_inline)) {
        const int kr = k4 * 4 + lr;
        // sign flip of the rows of a transposed P (its conjugate is stored)
        const long long flip = st * C::BK + kr < ntr ? (long long)(1ull << 63) : 0ll;
#pragma unroll
        for (int i = 0; i < C::TM; ++i) {
            a[i] = lp[kr * C::BMS + wm * C::WTM + i * 16 + lc];
            a[i].y = __longlong_as_double(__double_as_longlong(a[i].y) ^ flip);
        }
#pragma unroll
        for (int j = 0; j < C::TN; ++j) b[j] = lq[kr * C::BNS + wn * C::WTN + j * 16 + lc];
    };
    // the 4 TM TN real MFMAs of one K step, in four passes over the blocks so that
    // two MFMAs into one accumulator are 2 TM TN - 1 MFMAs apart
    auto mma = [&](const double2 (&a)[C::TM], const double2 (&b)[C::TN])
                   __attribute__((always_inline)) {
        double nbr[C::TN];
#pragma unroll
        for (int j = 0; j < C::TN; ++j) nbr[j] = -b[j].x;
#pragma unroll
        for (int i = 0; i < C::TM; ++i)
#pragma unroll
            for (int j = 0; j < C::TN; ++j)
                acc.re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].x, b[j].x, acc.re[i][j], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < C::TM; ++i)
#pragma unroll
            for (int j = 0; j < C::TN; ++j)
                acc.im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].x, b[j].y, acc.im[i][j], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < C::TM; ++i)
#pragma unroll
            for (int j = 0; j < C::TN; ++j)
                acc.re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].y, b[j].y, acc.re[i][j], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < C::TM; ++i)
#pragma unroll
            for (int j = 0; j < C::TN; ++j)
                acc.im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].y, nbr[j], acc.im[i][j], 0, 0, 0);
    };
    // one LDS fragment read, then a few MFMAs, for the next step's TM + TN
    // reads (1% faster than the scheduler's own order)
    auto interleave = [&]() __attribute__((always_inline)) {
        constexpr int NR = C::TM + C::TN;
        constexpr int NM = 4 * C::TM * C::TN;
        constexpr int PER = NM / (NR + 1);
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, PER, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, NM - NR * PER, 0);
    };
    auto compute = [&](const double2 *lp, const double2 *lq, int st) __attribute__((always_inline)) {
        // the last stage's second half holds no contraction rows: skip it
        const bool full = ktot - st * C::BK > C::BK / 2;
        double2 fa0[C::TM], fb0[C::TN], fa1[C::TM], fb1[C::TN];
        ldfrag(lp, lq, st, 0, fa0, fb0);
#pragma unroll
        for (int k4 = 0; k4 < C::BK / 4; k4 += 2) {
            if (k4 >= C::BK / 8 && !full) break;
            ldfrag(lp, lq, st, k4 + 1, fa1, fb1);
            mma(fa0, fb0);
            interleave();
            if (k4 + 2 < C::BK / 4) ldfrag(lp, lq, st, k4 + 2, fa0, fb0);
            mma(fa1, fb1);
            if (k4 + 2 < C::BK / 4) interleave();
        }
    };

    issue(lds, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    for (int s = 0; s < nst; ++s) {
        // the buffer being computed and the one being loaded are distinct:
        // saying so (restrict) keeps the compiler from waiting for the
        // direct loads before every LDS read of the stage
        auto stage = [&](const double2 *__restrict__ cur, double2 *__restrict__ nxt)
                         __attribute__((always_inline)) {
            if (s + 1 < nst) issue(nxt, s + 1);
            compute(cur, cur + C::BK * C::BMS, s);
        };
        stage(lds + (s & 1) * C::STAGE, lds + ((s + 1) & 1) * C::STAGE);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }
}

// Operands of atom a's X (which = 0) or Y (which = 1) product: r0, n, t0 its
// first row, N_L and first T element. X: T_AB B + M1^H A, the first segment
// transposed (ztile_atom's tr), T_AA A, the larger term, last: in the other
// order the smaller one's N_L roundings are at the size of the whole (mean error
// of H over small builds 1% to 8% larger). Y: T_AB^H A + M2^H B.
__device__ __forceinline__ Segs<2, false> atom_segs(int which, int n, int n_g, long long t0, int r0,
                                                    const double2 *A, const double2 *B,
                                                    const double2 *T_AB, const double2 *M1,
                                                    const double2 *M2) {
    Segs<2, false> t;
    t.nseg = 2;
    t.len = n;
    t.ldp = n;
    t.ldq = n_g;
    t.P[0] = T_AB + t0;
    t.P[1] = (which == 0 ? M1 : M2) + t0;
    t.Q[0] = (which == 0 ? B : A) + (long long)r0 * n_g;
    t.Q[1] = (which == 0 ? A : B) + (long long)r0 * n_g;
    t.qscale = nullptr;
    return t;
}

template <class C>
__device__ __forceinline__ void atom_store(const Acc<C> &acc, int m0, int n, int n0, int n_g,
                                           double2 *__restrict__ out) {
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j) {
            const int g = n0 + atom_col<C>(j);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int l = m0 + atom_row<C>(i, v);
                if (l < n && g < n_g)
                    out[(long long)l * n_g + g] = double2{acc.re[i][j][v], acc.im[i][j][v]};
            }
        }
}

}  // namespace hs
