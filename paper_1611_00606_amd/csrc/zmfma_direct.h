// Complex-double MFMA tile engine with direct global -> LDS operand loads,
// for the large reductions (k_reduce) and the eigenproblem reduction's
// products (k_gep). C = sum_s P_s^H Q_s over concatenated segments, 4 real
// V_MFMA_F64_16X16X4_F64 per complex step; the operand rows move from global
// memory straight into LDS with 16-byte loads (global_load_lds_dwordx4: lane
// l of a wave lands at base + 16 l), so no staging registers and no LDS-store
// instructions sit in the K loop.
//
// One stage is BK contraction rows of P (BM columns) and Q (BN columns, one
// row stride, ldp, for both), spread over all 8 waves' loads; NBUF stage buffers form a ring. A stage
// has one barrier, in its middle: before its last K step every wave waits
// for its own loads of the next stage (a counted wait: later stages stay in
// flight) and meets the others, then refills the buffer that every wave has
// finished with, then reads the next stage's first fragments beside the last
// K step's MFMAs. So no wave meets the barrier with nothing left to multiply
// and no stage starts with an LDS round trip.
//
// Rows past the end of the contraction (of the last stage, and of the stages
// the ring prefetches past it) load the last row, which keeps the number of
// loads in flight constant; their fragments are zeroed and their K steps
// skipped. Columns past the edge read the last column (they only feed outputs
// past the edge, which are not stored). The per-row scale of Q (SCALE) is
// applied to the Q fragment in registers, from scalar loads. The buffers reach the stage body as distinct (restrict) pointers,
// without which the compiler waits for every load before the LDS reads.
//
// G3: the complex product in 3 real products instead of 4 (the 3M or Gauss
// form): per contraction row, with p = pr + i pi and q = qr + i qi,
//   T1 += pr qr,   T2 += pi qi,   T3 += (pr - pi)(qr + qi)
// and at the end Re = T1 + T2, Im = T3 - T1 + T2, which is conj(p) q summed.
// T1 and T2 live in acc.re and acc.im until the final fold. The real part is
// the same sum as in the 4-product form; the imaginary part's rounding error
// is bounded by the unit roundoff times |pr - pi||qr + qi| + |pr||qr| +
// |pi||qi| (summed over the contraction) instead of |pr||qi| + |pi||qr|.
//
// Every tile shape adds the contraction rows to an output in the same order,
// so an output's bits do not depend on the shape that computed it.
#pragma once

#include "zmfma_tile.h"

namespace hs {

// BM x BN tile by WM x WN multiplying waves of 8; stages of BK rows in a
// ring of NBUF buffers.
template <int BM_, int BN_, int BK_, int WM_, int WN_, int NBUF_>
struct TileCfg {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_, NBUF = NBUF_;
    static constexpr int NT = 512;                     // threads per block
    static constexpr int WTM = BM / WM, WTN = BN / WN; // wave tile
    static constexpr int TM = WTM / 16, TN = WTN / 16; // 16x16 blocks per wave
    static constexpr int STAGE = BK * (BM + BN);       // complex elements per stage
    static constexpr int LDS_ELEMS = NBUF * STAGE;
    static constexpr int ROWS = BM >= 64 ? 1 : 64 / BM;    // rows per 64-lane load
    static constexpr int PH = BM >= 64 ? BM / 64 : 1;      // loads per row (or row group)
    static constexpr int QH = BN >= 64 ? BN / 64 : 1;
    static constexpr int RG = BK / ROWS / 8;               // row groups per wave
    static constexpr int LPW = RG * (PH + QH);             // loads per wave and stage
    static_assert(WM * WN <= 8, "8 waves");
    static_assert(BM % (16 * WM) == 0 && BN % (16 * WN) == 0, "wave tiling");
    static_assert(BK % (8 * ROWS) == 0, "every wave loads alike");
    static_assert((BM >= 64 && BN >= 64) || BM == BN, "a load takes whole rows of P and Q alike");
    static_assert(BK % 8 == 0 && NBUF >= 3, "an even number of K steps; a buffer to refill");
};

// Whether this wave multiplies (small tiles leave some waves loading only).
template <class C>
__device__ __forceinline__ bool wave_works() {
    return C::WM * C::WN == 8 || threadIdx.x < 64 * C::WM * C::WN;
}

struct No {
    static constexpr bool value = false;
};
struct Yes {
    static constexpr bool value = true;
};

template <class C, int NSEG, bool SCALE, bool G3 = false>
__device__ __forceinline__ void ztile_direct(const Segs<NSEG, SCALE> &t, int m0, int mlim,
                                             int n0, int nlim, Acc<C> &acc, double2 *lds) {
    constexpr int NK = C::BK / 4;   // K steps per stage
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % C::WM;
    const int wn = wave / C::WM;
    const bool works = C::WM * C::WN == 8 || wave < C::WM * C::WN;

#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j) {
            acc.re[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
            acc.im[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
        }
    v4d t3[G3 ? C::TM : 1][G3 ? C::TN : 1];
    if constexpr (G3) {
#pragma unroll
        for (int i = 0; i < C::TM; ++i)
#pragma unroll
            for (int j = 0; j < C::TN; ++j) t3[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
    }

    const int ktot = t.nseg * t.len;
    const int nst = (ktot + C::BK - 1) / C::BK;
    if (nst == 0) return;

    // per-lane byte offsets of the loaded columns (clamped at the edge)
    unsigned pvo[C::PH], qvo[C::QH];
#pragma unroll
    for (int h = 0; h < C::PH; ++h) {
        const int c = m0 + 64 * h + lane % (C::BM < 64 ? C::BM : 64);
        pvo[h] = (unsigned)(c < mlim ? c : mlim - 1) * 16u;
    }
#pragma unroll
    for (int h = 0; h < C::QH; ++h) {
        const int c = n0 + 64 * h + lane % (C::BN < 64 ? C::BN : 64);
        qvo[h] = (unsigned)(c < nlim ? c : nlim - 1) * 16u;
    }
    auto at = [](const double2 *row, unsigned vo) __attribute__((always_inline)) {
        return reinterpret_cast<const double2 *>(reinterpret_cast<const char *>(row) + vo);
    };
    // this wave's operand rows of stage st (rows past the end: the last one),
    // found half a stage before they are loaded
    const double2 *prow[C::RG], *qrow[C::RG];
    auto rows = [&](int st) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < C::RG; ++k) {
            int kk = st * C::BK + (wave + 8 * k) * C::ROWS + (C::ROWS > 1 ? lane / C::BM : 0);
            kk = kk < ktot ? kk : ktot - 1;
            int s = 0;
#pragma unroll
            for (int i = 1; i < NSEG; ++i) s += (i < t.nseg && kk >= i * t.len) ? 1 : 0;
            const long long off = (long long)(kk - s * t.len) * t.ldp;
            prow[k] = pick<NSEG>(t.P, s) + off;
            qrow[k] = pick<NSEG>(t.Q, s) + off;
        }
    };
    // their loads into buf
    auto issue = [&](double2 *buf) __attribute__((always_inline)) {
        double2 *lp = buf;
        double2 *lq = buf + C::BK * C::BM;
#pragma unroll
        for (int k = 0; k < C::RG; ++k) {
            const int r = (wave + 8 * k) * C::ROWS;
#pragma unroll
            for (int h = 0; h < C::PH; ++h)
                __builtin_amdgcn_global_load_lds(at(prow[k], pvo[h]), lp + r * C::BM + 64 * h, 16, 0, 0);
#pragma unroll
            for (int h = 0; h < C::QH; ++h)
                __builtin_amdgcn_global_load_lds(at(qrow[k], qvo[h]), lq + r * C::BN + 64 * h, 16, 0, 0);
        }
    };

    const int lr = lane >> 4;   // contraction row within a K step of 4
    const int lc = lane & 15;   // column within a 16-wide block
    // Q scales of the rows of stage st: wave-uniform values, read through the
    // scalar cache (a vector load of them would have to be waited for in line
    // with the operand loads), one per row
    typedef const __attribute__((address_space(4))) double cdouble;
    cdouble *qsc = (cdouble *)(uintptr_t)t.qscale;
    constexpr int NQ = SCALE ? C::BK : 1;
    auto load_scales = [&](auto mask, double (&dst)[NQ], int st) __attribute__((always_inline)) {
        if constexpr (SCALE) {
#pragma unroll
            for (int k = 0; k < C::BK; ++k) {
                const int kk = st * C::BK + k;
                dst[k] = qsc[!decltype(mask)::value || kk < ktot ? kk : ktot - 1];
            }
        }
    };

    // fragments of K step k4 of a stage; rows >= rem (the rows the stage
    // holds) read as zero (MASK)
    auto ldfrag = [&](auto mask, const double2 *buf, int k4, const double (&qs)[NQ], int rem,
                      double2 (&a)[C::TM], double2 (&b)[C::TN]) __attribute__((always_inline)) {
        const double2 *lp = buf;
        const double2 *lq = buf + C::BK * C::BM;
        const int kr = k4 * 4 + lr;
#pragma unroll
        for (int i = 0; i < C::TM; ++i) a[i] = lp[kr * C::BM + wm * C::WTM + i * 16 + lc];
#pragma unroll
        for (int j = 0; j < C::TN; ++j) {
            b[j] = lq[kr * C::BN + wn * C::WTN + j * 16 + lc];
            if constexpr (SCALE) {
                const double lo = lr & 1 ? qs[4 * k4 + 1] : qs[4 * k4];
                const double hi = lr & 1 ? qs[4 * k4 + 3] : qs[4 * k4 + 2];
                const double w = lr & 2 ? hi : lo;
                b[j].x *= w;
                b[j].y *= w;
            }
        }
        if constexpr (decltype(mask)::value) {
            const bool in = kr < rem;
#pragma unroll
            for (int i = 0; i < C::TM; ++i) {
                a[i].x = in ? a[i].x : 0.0;
                a[i].y = in ? a[i].y : 0.0;
            }
#pragma unroll
            for (int j = 0; j < C::TN; ++j) {
                b[j].x = in ? b[j].x : 0.0;
                b[j].y = in ? b[j].y : 0.0;
            }
        }
    };
    // 3M form: T1 and T2, then T3 from the sums formed before them
    auto sums = [&](const double2 (&a)[C::TM], const double2 (&b)[C::TN], double (&sa)[C::TM],
                    double (&sb)[C::TN]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < C::TM; ++i) sa[i] = a[i].x - a[i].y;
#pragma unroll
        for (int j = 0; j < C::TN; ++j) sb[j] = b[j].x + b[j].y;
    };
    auto mma12 = [&](const double2 (&a)[C::TM], const double2 (&b)[C::TN]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < C::TM; ++i)
#pragma unroll
            for (int j = 0; j < C::TN; ++j)
                acc.re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].x, b[j].x, acc.re[i][j], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < C::TM; ++i)
#pragma unroll
            for (int j = 0; j < C::TN; ++j)
                acc.im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].y, b[j].y, acc.im[i][j], 0, 0, 0);
    };
    auto mma3 = [&](const double (&sa)[C::TM], const double (&sb)[C::TN]) __attribute__((always_inline)) {
        if constexpr (G3) {
#pragma unroll
            for (int i = 0; i < C::TM; ++i)
#pragma unroll
                for (int j = 0; j < C::TN; ++j)
                    t3[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(sa[i], sb[j], t3[i][j], 0, 0, 0);
        }
    };
    auto mma = [&](const double2 (&a)[C::TM], const double2 (&b)[C::TN]) __attribute__((always_inline)) {
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
    // A few MFMAs, one LDS fragment read, a few MFMAs, ... and then NV operand
    // loads spread over the rest in the same way: no stretch of address
    // arithmetic that both waves of a SIMD would run through at the same time,
    // right after their barrier, with the matrix cores idle. NM: the MFMAs.
    auto interleave = [&](auto nv) __attribute__((always_inline)) {
        constexpr int NR = C::TM + C::TN, NV = decltype(nv)::value;
        constexpr int NM = (G3 ? 1 : 4) * C::TM * C::TN;
        constexpr int PER = NM / (NR + NV + 1) > 0 ? NM / (NR + NV + 1) : 1;
        if constexpr (NM >= NR + NV) {
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, PER, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, PER, 0);
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            }
            if constexpr (NM > PER * (NR + NV))
                __builtin_amdgcn_sched_group_barrier(0x008, NM - PER * (NR + NV), 0);
        } else {
            constexpr int OPS = (NR + NV + NM - 1) / NM;
#pragma unroll
            for (int i = 0; i < NM; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x120, OPS, 0);
            }
        }
    };
    struct NoLoads {
        enum { value = 0 };
    };
    struct StageLoads {
        enum { value = C::LPW };
    };

    double2 fa0[C::TM], fb0[C::TN], fa1[C::TM], fb1[C::TN];

    // Stage s: fa0, fb0 hold its first fragments on entry and the next stage's
    // on return; q, qn: the scales of the two stages. The fragments are
    // double-buffered, except in the 3M form, whose accumulators (192 of the
    // 256 registers of a wave at two waves per SIMD) leave room for one K
    // step's only: there the next ones are read when T1 and T2 are done with
    // them, beside the MFMAs of T3.
    auto stage = [&](auto mask, int s, const double (&q)[NQ], const double (&qn)[NQ])
                     __attribute__((always_inline)) {
        auto body = [&](const double2 *__restrict__ cur, const double2 *__restrict__ nxt,
                        double2 *__restrict__ refill) __attribute__((always_inline)) {
            const int rem = ktot - s * C::BK;
            auto on = [&](int k4) __attribute__((always_inline)) {
                return works && (!decltype(mask)::value || 4 * k4 < rem);
            };
            auto meet = [&]() __attribute__((always_inline)) {
                // this wave's loads of the next stage are done (those of the
                // NBUF - 3 stages after it may be in flight); past the barrier
                // everyone's are, and everyone has consumed the stage before
                // this one, whose buffer is refilled
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((C::NBUF - 3) * C::LPW)
                             : "memory");
                __builtin_amdgcn_sched_barrier(0);
            };
            rows(s + C::NBUF - 1);
            if constexpr (!G3) {
#pragma unroll
                for (int k4 = 0; k4 + 1 < NK; k4 += 2) {
                    if (on(k4)) {
                        ldfrag(mask, cur, k4 + 1, q, rem, fa1, fb1);
                        mma(fa0, fb0);
                        interleave(NoLoads{});
                    }
                    if (k4 + 2 < NK && on(k4 + 1)) {
                        ldfrag(mask, cur, k4 + 2, q, rem, fa0, fb0);
                        mma(fa1, fb1);
                        interleave(NoLoads{});
                    }
                }
                meet();
                if (works) ldfrag(mask, nxt, 0, qn, rem - C::BK, fa0, fb0);
                issue(refill);
                if (on(NK - 1)) {
                    mma(fa1, fb1);
                    interleave(StageLoads{});
                }
            } else {
#pragma unroll
                for (int k4 = 0; k4 < NK; ++k4) {
                    double sa[C::TM], sb[C::TN];
                    if (on(k4)) {
                        sums(fa0, fb0, sa, sb);
                        mma12(fa0, fb0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if (k4 + 1 < NK) {
                        if (on(k4 + 1)) ldfrag(mask, cur, k4 + 1, q, rem, fa0, fb0);
                        if (on(k4)) {
                            mma3(sa, sb);
                            interleave(NoLoads{});
                        }
                    } else {
                        meet();
                        if (works) ldfrag(mask, nxt, 0, qn, rem - C::BK, fa0, fb0);
                        issue(refill);
                        if (on(k4)) {
                            mma3(sa, sb);
                            interleave(StageLoads{});
                        }
                    }
                }
            }
        };
        body(lds + s % C::NBUF * C::STAGE, lds + (s + 1) % C::NBUF * C::STAGE,
             lds + (s + C::NBUF - 1) % C::NBUF * C::STAGE);
    };

    double qa[NQ], qb[NQ];   // scales of the even and of the odd stages
    load_scales(Yes{}, qa, 0);
#pragma unroll
    for (int s = 0; s < C::NBUF - 1; ++s) {
        rows(s);
        issue(lds + s * C::STAGE);
    }
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((C::NBUF - 2) * C::LPW) : "memory");
    if (works) ldfrag(Yes{}, lds, 0, qa, ktot, fa0, fb0);
    int s = 0;
    for (; (s + 3) * C::BK <= ktot; s += 2) {   // stages s, s + 1 and s + 2 are whole
        load_scales(No{}, qb, s + 1);
        stage(No{}, s, qa, qb);
        load_scales(No{}, qa, s + 2);
        stage(No{}, s + 1, qb, qa);
    }
    for (; s < nst; s += 2) {
        load_scales(Yes{}, qb, s + 1);
        stage(Yes{}, s, qa, qb);
        load_scales(Yes{}, qa, s + 2);
        if (s + 1 < nst) stage(Yes{}, s + 1, qb, qa);
    }
    // the ring's prefetches past the end land before the caller uses LDS again
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if constexpr (G3) {
#pragma unroll
        for (int i = 0; i < C::TM; ++i)
#pragma unroll
            for (int j = 0; j < C::TN; ++j) {
                const v4d t1 = acc.re[i][j], t2 = acc.im[i][j];
                acc.re[i][j] = t1 + t2;
                acc.im[i][j] = (t3[i][j] - t1) + t2;
            }
    }
}

}  // namespace hs
