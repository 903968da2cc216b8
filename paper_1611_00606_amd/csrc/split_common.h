// Device helpers shared by the split-precision reductions (k_split.hip) and
// the modular INT8 form (k_crt.hip): the sliced operands' values, column
// exponents, the (Re, Im) -> (Im, -Re) byte-pair form and the banded
// lower-triangle tile order.
#pragma once

#include "hs_internal.h"

namespace hs {

// v[z], formed arithmetically (a dynamic index into the argument block would
// copy it to scratch memory).
template <class T, int N>
__device__ __forceinline__ T *slice_ptr(T *const (&v)[N], int z) {
    const uintptr_t base = reinterpret_cast<uintptr_t>(v[0]);
    uintptr_t p = base;
#pragma unroll
    for (int i = 1; i < N; ++i) p += z == i ? reinterpret_cast<uintptr_t>(v[i]) - base : 0;
    return reinterpret_cast<T *>(p);
}

// Exponent e of row k: A's row times 2^e and X's times 2^-e have about equal
// maxima. Every operand is cut relative to its column's maximum over all rows,
// so an error of A^H X is that of the largest rows of A and of X against all
// rows of the other, and X carries the whole of T_AA: with T_AA = D T D, A =
// D^-1 A' (row magnitudes over a factor 1e4) the FP16 form's H was 2e-7 off
// unscaled, 3e-10 in Alg. 1's grouping, whose Cholesky factors share T_AA
// evenly between both operands, and 4e-10 with e. The upper half of a double is its
// logarithm in units of 2^-20, to 0.09; a zero row counts as 2^-1023.
__device__ __forceinline__ int slice_row_exp(const SliceJobs &jobs, int k) {
    const int g = jobs.rgroup == 1 ? k : k / jobs.rgroup;
    return ((int)jobs.rmx[1][g] - (int)jobs.rmx[0][g] + (1 << 20)) >> 21;
}

// How operand z is made from its matrix: as it is, with sqrt(rscale), with 2^-e
// or 2^e (scaled: *jobs.scaled, read once by the caller).
enum SliceForm { SLICE_RAW, SLICE_U, SLICE_DOWN, SLICE_UP };
__device__ __forceinline__ SliceForm slice_form(int z, bool scaled) {
    return z == 4 ? SLICE_U : !scaled ? SLICE_RAW : z == 2 ? SLICE_DOWN : z == 5 ? SLICE_UP : SLICE_RAW;
}
// Element v of row k in that form.
__device__ __forceinline__ double2 slice_value(const SliceJobs &jobs, SliceForm f, double2 v, int k) {
    if (f == SLICE_RAW) return v;
    if (f == SLICE_U) {
        const double w = sqrt(jobs.rscale[k]);
        return double2{v.x * w, v.y * w};
    }
    const int e = f == SLICE_UP ? slice_row_exp(jobs, k) : -slice_row_exp(jobs, k);
    return double2{ldexp(v.x, e), ldexp(v.y, e)};
}
// The operands made from matrix z: its values brought into a form in place, and
// cut, once or twice (X 2^-e; A and, if rows are scaled, A 2^e; B and U B). One
// copy of `cut` for all of them.
template <class Bring, class Cut>
__device__ __forceinline__ void slice_operands(const SliceJobs &jobs, int z, Bring bring, Cut cut) {
    const bool scaled = *jobs.scaled;
    const int other = z == 1 ? 4 : z == 0 && scaled ? 5 : -1;
    for (int op = z;; op = other) {
        const SliceForm form = slice_form(op, scaled);
        if (form != SLICE_RAW) bring(form);
        cut(op);
        if (op == other || other < 0) break;
    }
}

// Column scale of the sliced forms: the maximum itself, so that the first
// slice's range is used in full (with the next power of two the dropped pairs
// of slices weigh 1.4 times as much per operand, in the mean). At least
// 2^-1021, so that it has a reciprocal; an all-zero column takes any.
__device__ __forceinline__ double col_scale(const unsigned long long *mx, int n) {
    return fmax(__longlong_as_double((long long)mx[n]), 0x1p-1021);
}

// (Re, Im) int8 byte pairs -> (Im, -Re): conj(p) q's imaginary part as a dot
// product. The bytes must not hold -128.
__device__ __forceinline__ unsigned im_pairs(unsigned d) {
    typedef unsigned short us2 __attribute__((ext_vector_type(2)));
    const unsigned t = __builtin_amdgcn_perm(d, d, 0x02030001u) ^ 0xff00ff00u;
    us2 h = __builtin_bit_cast(us2, t);
    h += us2{0x0100, 0x0100};   // per 16-bit half: high byte ~b + 1 = -b, no carry across
    return __builtin_bit_cast(unsigned, h);
}

// Tile (i, j), j <= i, at position t of the banded order over an nt x nt
// lower triangle of tiles: bands of `band` tile columns, each band walked
// from its diagonal triangle down; (-1, -1) past the end.
__host__ __device__ __forceinline__ void sband_tile(int t, int nt, int &ti, int &tj, int band) {
    int c0 = 0;
    for (;;) {
        const int m = nt - c0;
        if (m <= 0) {
            ti = tj = -1;
            return;
        }
        const int w = m < band ? m : band;
        const int tri = w * (w + 1) / 2;
        const int cnt = tri + (m - w) * w;
        if (t < cnt) {
            if (t < tri) {
                int r = 0;
                while ((r + 1) * (r + 2) / 2 <= t) ++r;
                ti = c0 + r;
                tj = c0 + (t - r * (r + 1) / 2);
            } else {
                const int u = t - tri;
                ti = c0 + w + u / w;
                tj = c0 + u % w;
            }
            return;
        }
        t -= cnt;
        c0 += band;
    }
}

// Tiles of H and S over the lower triangle of nt x nt 64-tiles, H's first in
// banded order, then S's: the first `whole` as 64-tiles, the others as two
// 64 x 32 halves each.
struct SplitPlan {
    int nt, ntri, whole;
};
inline unsigned split_blocks(const SplitPlan &p) {
    return (unsigned)(xcd_blocks(p.whole) + 2 * (2 * p.ntri - p.whole));
}
// The split with the earliest end when a half takes `half` of a whole tile's
// time and the compute units take them in turn: all whole, whole rounds only,
// or none.
inline SplitPlan split_plan(int n_g, int cus, double half) {
    SplitPlan p;
    p.nt = (n_g + 63) / 64;
    p.ntri = p.nt * (p.nt + 1) / 2;
    const int all = 2 * p.ntri;
    double best = -1.0;
    for (int w : {all, all / cus * cus, 0}) {
        const double t = (w + cus - 1) / cus + (2 * (all - w) + cus - 1) / cus * half;
        if (best < 0.0 || t < best) {
            best = t;
            p.whole = w;
        }
    }
    return p;
}
// Tile of block b: (ti, tj), half 0 or 1 of its columns or -1 for all of them;
// ti < 0: none.
struct SplitPlace {
    bool isH;
    int ti, tj, half;
};
__host__ __device__ __forceinline__ SplitPlace split_place(const SplitPlan &p, int b, int band) {
    SplitPlace r;
    int t;
    r.half = -1;
    if (b < xcd_blocks(p.whole)) {
        t = xcd_item(b, p.whole, p.ntri);
        if (t < 0) {
            r.ti = -1;
            return r;
        }
    } else {
        b -= xcd_blocks(p.whole);
        t = p.whole + (b >> 1);
        r.half = b & 1;
    }
    r.isH = t < p.ntri;
    sband_tile(r.isH ? t : t - p.ntri, p.nt, r.ti, r.tj, band);
    return r;
}

}  // namespace hs
