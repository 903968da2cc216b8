// Reduction of the generalized eigenproblem H x = lambda S x (Sec. 1.1) to
// standard form, the step after the build:
//     S = L L^H  (L lower, positive real diagonal),   Ht = L^{-1} H L^{-H}.
//
// The O(N^3) work runs as products on the complex FP64 MFMA tile engine with
// direct global -> LDS loads (zmfma_direct.h):
//   factor, right-looking over panels of LB = 128 columns (lookahead on a
//   second stream):
//     k_gep_leaf                        Cholesky of the diagonal block and the
//                                       inverse M11 = L11^{-1} (one workgroup)
//     LH21 = M11 S21^H                  (= L21^H, the panel)
//     S22 -= L21 L21^H                  lower triangle, contraction over 128
//   invert, recursive over the blocks of a diagonal block of L (split at m):
//     M21 = -M22 (L21 M11)              M, its inverse
//   step, over diagonal blocks c of some hundred columns, R the rows below:
//     Ht_c,: = M E_c,:                  left of the block
//     E_R,: -= L_Rc Ht_c,:
//     W = M^H L_Rc^H, F = K_cR - K_cc W, E_Rc = F^H M^H
//     K_RR -= F^H W + W^H K_cR          lower triangle, mirrored
//     V = K_cc M^H, Ht_cc = M V         lower triangle
// with K = H at first; Ht's lower triangle is mirrored at the end.
//
// Work: N^3/6 complex multiply-adds for the factor, N^3/2 for the steps in the
// limit of small blocks: 16/3 N^3 real flops, the minimal count of the
// reduction (LAPACK's zpotrf + zhegst); with the products
// over one block 5.56 N^3 at N = 8000 and 6.06 N^3 at 2000. Through the inverse of all of L
// (Ht = M H M^H) it was 20/3 N^3 (8 N^3 below N = 2500) and nearly all of it
// waited for the end of the factorization: N = 2000 2.39 ms, now 2.05, 8000
// 56.9 and 51.5 ms. From 4 panels on, the first steps run on a third stream
// beside the factorization.
//
// Storage (all N x N row-major complex): L (output; working copy of S's
// lower triangle during the factorization), LH (panels L21^H, then V in the
// diagonal blocks), M and MH = M^H of the diagonal blocks (zero in their
// other triangles), E left of M's diagonal blocks, F right of MH's, W (S21^H,
// L21 M11 of the invert, W of the steps), K, Ht (output).
#include <algorithm>
#include <cstdint>
#include <mutex>
#include <set>
#include <string>
#include <vector>

#include "hs_internal.h"
#include "zmfma_direct.h"
#include "zmfma_tile.h"

namespace hs {

namespace {

// Tile shapes of the products: a launch takes the one whose tiles fill the
// device best (mm_shape). The factorization's panels and the products of a
// small matrix are a few dozen 128-tiles, each 70 us long at 128 contraction
// rows; in 64 or 32-tiles they spread over the whole device.
using Mm128 = TileCfg<128, 128, 8, 2, 4, 4>;
// The 32-tiles' ring takes 64 KiB, so that two blocks share a compute unit
// (N = 300 489 us with one, 453 with two); 64-tiles are faster alone with a
// ring of 16-row stages (N = 2000 3.22 against 3.45 ms).
using Mm64 = TileCfg<64, 64, 16, 2, 4, 4>;
using Mm32 = TileCfg<32, 32, 16, 2, 2, 4>;
constexpr int MM_THREADS = 512;

// Compute units that the steps beside the factorization may occupy: 7/8 below
// N = 2500, where it is a chain of small launches, 3/4 above, where its bulk
// updates need them (us, 3/4 and 7/8: N = 1500 1370 and 1366, 2000 2232 and
// 2118, 2300 2744 and 2667, 4000 8596 and 8877, 10000 96971 and 97750; 3M form
// 2000 2026 and 1972, 3700 6189 and 6490; 1/2: 2000 2456, 8000 63259).
inline int bg_cap(int N, int cus) { return N < 2500 ? cus * 7 / 8 : cus * 3 / 4; }

// product flags
constexpr int MM_PU = 1;      // P upper triangular: k <= row of C
constexpr int MM_QL = 2;      // Q lower triangular: k >= column of C
constexpr int MM_QU = 4;      // Q upper triangular: k <= column of C
constexpr int MM_LOWER = 8;   // only C's lower triangle (square region)
constexpr int MM_MASK = 16;   // only elements on or below the diagonal (any region)
constexpr int MM_PL = 32;     // P lower triangular: k >= row of C
// epilogue
constexpr int OP_STORE = 0, OP_NEG = 1, OP_SUB = 2;

// One product, or several independent ones on the same three matrices
// (the nodes of one level of the inverse's recursion) in one launch.
struct MmJob {
    int i0, i1, j0, j1;       // C rows (P columns), C columns (Q columns)
    int k0, k1;               // contraction rows of P and Q
    int ntr, ntc;             // tile rows / columns of the rectangle
    int start;                // first block of this job
};
// Nodes of one depth of a step's recursion: steps end at multiples of LB = 128 and
// hold at most 1024 columns (split_steps), 8 blocks, so 4. (The fall-back
// without auxiliary streams takes several launches for more.)
constexpr int MM_JOBS = 4;

struct MmArgs {
    const double2 *P, *Q;
    const double2 *P2, *Q2;   // second term, same rectangle and contraction range
    double2 *C;
    const double2 *S;         // OP_SUB: C = S - the product
    double2 *T;               // or null: C's elements with one index below w0 and one
    int w0;                   // not (w0 < 0: below the diagonal) also as T = C^H
    int N;                    // leading dimension of all
    int op;
    int flags;                // MM_*
    int tile;                 // 128, 64 or 32
    int njobs;
    int total;                // tiles over all jobs (blocks loop over them)
    MmJob job[MM_JOBS];
};

// The engine's one call for each shape (clang's host pass instantiates a
// specialization of it for one caller only).
template <class Cfg, int NSEG, bool G3>
__device__ __forceinline__ void mm_product(const Segs<NSEG, false> &t, int m0, int i1, int n0,
                                           int j1, Acc<Cfg> &acc, double2 *lds) {
    ztile_direct<Cfg, NSEG, false, G3>(t, m0, i1, n0, j1, acc, lds);
}

// C[i][j] (op)= sum_k conj(P[k][i]) Q[k][j] over each job's rectangle, in
// absolute indices; the triangular flags trim each tile's contraction range
// to the rows where both operands can be nonzero. G3: 3 real products per
// complex product (the 3M form of the tile engine). TR: args.T is written too
// (kernels of their own: in the ones that do not, the longer epilogue made
// N = 8000 0.4% slower).
template <class Cfg, int NSEG, bool G3, bool TR>
__device__ __forceinline__ void mm_tile(const MmArgs &args, int tile, double2 *lds) {
    const int N = args.N;
    int jb = 0;
#pragma unroll
    for (int t = 1; t < MM_JOBS; ++t)
        if (t < args.njobs && tile >= args.job[t].start) jb = t;
    const int flags = args.flags;
    const int bid = tile - args.job[jb].start;
    const int ntr = args.job[jb].ntr, ntc = args.job[jb].ntc;
    const int i0 = args.job[jb].i0, i1 = args.job[jb].i1;
    const int j0 = args.job[jb].j0, j1 = args.job[jb].j1;
    // Tiles whose contraction is longest go first (the triangular flags
    // make it depend on the tile row or column).
    int ti, tj;
    if (flags & MM_LOWER) {   // lower triangle, tj <= ti
        const bool byc = flags & MM_QU;   // contraction grows with tj: last columns first
        const int t = byc ? bid : ntr * (ntr + 1) / 2 - 1 - bid;
        int r = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
        while ((r + 1) * (r + 2) / 2 <= t) ++r;
        while (r * (r + 1) / 2 > t) --r;
        if (byc) {   // column ntr-1-r, its r+1 tiles from the diagonal down
            tj = ntr - 1 - r;
            ti = tj + (t - r * (r + 1) / 2);
        } else {     // reversed row-major
            ti = r;
            tj = t - r * (r + 1) / 2;
        }
    } else if (flags & MM_PU) {   // longest: last tile rows
        ti = ntr - 1 - bid / ntc;
        tj = bid % ntc;
    } else if (flags & MM_QU) {   // longest: last tile columns
        tj = ntc - 1 - bid / ntr;
        ti = bid % ntr;
    } else {                      // MM_QL: first tile columns; MM_PL: first rows of each
        tj = bid / ntr;
        ti = bid % ntr;
    }
    const int m0 = i0 + ti * Cfg::BM;
    const int n0 = j0 + tj * Cfg::BN;
    if (m0 >= i1 || n0 >= j1) return;
    int klo = args.job[jb].k0, khi = args.job[jb].k1;
    if (flags & MM_PU) khi = min(khi, m0 + Cfg::BM);
    if (flags & MM_QU) khi = min(khi, n0 + Cfg::BN);
    if (flags & MM_QL) klo = max(klo, n0);
    if (flags & MM_PL) klo = max(klo, m0);

    Segs<NSEG, false> t;
    t.nseg = NSEG;
    t.len = khi > klo ? khi - klo : 0;
    t.ldp = N;
    t.ldq = N;
    const long long k0 = (long long)(t.len ? klo : 0) * N;
    t.P[0] = args.P + k0;
    t.Q[0] = args.Q + k0;
    if constexpr (NSEG == 2) {
        t.P[1] = args.P2 + k0;
        t.Q[1] = args.Q2 + k0;
    }
    t.qscale = nullptr;
    Acc<Cfg> acc;
    mm_product<Cfg, NSEG, G3>(t, m0, i1, n0, j1, acc, lds);
    if (!wave_works<Cfg>()) return;

    const bool lower = flags & (MM_LOWER | MM_MASK);
    const int op = args.op;
    double2 *C = args.C;
#pragma unroll
    for (int i = 0; i < Cfg::TM; ++i)
#pragma unroll
        for (int j = 0; j < Cfg::TN; ++j) {
            const int g = n0 + acc_col<Cfg>(j);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gp = m0 + acc_row<Cfg>(i, v);
                if (gp < i1 && g < j1 && (!lower || g <= gp)) {
                    double2 *o = C + (long long)gp * N + g;
                    const double re = acc.re[i][j][v], im = acc.im[i][j][v];
                    if (op == OP_SUB) {
                        double2 r = args.S[(long long)gp * N + g];
                        r.x -= re;
                        r.y -= im;
                        *o = r;
                        if constexpr (TR) {
                            acc.re[i][j][v] = r.x;
                            acc.im[i][j][v] = r.y;
                        }
                    } else if (op == OP_NEG) {
                        *o = double2{-re, -im};
                    } else {
                        *o = double2{re, im};
                    }
                }
            }
        }
    if constexpr (TR) {   // of OP_STORE or OP_SUB
        double2 *T = args.T;
        const int w0 = args.w0;
#pragma unroll
        for (int i = 0; i < Cfg::TM; ++i)
#pragma unroll
            for (int j = 0; j < Cfg::TN; ++j) {
                const int g = n0 + acc_col<Cfg>(j);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int gp = m0 + acc_row<Cfg>(i, v);
                    if (gp < i1 && g < j1 && (w0 < 0 ? g < gp : (g < w0) != (gp < w0)))
                        T[(long long)g * N + gp] = double2{acc.re[i][j][v], -acc.im[i][j][v]};
                }
            }
    }
}

// Blocks loop over the tiles (a launch may have fewer blocks than tiles when
// it runs beside latency-critical work).
template <class Cfg, int NSEG, bool G3, bool TR>
__global__ void __launch_bounds__(MM_THREADS) k_gep_mm(const MmArgs args) {
    __shared__ double2 lds[Cfg::LDS_ELEMS];
    for (int tile = blockIdx.x; tile < args.total; tile += gridDim.x) {
        mm_tile<Cfg, NSEG, G3, TR>(args, tile, lds);
        __syncthreads();   // LDS is reused by the next tile
    }
}

template <class Cfg>
void mm_launch(const MmArgs &a, bool g3, unsigned grid, hipStream_t st) {
    const dim3 gd(grid), bd(MM_THREADS);
    if (a.P2 && g3)   // always with a transpose
        hipLaunchKernelGGL((k_gep_mm<Cfg, 2, true, true>), gd, bd, 0, st, a);
    else if (a.P2)
        hipLaunchKernelGGL((k_gep_mm<Cfg, 2, false, true>), gd, bd, 0, st, a);
    else if (a.T && g3)
        hipLaunchKernelGGL((k_gep_mm<Cfg, 1, true, true>), gd, bd, 0, st, a);
    else if (a.T)
        hipLaunchKernelGGL((k_gep_mm<Cfg, 1, false, true>), gd, bd, 0, st, a);
    else if (g3)
        hipLaunchKernelGGL((k_gep_mm<Cfg, 1, true, false>), gd, bd, 0, st, a);
    else
        hipLaunchKernelGGL((k_gep_mm<Cfg, 1, false, false>), gd, bd, 0, st, a);
}

// Leaf: Cholesky of the diagonal block [kb, kb + nb) (nb <= LB = 128) of the
// working matrix (lower triangle in L) and the inverse X of the factor, by one
// workgroup of 8 waves. The block, padded to 128 x 128 with the identity,
// sits in LDS as the 36 lower 16 x 16 tiles (rows XOR-swizzled, so that the
// MFMA fragment loads and the accumulator stores hit distinct banks).
// Per panel P of 16 columns, two phases with a barrier after each:
//   wave 0:    the diagonal tile's update with panel P - 1, then its Cholesky
//              and inverse (diag16), X_PP replacing the tile;
//   waves 1-7: the rest of the trailing update C_IJ -= L_I,P-1 L_J,P-1^H; row
//              P - 1 of the inverse, X_IJ = -X_II sum_{J<=K<I} L_IK X_KJ, held
//              in registers, and row P's sum as far as its terms are there;
//   all waves: L_IP = C_IP X_PP^H, one tile per wave; the row of the inverse
//              is stored (over L's row, which nothing reads any more).
// Outputs go to global memory from the registers that form them: the block of
// L, of M = X (lower) and of MH = X^H (upper). Bound: the chain of diagonal
// tiles (3.5 us each) and the matrix products of one compute unit (24 us). A
// pivot that is not > 0 (NaN included) records kb + j + 1 in *info unless an
// earlier block failed (the outputs are undefined then).
constexpr int LB = 128;
constexpr int LT = LB / 16;               // tiles per side
constexpr int LNT = LT * (LT + 1) / 2;    // lower tiles

__device__ __forceinline__ double2 *ltile(double2 *T, int I, int K) {
    return T + (I * (I + 1) / 2 + K) * 256;
}
__device__ __forceinline__ int lsw(int a, int b) { return a * 16 + (b ^ a); }

// value of v in lane `src` (wave-uniform src)
__device__ __forceinline__ double bcast(double v, int src) {
    const long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)u, src);
    const int hi = __builtin_amdgcn_readlane((int)(u >> 32), src);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

struct Cacc {
    v4d re, im;
};

__device__ __forceinline__ void acc_zero(Cacc &c) {
    c.re = v4d{0.0, 0.0, 0.0, 0.0};
    c.im = v4d{0.0, 0.0, 0.0, 0.0};
}

// c += A B^H for 16 x 16 tiles (c[i][j] += sum_k A[i][k] conj(B[j][k]))
__device__ __forceinline__ void mma_abh(Cacc &c, const double2 *A, const double2 *B, int lane) {
#pragma unroll
    for (int k0 = 0; k0 < 16; k0 += 4) {
        const double2 x = A[lsw(lane & 15, k0 + (lane >> 4))];
        const double2 y = B[lsw(lane & 15, k0 + (lane >> 4))];
        c.re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, y.x, c.re, 0, 0, 0);
        c.im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, y.x, c.im, 0, 0, 0);
        c.re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, y.y, c.re, 0, 0, 0);
        c.im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, -y.y, c.im, 0, 0, 0);
    }
}

// c += A B for 16 x 16 tiles
__device__ __forceinline__ void mma_ab(Cacc &c, const double2 *A, const double2 *B, int lane) {
#pragma unroll
    for (int k0 = 0; k0 < 16; k0 += 4) {
        const double2 x = A[lsw(lane & 15, k0 + (lane >> 4))];
        const double2 y = B[lsw(k0 + (lane >> 4), lane & 15)];
        c.re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, y.x, c.re, 0, 0, 0);
        c.im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, y.y, c.im, 0, 0, 0);
        c.re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, -y.y, c.re, 0, 0, 0);
        c.im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, y.x, c.im, 0, 0, 0);
    }
}

// Cholesky and inverse of a 16 x 16 Hermitian tile by one wave, four columns
// at a time: those four columns (and the four rows of the identity under
// elimination) are copied to all four 16-lane groups through LDS, factored
// with readlane broadcasts inside the four, and the rest of the tile takes
// them as one rank-4 update on the matrix cores. With lane l = r + 16 q the
// accumulator layout D[4 v + q][r] of G = S^T holds S[r][4 v + q], which is
// the A and B operand layout of a rank-4 update with columns 4 v .. 4 v + 3,
// so nothing is re-laid out. (One column at a time over all sixteen, with
// the inverse by substitution afterwards: 6 + 5 us instead of 3.5; the leaf
// 103 us, 60 now.) Every update is formed by itself and subtracted once:
// accumulated onto S and E its eight roundings per four columns at their size
// made the error of L for random pairs of N = 16 1.67e-16 instead of 0.99e-16
// (one column at a time 1.18e-16), and the leaf 58 us.
//   D    the tile (row-major, swizzled; lower triangle used); X on return
//   scr  128 complex values of LDS of this wave
//   fac  receives L[r][4 v + q] of step v as fac(v, value), zero above the
//        diagonal
// Returns 0 or the 1-based index of the first pivot that is not > 0. 1/sqrt
// of a pivot: the hardware estimate y (good to 2^-22 or better) refined by one
// third-order step, y (1 + e/2 + 3 e^2 / 8) with e = 1 - d y^2, which leaves
// 5/16 e^3; sqrt(d) = d / sqrt(d).
template <class Fac>
__device__ __forceinline__ int diag16(double2 *D, double2 *scr, int lane, Fac fac) {
    const int r = lane & 15, q = lane >> 4;
    Cacc g, e;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const double2 s = D[lsw(r, 4 * v + q)];
        g.re[v] = s.x;
        g.im[v] = s.y;
        e.re[v] = 4 * v + q == r ? 1.0 : 0.0;
        e.im[v] = 0.0;
    }
    int inf = 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        scr[lane] = double2{g.re[v], g.im[v]};
        double2 s[4], x[4], l[4];   // columns 4 v + p of S; rows 4 v + p of E, then of X
        double rc[4], lkx[4][4], lky[4][4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            s[p] = scr[r + 16 * p];
            asm volatile("" : "+v"(s[p].x), "+v"(s[p].y));   // read here, not under a branch
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int j = 4 * v + p;
            const double d = bcast(s[p].x, j);
            if (!(d > 0.0) && inf == 0) inf = j + 1;
            const double y = __builtin_amdgcn_rsq(d);
            const double t = d * y;
            const double er = fma(-fma(d, y, -t), y, fma(-t, y, 1.0));   // 1 - d y^2
            rc[p] = fma(y * er, fma(0.375, er, 0.5), y);
            l[p].x = s[p].x * rc[p];   // sqrt(d) in row j
            l[p].y = r == j ? 0.0 : s[p].y * rc[p];
#pragma unroll
            for (int k = p + 1; k < 4; ++k) {
                const double lx = bcast(l[p].x, 4 * v + k), ly = bcast(l[p].y, 4 * v + k);
                lkx[p][k] = lx;
                lky[p][k] = ly;
                // s_rk -= l_rj conj(l_kj)
                s[k].x -= fma(ly, l[p].y, lx * l[p].x);
                s[k].y -= fma(-ly, l[p].x, lx * l[p].y);
            }
        }
        // this lane's element of four values (selected by component: a select
        // between aggregates goes through scratch memory)
        const auto own = [&](double a0, double a1, double a2, double a3) {
            const double lo = q & 1 ? a1 : a0, hi = q & 1 ? a3 : a2;
            return q & 2 ? hi : lo;
        };
        const bool low = r >= 4 * v + q;
        const double lre = own(l[0].x, l[1].x, l[2].x, l[3].x);
        const double lim = own(l[0].y, l[1].y, l[2].y, l[3].y);
        const double2 lq = {low ? lre : 0.0, low ? lim : 0.0};
        if (v < 3) {   // G[i][j] -= conj(L[i][p]) L[j][p]
            Cacc t;
            acc_zero(t);
            t.re = __builtin_amdgcn_mfma_f64_16x16x4f64(lq.x, lq.x, t.re, 0, 0, 0);
            t.im = __builtin_amdgcn_mfma_f64_16x16x4f64(lq.x, lq.y, t.im, 0, 0, 0);
            t.re = __builtin_amdgcn_mfma_f64_16x16x4f64(lq.y, lq.y, t.re, 0, 0, 0);
            t.im = __builtin_amdgcn_mfma_f64_16x16x4f64(-lq.y, lq.x, t.im, 0, 0, 0);
#pragma unroll
            for (int u = v + 1; u < 4; ++u) {
                g.re[u] -= t.re[u];
                g.im[u] -= t.im[u];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // the rows of the identity beside that update
        fac(v, lq);
        scr[64 + lane] = double2{e.re[v], e.im[v]};
#pragma unroll
        for (int p = 0; p < 4; ++p) x[p] = scr[64 + r + 16 * p];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            x[p].x *= rc[p];
            x[p].y *= rc[p];
#pragma unroll
            for (int k = p + 1; k < 4; ++k) {   // row k of E -= l_kj (row j of X)
                x[k].x -= fma(-lky[p][k], x[p].y, lkx[p][k] * x[p].x);
                x[k].y -= fma(lky[p][k], x[p].x, lkx[p][k] * x[p].y);
            }
        }
        const double2 xq = {own(x[0].x, x[1].x, x[2].x, x[3].x), own(x[0].y, x[1].y, x[2].y, x[3].y)};
        D[lsw(4 * v + q, r)] = xq;
        if (v < 3) {   // E[i][c] -= L[i][p] X[p][c]
            Cacc t;
            acc_zero(t);
            t.re = __builtin_amdgcn_mfma_f64_16x16x4f64(lq.x, xq.x, t.re, 0, 0, 0);
            t.im = __builtin_amdgcn_mfma_f64_16x16x4f64(lq.x, xq.y, t.im, 0, 0, 0);
            t.re = __builtin_amdgcn_mfma_f64_16x16x4f64(-lq.y, xq.y, t.re, 0, 0, 0);
            t.im = __builtin_amdgcn_mfma_f64_16x16x4f64(lq.y, xq.x, t.im, 0, 0, 0);
#pragma unroll
            for (int u = v + 1; u < 4; ++u) {
                e.re[u] -= t.re[u];
                e.im[u] -= t.im[u];
            }
        }
    }
    return inf;
}

// lower-triangle tile t of an n x n tile grid -> (i, j), j <= i
__device__ __forceinline__ void tri_decode(int t, int &i, int &j) {
    i = 0;
    while ((i + 1) * (i + 2) / 2 <= t) ++i;
    j = t - i * (i + 1) / 2;
}

__global__ void __launch_bounds__(512)
k_gep_leaf(double2 *__restrict__ L, double2 *__restrict__ M, double2 *__restrict__ MH, int N,
           int kb, int nb, int *__restrict__ info) {
    __shared__ double2 T[LNT * 256 + 128];   // 146 KiB
    double2 *scr = T + LNT * 256;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, q = lane >> 4;
    const long long blk = (long long)kb * N + kb;   // the block's first element
    L += blk;
    M += blk;
    MH += blk;

    if (nb == LB) {
        // whole block: 16-byte direct loads, lane l of tile quarter h to slot
        // 64 h + l, which holds element (s / 16, (s % 16) ^ (s / 16)) of the tile
        for (int u = w; u < 4 * LNT; u += 8) {
            int I, K;
            tri_decode(u >> 2, I, K);
            const int sl = 64 * (u & 3) + lane, a = sl >> 4, c = (sl & 15) ^ a;
            __builtin_amdgcn_global_load_lds(L + (long long)(16 * I + a) * N + 16 * K + c, T + 64 * u,
                                             16, 0, 0);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    } else {
        for (int e = tid; e < LB * LB; e += 512) {
            const int i = e / LB, k = e % LB;
            double2 v = {i == k ? 1.0 : 0.0, 0.0};
            if (k <= i && i < nb) v = L[(long long)i * N + k];
            if (k <= i) ltile(T, i >> 4, k >> 4)[lsw(i & 15, k & 15)] = v;
        }
    }
    __syncthreads();

    // C_IJ -= L_IP L_JP^H for the t-th tile of the trailing triangle of panel
    // P, NT tiles at once (t, t + 7), so that their LDS reads overlap. The
    // product is summed by itself: added to C term by term its 32 roundings at
    // the size of C made the error of L at N = 128 4.0e-16 instead of 1.6e-16.
    const auto trail = [&](auto nt, int P, int t) {
        constexpr int NT = decltype(nt)::value;
        Cacc c[NT];
        double2 *C[NT], *A[NT], *B[NT];
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            int ti, tj;
            tri_decode(t + 7 * u, ti, tj);
            A[u] = ltile(T, P + 1 + ti, P);
            B[u] = ltile(T, P + 1 + tj, P);
            C[u] = ltile(T, P + 1 + ti, P + 1 + tj);
            acc_zero(c[u]);
        }
#pragma unroll
        for (int k0 = 0; k0 < 16; k0 += 4)
#pragma unroll
            for (int u = 0; u < NT; ++u) {
                const double2 x = A[u][lsw(r, k0 + q)], y = B[u][lsw(r, k0 + q)];
                c[u].re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, y.x, c[u].re, 0, 0, 0);
                c[u].im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, y.x, c[u].im, 0, 0, 0);
                c[u].re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, y.y, c[u].re, 0, 0, 0);
                c[u].im = __builtin_amdgcn_mfma_f64_16x16x4f64(-x.x, y.y, c[u].im, 0, 0, 0);
            }
#pragma unroll
        for (int u = 0; u < NT; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                double2 *o = C[u] + lsw(4 * v + q, r);
                const double2 x = *o;
                *o = double2{x.x - c[u].re[v], x.y - c[u].im[v]};
            }
    };
    struct One {
        enum { value = 1 };
    };
    struct Two {
        enum { value = 2 };
    };
    // o = -X_II c
    const auto scale_x = [&](int I, const Cacc &c, Cacc &o) {
        const double2 *X = ltile(T, I, I);
        acc_zero(o);
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {   // B fragment rows 4 s4 .. = accumulator element s4
            const double2 x = X[lsw(r, 4 * s4 + q)];
            const double br = c.re[s4], bi = c.im[s4];
            o.re = __builtin_amdgcn_mfma_f64_16x16x4f64(-x.x, br, o.re, 0, 0, 0);
            o.im = __builtin_amdgcn_mfma_f64_16x16x4f64(-x.x, bi, o.im, 0, 0, 0);
            o.re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, bi, o.re, 0, 0, 0);
            o.im = __builtin_amdgcn_mfma_f64_16x16x4f64(-x.y, br, o.im, 0, 0, 0);
        }
    };
    // element (i, k) of X, k <= i, to M and MH
    const auto put_x = [&](int i, int k, double2 x) {
        if (i < nb) {
            M[(long long)i * N + k] = x;
            MH[(long long)k * N + i] = double2{x.x, -x.y};
        }
    };
    const auto put_x_tile = [&](int I, int J, const Cacc &o) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            put_x(16 * I + 4 * v + q, 16 * J + r, double2{o.re[v], o.im[v]});
    };

    // Wave w's column J of the inverse, so that the longest and the shortest
    // sums share a SIMD (waves w and w + 4); wave 4 shares one with wave 0,
    // which has the chain of diagonal tiles and goes first.
    const int J = w == 0 ? LT : w < 4 ? w - 1 : w == 4 ? 6 : 10 - w;
    // trailing tiles are dealt in turns of 13, two for each wave but wave 4
    const int turn = w == 4 ? 6 : w > 4 ? 7 - w : 6 - w;
    if (w == 0) __builtin_amdgcn_s_setprio(3);
    int inf = 0;
    Cacc c;   // sum_{J<=K<=P-2} L_PK X_KJ, begun a step before row P is due
#pragma unroll
    for (int P = 0; P < LT; ++P) {
        Cacc o;   // this wave's tile of row P - 1 of the inverse
        const bool has = J < P - 1;
        if (w == 0) {
            if (P > 0) {
                trail(One{}, P - 1, 0);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
            double2 *D = ltile(T, P, P);
            const int f = diag16(D, scr, lane, [&](int v, double2 l) {
                const int i = 16 * P + r, k = 16 * P + 4 * v + q;
                if (k <= i && i < nb) L[(long long)i * N + k] = l;
            });
            if (f != 0 && inf == 0 && 16 * P + f <= nb) inf = 16 * P + f;
        } else if (P > 0) {
            if (has) {
                if (J == P - 2) acc_zero(c);
                mma_ab(c, ltile(T, P - 1, P - 2), ltile(T, P - 2, J), lane);
                scale_x(P - 1, c, o);
                acc_zero(c);
#pragma unroll 2
                for (int K = J; K <= P - 2; ++K) mma_ab(c, ltile(T, P, K), ltile(T, K, J), lane);
            }
            const int n = LT - P;
            for (int t = 1 + turn; t < n * (n + 1) / 2; t += 13) {
                if (w != 4 && t + 7 < n * (n + 1) / 2) trail(Two{}, P - 1, t);
                else trail(One{}, P - 1, t);
            }
        }
        __syncthreads();
        if (has) {
            double2 *C = ltile(T, P - 1, J);
#pragma unroll
            for (int v = 0; v < 4; ++v) C[lsw(4 * v + q, r)] = double2{o.re[v], o.im[v]};
            put_x_tile(P - 1, J, o);
        }
        if (w == 0) {   // X_PP
            const double2 *D = ltile(T, P, P);
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (r <= 4 * v + q) put_x(16 * P + 4 * v + q, 16 * P + r, D[lsw(4 * v + q, r)]);
        }
        const int I = P + 8 - w;   // waves 7, 6, ...: panel tiles P + 1, P + 2, ...
        if (I < LT) {
            double2 *C = ltile(T, I, P);
            Cacc c;
            acc_zero(c);
            mma_abh(c, C, ltile(T, P, P), lane);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = 16 * I + 4 * v + q;
                const double2 l = {c.re[v], c.im[v]};
                C[lsw(4 * v + q, r)] = l;
                if (i < nb) L[(long long)i * N + 16 * P + r] = l;
            }
        }
        __syncthreads();
    }
    if (tid == 0 && inf != 0 && *info == 0) *info = kb + inf;
    if (w > 0) {   // the inverse's last row
        if (J == LT - 2) acc_zero(c);
        mma_ab(c, ltile(T, LT - 1, LT - 2), ltile(T, LT - 2, J), lane);
        Cacc o;
        scale_x(LT - 1, c, o);
        put_x_tile(LT - 1, J, o);
    }
}

// L := lower(S) (upper triangle zero), M := 0, MH := 0, K := H, info := 0
__global__ void __launch_bounds__(256)
k_gep_init(const double2 *__restrict__ H, const double2 *__restrict__ S, double2 *__restrict__ L,
           double2 *__restrict__ M, double2 *__restrict__ MH, double2 *__restrict__ K, int N, int *__restrict__ info) {
    const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
    if (e >= (long long)N * N) return;
    if (e == 0) *info = 0;
    const int i = (int)(e / N), j = (int)(e % N);
    const double2 z = double2{0.0, 0.0};
    double2 sv = z;
    if (j <= i) sv = S[e];
    L[e] = sv;
    M[e] = z;
    MH[e] = z;
    if (K) K[e] = H[e];
}

// D[j][i] = conj(X[i][j]) for i in [i0, i1), j in [j0, j1) of each job
// (blockIdx.z), through 32 x 32 LDS tiles (blockIdx.y: source tile row,
// blockIdx.x: source tile column)
struct CtJobs {
    int r[MM_JOBS][4];   // i0, i1, j0, j1
};

__global__ void __launch_bounds__(256)
k_gep_conj_t(const double2 *__restrict__ X, double2 *__restrict__ D, int N, const CtJobs jobs) {
    __shared__ double2 tile[32][33];
    const int z = blockIdx.z;
    const int i0 = jobs.r[z][0], i1 = jobs.r[z][1], j0 = jobs.r[z][2], j1 = jobs.r[z][3];
    const int si = i0 + blockIdx.y * 32, sj = j0 + blockIdx.x * 32;
    if (si >= i1 || sj >= j1) return;   // the grid covers the largest job
    const int tx = threadIdx.x % 32, ty = threadIdx.x / 32;
    for (int r = ty; r < 32; r += 8) {
        const int gr = si + r, gc = sj + tx;
        if (gr < i1 && gc < j1) tile[r][tx] = X[(long long)gr * N + gc];
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
        const int dr = sj + r, dc = si + tx;   // D[dr][dc] = conj(X[dc][dr])
        if (dr < j1 && dc < i1) {
            double2 v = tile[tx][r];
            v.y = -v.y;
            D[(long long)dr * N + dc] = v;
        }
    }
}

struct Gep {
    double2 *L, *LH, *M, *MH, *W, *K;
    int N;
    int *info;
    hipStream_t st;
    int cap;   // most blocks per product launch (0: one per tile)
    bool g3;   // products in the 3M form
};

#define GEP_TRY(x)                              \
    do {                                        \
        hipError_t e_ = (x);                    \
        if (e_ != hipSuccess) return e_;        \
    } while (0)

struct Rect {
    int i0, i1, j0, j1, k0, k1;
};

// ---------------------------------------------------------------------------
// Schedule check (host only). With a recorder installed the orchestration
// below runs unchanged but issues nothing: every launch is logged with its
// stream and the rectangles of each matrix it reads and writes (per output
// tile, with the tile's trimmed contraction range), every event record and
// stream wait with its stream and event. sched_check then runs a
// vector-clock pass over the log: two launches on different streams that
// touch a common 128 x 128 cell of a matrix, one of them writing, must be
// ordered by a chain of stream order and event waits.
enum SchedBuf { SB_H, SB_S, SB_L, SB_HT, SB_LH, SB_M, SB_MH, SB_W, SB_K, SB_INFO, SB_COUNT };
const char *const kSchedBufName[SB_COUNT] = {"H", "S", "L", "Ht", "LH", "M", "MH", "W", "K", "info"};

struct SchedAcc {
    int buf, r0, r1, c0, c1;   // element rectangle [r0, r1) x [c0, c1)
    bool write;
};
struct SchedOp {
    int kind;          // 0 launch, 1 event record, 2 stream wait
    hipStream_t st;
    hipEvent_t ev;
    const char *name;
    std::vector<SchedAcc> acc;
};
struct Sched {
    std::vector<SchedOp> ops;
    const void *base[SB_COUNT] = {};
    int drop_tag = 0;            // waits with this tag are left out (a test hook)
    int fail_call = 0;           // the call that fails: launches and event calls, from 1
    int calls = 0;
    uintptr_t next_event = 1;
    // Whether the call at hand fails.
    bool fails() { return ++calls == fail_call; }
    int buf(const void *p) const {
        for (int i = 0; i < SB_COUNT; ++i)
            if (base[i] == p) return i;
        return -1;
    }
    SchedOp &launch(hipStream_t st, const char *name) {
        ops.push_back(SchedOp{0, st, nullptr, name, {}});
        return ops.back();
    }
    void add(SchedOp &op, const void *p, int r0, int r1, int c0, int c1, bool write) {
        const int b = buf(p);
        if (b >= 0 && r1 > r0 && c1 > c0) op.acc.push_back(SchedAcc{b, r0, r1, c0, c1, write});
    }
};
thread_local Sched *g_sched = nullptr;

hipError_t ev_create(hipEvent_t *e) {
    if (g_sched) {
        if (g_sched->fails()) return hipErrorUnknown;
        *e = reinterpret_cast<hipEvent_t>(g_sched->next_event++);
        return hipSuccess;
    }
    return hipEventCreateWithFlags(e, hipEventDisableTiming);
}
void ev_destroy(hipEvent_t e) {
    if (!g_sched && e) (void)hipEventDestroy(e);
}
hipError_t ev_record(hipEvent_t e, hipStream_t st) {
    if (g_sched) {
        if (g_sched->fails()) return hipErrorUnknown;
        g_sched->ops.push_back(SchedOp{1, st, e, "record", {}});
        return hipSuccess;
    }
    return hipEventRecord(e, st);
}
// Wait sites, by tag (hs_gep_check_schedule's drop argument).
enum WaitTag {
    WT_TRANSPOSE_AFTER_BLOCK = 1,   // first panel's S21^H after the preparation of L
    WT_PANEL_AFTER_TRANSPOSE = 2,   // first panel product after S21^H
    WT_BLOCK_AFTER_BULK = 3,        // next column blocks after the previous bulk update
    WT_AHEAD_AFTER_PANEL = 4,       // L21 and bulk update after the panel product
    WT_JOIN_AHEAD = 5,              // end of the factorization: lookahead stream
    WT_FORK = 7,                    // a step on the background stream after its last panel
    WT_FORK_AHEAD = 8,              // the same after the lookahead stream's reads of LH
    WT_END_AFTER_INVERSE = 9,       // first step after the factorization after the one before it
    WT_END_AFTER_BACKGROUND = 10,   // mirror after the background stream's products
    WT_JOIN_AFTER_ERROR = 11
};
hipError_t ev_wait(hipStream_t st, hipEvent_t e, int tag) {
    if (g_sched) {
        if (g_sched->fails()) return hipErrorUnknown;
        if (tag != g_sched->drop_tag) g_sched->ops.push_back(SchedOp{2, st, e, "wait", {}});
        return hipSuccess;
    }
    return hipStreamWaitEvent(st, e, 0);
}

// The vector-clock pass. Returns the number of unordered conflicting pairs
// of launches and describes the first few in `report`.
// `unjoined`: launches that the work after the call on stream `st` would not
// be ordered after.
int sched_check(const Sched &sc, int N, std::string &report, hipStream_t st = nullptr,
                int *unjoined = nullptr) {
    constexpr int CB = 128;
    const int nc = (N + CB - 1) / CB;
    std::vector<hipStream_t> streams;
    auto sid = [&](hipStream_t st) {
        for (size_t i = 0; i < streams.size(); ++i)
            if (streams[i] == st) return (int)i;
        streams.push_back(st);
        return (int)streams.size() - 1;
    };
    for (const SchedOp &op : sc.ops) sid(op.st);
    const int ns = (int)streams.size();
    std::vector<std::vector<int>> vc(ns, std::vector<int>(ns, 0));
    std::vector<std::pair<hipEvent_t, std::vector<int>>> evc;
    struct Last {
        int op = -1, st = 0, clk = 0;
    };
    struct CellState {
        Last w;
        std::vector<Last> r;   // latest read per stream since the last write
    };
    const size_t ncell = (size_t)SB_COUNT * nc * nc;
    std::vector<CellState> cells(ncell);
    std::vector<signed char> mark(ncell, -1);   // per launch: 0 read, 1 write
    std::vector<size_t> touched;
    std::set<std::pair<int, int>> races;
    std::vector<std::pair<int, int>> at;   // stream and clock of each launch
    for (int i = 0; i < (int)sc.ops.size(); ++i) {
        const SchedOp &op = sc.ops[i];
        const int s = sid(op.st);
        if (op.kind == 1) {
            bool found = false;
            for (auto &e : evc)
                if (e.first == op.ev) {
                    e.second = vc[s];
                    found = true;
                }
            if (!found) evc.push_back({op.ev, vc[s]});
            continue;
        }
        if (op.kind == 2) {
            for (auto &e : evc)
                if (e.first == op.ev)
                    for (int k = 0; k < ns; ++k) vc[s][k] = std::max(vc[s][k], e.second[k]);
            continue;
        }
        ++vc[s][s];
        const std::vector<int> &me = vc[s];
        at.push_back({s, me[s]});
        touched.clear();
        for (const SchedAcc &a : op.acc) {
            const int cr0 = a.buf == SB_INFO ? 0 : a.r0 / CB, cr1 = a.buf == SB_INFO ? 0 : (a.r1 - 1) / CB;
            const int cc0 = a.buf == SB_INFO ? 0 : a.c0 / CB, cc1 = a.buf == SB_INFO ? 0 : (a.c1 - 1) / CB;
            for (int r = cr0; r <= cr1; ++r)
                for (int c = cc0; c <= cc1; ++c) {
                    const size_t id = ((size_t)a.buf * nc + r) * nc + c;
                    if (mark[id] < 0) touched.push_back(id);
                    mark[id] = std::max<signed char>(mark[id], a.write ? 1 : 0);
                }
        }
        auto ordered = [&](const Last &l) { return l.st == s || me[l.st] >= l.clk; };
        auto race = [&](int other, size_t id) {
            if (races.count({other, i})) return;
            if (races.size() < 5) {
                const int b = (int)(id / ((size_t)nc * nc));
                const int r = (int)(id / nc % nc), c = (int)(id % nc);
                report += std::string(sc.ops[other].name) + " and " + op.name + " on " +
                          kSchedBufName[b] + " cell (" + std::to_string(r) + ", " +
                          std::to_string(c) + "); ";
            }
            races.insert({other, i});
        };
        for (size_t id : touched) {
            CellState &cs = cells[id];
            const bool w = mark[id] == 1;
            mark[id] = -1;
            if (cs.w.op >= 0 && !ordered(cs.w)) race(cs.w.op, id);
            if (w) {
                for (const Last &l : cs.r)
                    if (!ordered(l)) race(l.op, id);
                cs.r.clear();
                cs.w = Last{i, s, me[s]};
            } else {
                bool had = false;
                for (Last &l : cs.r)
                    if (l.st == s) {
                        l = Last{i, s, me[s]};
                        had = true;
                    }
                if (!had) cs.r.push_back(Last{i, s, me[s]});
            }
        }
    }
    if (unjoined) {
        const std::vector<int> &end = vc[sid(st)];
        *unjoined = 0;
        for (const auto &l : at) *unjoined += end[l.first] < l.second;
    }
    return (int)races.size();
}

// The footprint of one product launch, tile by tile as mm_tile trims it.
void sched_mm(const Gep &g, const MmArgs &a) {
    const int bt = a.tile;
    SchedOp &op = g_sched->launch(g.st, a.P2 ? "k_gep_mm<2>" : "k_gep_mm<1>");
    for (int jb = 0; jb < a.njobs; ++jb) {
        const MmJob &j = a.job[jb];
        const int flags = a.flags;
        for (int ti = 0; ti < j.ntr; ++ti)
            for (int tj = 0; tj < j.ntc; ++tj) {
                if ((flags & MM_LOWER) && tj > ti) continue;
                const int m0 = j.i0 + ti * bt, n0 = j.j0 + tj * bt;
                if (m0 >= j.i1 || n0 >= j.j1) continue;
                const int m1 = std::min(m0 + bt, j.i1), n1 = std::min(n0 + bt, j.j1);
                int klo = j.k0, khi = j.k1;
                if (flags & MM_PU) khi = std::min(khi, m0 + bt);
                if (flags & MM_QU) khi = std::min(khi, n0 + bt);
                if (flags & MM_QL) klo = std::max(klo, n0);
                if (flags & MM_PL) klo = std::max(klo, m0);
                g_sched->add(op, a.P, klo, khi, m0, m1, false);
                g_sched->add(op, a.Q, klo, khi, n0, n1, false);
                if (a.P2) {
                    g_sched->add(op, a.P2, klo, khi, m0, m1, false);
                    g_sched->add(op, a.Q2, klo, khi, n0, n1, false);
                }
                g_sched->add(op, a.C, m0, m1, n0, n1, true);
                if (a.op == OP_SUB) g_sched->add(op, a.S, m0, m1, n0, n1, false);
                if (a.T && a.w0 < 0) g_sched->add(op, a.T, n0, n1, m0, m1, true);
                if (a.T && a.w0 >= 0) {
                    g_sched->add(op, a.T, n0, std::min(n1, a.w0), std::max(m0, a.w0), m1, true);
                    g_sched->add(op, a.T, std::max(n0, a.w0), n1, m0, std::min(m1, a.w0), true);
                }
            }
    }
}

// Tiles of one rectangle.
long long mm_tiles(const Rect &r, int flags, int tile) {
    const long long ntr = (r.i1 - r.i0 + tile - 1) / tile, ntc = (r.j1 - r.j0 + tile - 1) / tile;
    return flags & MM_LOWER ? ntr * (ntr + 1) / 2 : ntr * ntc;
}

// The tile shape of a launch over n rectangles on cus compute units, by an
// estimate of its time: the longest tile, or the tiles in rounds at their
// average contraction (a half of the range for each triangular operand's
// trimming). A tile takes 8 us besides the contraction (first loads, stores)
// and 0.44, 0.13 or 0.041 us per contraction row (and term) for 128, 64 or 32
// (measured on a full device; a 128-tile alone 70 us for 128 rows); two
// blocks of 32-tiles on one compute unit take turns and hide each other's
// 8 us.
int mm_shape(const Rect *r, int flags, int n, int nseg, int cus) {
    constexpr int SHAPES[3] = {128, 64, 32};
    constexpr double PER_ROW[3] = {0.44, 0.13, 0.041};
    int best = 128;
    double tbest = -1.0;
    for (int s = 0; s < 3; ++s) {
        double longest = 0.0, rows = 0.0;
        long long tiles = 0;
        for (int t = 0; t < n; ++t) {
            const long long nt = mm_tiles(r[t], flags, SHAPES[s]);
            const double k = (double)(r[t].k1 - r[t].k0) * nseg;
            double avg = k;
            for (int f : {MM_PU | MM_PL, MM_QU | MM_QL})
                if (flags & f) avg *= 0.5;
            longest = std::max(longest, 8.0 + k * PER_ROW[s]);
            rows += nt * avg;
            tiles += nt;
        }
        const long long per = s < 2 || tiles <= cus ? 1 : 2;   // blocks that share a compute unit
        const double rounds = (double)((tiles + per * cus - 1) / (per * cus));
        const double est =
            std::max(longest, rounds * (8.0 + per * rows / tiles * PER_ROW[s]));
        if (tbest < 0.0 || est < tbest) {
            tbest = est;
            best = SHAPES[s];
        }
    }
    return best;
}

// Products over the rectangles r[0 .. n), up to MM_JOBS per launch; the blocks
// take the rectangles in the order given.
hipError_t mm_batch(const Gep &g, const double2 *P, const double2 *Q, double2 *C, const Rect *r,
                    int n, int flags, int op, const double2 *P2 = nullptr,
                    const double2 *Q2 = nullptr, double2 *T = nullptr, int w0 = 0,
                    const double2 *S = nullptr) {
    for (int b = 0; b < n; b += MM_JOBS) {
        MmArgs a = {};
        a.P = P;
        a.Q = Q;
        a.P2 = P2;
        a.Q2 = Q2;
        a.C = C;
        a.S = S ? S : C;
        a.T = T;
        a.w0 = w0;
        a.N = g.N;
        a.op = op;
        a.flags = flags;
        Rect rj[MM_JOBS];
        for (int t = b; t < n && t < b + MM_JOBS; ++t) {
            if (r[t].i1 <= r[t].i0 || r[t].j1 <= r[t].j0) continue;
            rj[a.njobs++] = r[t];
        }
        if (a.njobs == 0) continue;
        const int cus = g.cap > 0 ? g.cap : g_sched ? 256 : num_cus();
        a.tile = mm_shape(rj, flags, a.njobs, P2 ? 2 : 1, cus);
        long long nblk = 0;
        for (int t = 0; t < a.njobs; ++t) {
            MmJob &j = a.job[t];
            j.i0 = rj[t].i0;
            j.i1 = rj[t].i1;
            j.j0 = rj[t].j0;
            j.j1 = rj[t].j1;
            j.k0 = rj[t].k0;
            j.k1 = rj[t].k1;
            j.ntr = (j.i1 - j.i0 + a.tile - 1) / a.tile;
            j.ntc = (j.j1 - j.j0 + a.tile - 1) / a.tile;
            j.start = (int)nblk;
            if ((flags & MM_LOWER) && (j.i0 != j.j0 || j.i1 != j.j1)) return hipErrorInvalidValue;
            nblk += mm_tiles(rj[t], flags, a.tile);
        }
        a.total = (int)nblk;
        if (g_sched) {
            if (g_sched->fails()) return hipErrorUnknown;
            sched_mm(g, a);
            continue;
        }
        const unsigned grid = (unsigned)(g.cap > 0 && nblk > g.cap ? g.cap : nblk);
        if (a.tile == 128) mm_launch<Mm128>(a, g.g3, grid, g.st);
        else if (a.tile == 64) mm_launch<Mm64>(a, g.g3, grid, g.st);
        else mm_launch<Mm32>(a, g.g3, grid, g.st);
        GEP_TRY(hipGetLastError());
    }
    return hipSuccess;
}

hipError_t mm(const Gep &g, const double2 *P, const double2 *Q, double2 *C, int i0, int i1,
              int j0, int j1, int k0, int k1, int flags, int op, double2 *T = nullptr,
              int w0 = 0) {
    const Rect r = {i0, i1, j0, j1, k0, k1};
    return mm_batch(g, P, Q, C, &r, 1, flags, op, nullptr, nullptr, T, w0);
}

// Transposes of the rectangles r[0 .. n), up to MM_JOBS per launch.
hipError_t conj_t_batch(const Gep &g, const double2 *X, double2 *D, const Rect *r, int n) {
    for (int b = 0; b < n; b += MM_JOBS) {
        CtJobs j = {};
        int nj = 0, gx = 0, gy = 0;
        for (int t = b; t < n && t < b + MM_JOBS; ++t) {
            if (r[t].i1 <= r[t].i0 || r[t].j1 <= r[t].j0) continue;
            j.r[nj][0] = r[t].i0;
            j.r[nj][1] = r[t].i1;
            j.r[nj][2] = r[t].j0;
            j.r[nj][3] = r[t].j1;
            gx = std::max(gx, (r[t].j1 - r[t].j0 + 31) / 32);
            gy = std::max(gy, (r[t].i1 - r[t].i0 + 31) / 32);
            ++nj;
        }
        if (nj == 0) continue;
        if (g_sched) {
            if (g_sched->fails()) return hipErrorUnknown;
            SchedOp &op = g_sched->launch(g.st, "k_gep_conj_t");
            for (int t = 0; t < nj; ++t) {
                g_sched->add(op, X, j.r[t][0], j.r[t][1], j.r[t][2], j.r[t][3], false);
                g_sched->add(op, D, j.r[t][2], j.r[t][3], j.r[t][0], j.r[t][1], true);
            }
            continue;
        }
        hipLaunchKernelGGL(k_gep_conj_t, dim3(gx, gy, nj), dim3(256), 0, g.st, X, D, g.N, j);
        GEP_TRY(hipGetLastError());
    }
    return hipSuccess;
}

hipError_t conj_t(const Gep &g, const double2 *X, double2 *D, int i0, int i1, int j0, int j1) {
    const Rect r = {i0, i1, j0, j1, 0, 0};
    return conj_t_batch(g, X, D, &r, 1);
}

// Auxiliary streams per device (0: the factorization's lookahead, 1: work
// moved off the critical path, 2: the panels' transposes; with the caller's
// stream that is one hardware queue each at the default of four per
// process); default priority,
// created once and kept for the life of the process.
constexpr int AUX_STREAMS = 3;
hipStream_t aux_stream(int which) {
    if (g_sched) return reinterpret_cast<hipStream_t>((uintptr_t)(0x100 + which));
    static std::mutex mu;
    static hipStream_t cached[64][AUX_STREAMS] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    std::lock_guard<std::mutex> lk(mu);
    if (!cached[dev][which]) {
        hipStream_t s = nullptr;
        if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) return nullptr;
        cached[dev][which] = s;
    }
    return cached[dev][which];
}

// After a failed call: everything enqueued so far on the auxiliary streams
// before later work on st (a call that failed between a launch there and its
// event leaves it unordered). A stream that cannot be joined with an event is
// waited for.
void join_after_error(hipStream_t st) {
    for (int which = 0; which < AUX_STREAMS; ++which) {
        const hipStream_t s = aux_stream(which);
        hipEvent_t e = nullptr;
        if (!s) continue;
        if (ev_create(&e) != hipSuccess || ev_record(e, s) != hipSuccess ||
            ev_wait(st, e, WT_JOIN_AFTER_ERROR) != hipSuccess) {
            if (!g_sched) (void)hipStreamSynchronize(s);
        }
        ev_destroy(e);
    }
}

// Cholesky, right-looking over panels of LB columns: factor and invert the
// diagonal block, then the panel L21 = S21 L11^{-H} (as LH21 = M11 S21^H) and
// the update of the trailing lower triangle S22 -= L21 L21^H, whose epilogue
// also writes the next panel's S21^H. A panel is a chain of one workgroup and
// two small products, so what stands between them counts: an event record
// between two kernels of a stream takes 6 us, next to none 1 us (with S21^H
// and L21 as transposes of their own behind events on each panel, N = 300 316
// us and N = 2000 2.50 ms).
// Lookahead (from 4 panels on), with three streams and panels in pairs:
//   caller's    leaf, panel product; after the first panel of a pair the
//               update of the next column block with it, after the second
//               the update of the next two column blocks with both panels
//               (contraction 2 LB);
//   lookahead   after the second panel of a pair its L21 = LH21^H (an output
//               only; it gives the caller's update a start on the bulk, which
//               would take its compute units: N = 4000 9.15 ms, 9.4 without),
//               the bulk of the update with both panels (contraction 2 LB),
//               beside the next two leaves and panels, and the first's L21;
//   transposes  the first panel's S21^H, beside the first leaf.
// The update of the two column blocks after a pair waits for the previous
// pair's bulk update (both write those blocks); the bulk update and L21
// wait for the panels they use.
template <class Hook>
hipError_t factor(const Gep &g, Hook after_panel) {
    const int N = g.N;
    const int np = (N + LB - 1) / LB;
    Gep ga = g, gc = g;
    hipEvent_t e_panel = nullptr, e_bulk = nullptr, e_look = nullptr, e_next = nullptr,
               e_w = nullptr;
    bool ahead = np >= 4;
    if (ahead) {
        ga.st = aux_stream(0);
        gc.st = aux_stream(2);
        ahead = ga.st != nullptr && gc.st != nullptr && ev_create(&e_panel) == hipSuccess &&
                ev_create(&e_bulk) == hipSuccess && ev_create(&e_look) == hipSuccess &&
                ev_create(&e_next) == hipSuccess && ev_create(&e_w) == hipSuccess;
    }
    // recorded events still to be waited for (no wait on an unrecorded event);
    // e_bulk: the last bulk update, e_look: everything on the lookahead stream
    bool bulk_pending = false, look_pending = false, w_pending = false;
    hipError_t err = hipSuccess;
    // S21^H of the first panel
    const auto first_s21h = [&]() -> hipError_t {
        if (!ahead) return conj_t(g, g.L, g.W, LB, N, 0, LB);
        GEP_TRY(ev_record(e_next, g.st));
        GEP_TRY(ev_wait(gc.st, e_next, WT_TRANSPOSE_AFTER_BLOCK));
        GEP_TRY(conj_t(gc, g.L, g.W, LB, N, 0, LB));
        GEP_TRY(ev_record(e_w, gc.st));
        w_pending = true;
        return hipSuccess;
    };
    if (np > 1) err = first_s21h();
    for (int kb = 0; kb < N && err == hipSuccess; kb += LB) {
        const int nb = N - kb < LB ? N - kb : LB;
        const int t0 = kb + nb;
        if (g_sched && g_sched->fails()) {
            err = hipErrorUnknown;
        } else if (g_sched) {
            SchedOp &op = g_sched->launch(g.st, "k_gep_leaf");
            for (const double2 *X : {(const double2 *)g.L, (const double2 *)g.M,
                                     (const double2 *)g.MH})
                g_sched->add(op, X, kb, kb + nb, kb, kb + nb, true);
            g_sched->add(op, g.info, 0, 1, 0, 1, true);
        } else {
            hipLaunchKernelGGL(k_gep_leaf, dim3(1), dim3(512), 0, g.st, g.L, g.M, g.MH, N, kb, nb,
                               g.info);
            err = hipGetLastError();
        }
        if (err != hipSuccess || t0 >= N) break;
        const int t1 = N - t0 < LB ? N : t0 + LB;   // the next column block
        if (!ahead) {
            if ((err = mm(g, g.MH, g.W, g.LH, kb, t0, t0, N, kb, t0, MM_PU, OP_STORE, g.L, t0)) !=
                hipSuccess)
                break;                                                // LH21 = M11 S21^H, L21
            Rect none = {};
            if ((err = after_panel(t0, nullptr, none)) != hipSuccess) break;
            err = mm(g, g.LH, g.LH, g.L, t0, N, t0, N, kb, t0, MM_LOWER, OP_SUB, g.W,
                     t1);                                             // S22 -= L21 L21^H, next S21^H
            continue;
        }
        if (w_pending) {
            if ((err = ev_wait(g.st, e_w, WT_PANEL_AFTER_TRANSPOSE)) != hipSuccess) break;
            w_pending = false;
        }
        if ((err = mm(g, g.MH, g.W, g.LH, kb, t0, t0, N, kb, t0, MM_PU, OP_STORE)) != hipSuccess)
            break;                                                    // LH21 = M11 S21^H
        const bool second = ((kb / LB) & 1) != 0;    // second panel of a pair
        const int k0 = second ? kb - LB : kb;        // first contraction row of the update
        const int u1 = second ? std::min(N, t0 + 2 * LB) : t1;   // columns the caller updates
        // the first panel's L21 of a pair is still to come: the hook also gets
        // its rectangle, and empties it when it takes that on itself, and the
        // latest L21's event (or null), which orders the lookahead stream's
        // reads of LH before anything that the hook forks
        Rect first = {kb - LB, second ? kb : kb - LB, kb, N, 0, 0};
        if ((err = after_panel(t0, look_pending ? e_look : nullptr, first)) != hipSuccess) break;
        if (second || t1 == N) {   // L21 of the pair, or of a first panel that stays alone
            if ((err = ev_record(e_panel, g.st)) != hipSuccess) break;
            if ((err = ev_wait(ga.st, e_panel, WT_AHEAD_AFTER_PANEL)) != hipSuccess) break;
            if ((err = conj_t(ga, g.LH, g.L, kb, t0, t0, N)) != hipSuccess) break;
            if (second) {
                if (bulk_pending &&
                    (err = ev_wait(g.st, e_bulk, WT_BLOCK_AFTER_BULK)) != hipSuccess)
                    break;
                if (u1 < N && (err = mm(ga, g.LH, g.LH, g.L, u1, N, u1, N, k0, t0, MM_LOWER,
                                        OP_SUB)) != hipSuccess)
                    break;                                            // the rest
                if ((err = ev_record(e_bulk, ga.st)) != hipSuccess) break;
                bulk_pending = true;
                if ((err = conj_t_batch(ga, g.LH, g.L, &first, 1)) != hipSuccess) break;
            }
            if ((err = ev_record(e_look, ga.st)) != hipSuccess) break;
            look_pending = true;
        }
        err = mm(g, g.LH, g.LH, g.L, t0, N, t0, u1, k0, t0, MM_MASK, OP_SUB, g.W,
                 t1);                                  // next column block(s), next S21^H
    }
    // join the other streams
    if (err == hipSuccess && look_pending) err = ev_wait(g.st, e_look, WT_JOIN_AHEAD);
    for (hipEvent_t e : {e_panel, e_bulk, e_look, e_next, e_w}) ev_destroy(e);
    return err;
}

// Inverse of the factor, M = L^{-1}, over the recursion tree of [0, N) split
// at multiples of LB (the leaves' inverses are in place): per node [a, b)
// split at m, M21 = -M22 (L21 M11) and MH12 = M21^H. The nodes of one depth
// are independent; each depth, deepest first, runs as two batched launches.
struct Node {
    int a, m, b;
};

void tree(int a, int b, int depth, std::vector<std::vector<Node>> &lv) {
    const int n = b - a;
    if (n <= LB) return;
    const int m = a + (n / 2 + LB - 1) / LB * LB;   // multiple of LB, < b
    if ((int)lv.size() <= depth) lv.resize(depth + 1);
    lv[depth].push_back(Node{a, m, b});
    tree(a, m, depth + 1, lv);
    tree(m, b, depth + 1, lv);
}

// The two products and the transpose of a set of independent nodes.
hipError_t node_w21(const Gep &g, const std::vector<Node> &nodes) {   // W21 = L21 M11
    std::vector<Rect> r;
    for (const Node &n : nodes) r.push_back(Rect{n.m, n.b, n.a, n.m, n.a, n.m});
    return mm_batch(g, g.LH, g.M, g.W, r.data(), (int)r.size(), MM_QL, OP_STORE);
}
hipError_t node_m21(const Gep &g, const std::vector<Node> &nodes) {   // M21 = -M22 W21, MH12
    std::vector<Rect> r;
    for (const Node &n : nodes) r.push_back(Rect{n.m, n.b, n.a, n.m, n.m, n.b});
    GEP_TRY(mm_batch(g, g.MH, g.W, g.M, r.data(), (int)r.size(), MM_PU, OP_NEG));
    r.clear();
    for (const Node &n : nodes) r.push_back(Rect{n.m, n.b, n.a, n.m, 0, 0});
    return conj_t_batch(g, g.M, g.MH, r.data(), (int)r.size());
}

hipError_t invert(const Gep &g, const std::vector<std::vector<Node>> &lv) {
    for (int d = (int)lv.size() - 1; d >= 0; --d) {
        GEP_TRY(node_w21(g, lv[d]));
        GEP_TRY(node_m21(g, lv[d]));
    }
    return hipSuccess;
}

// Columns whose steps run beside the factorization: as many as it leaves time
// for. Up to N = 2000 it is a chain of small launches that leaves the device
// nearly empty, from 4000 on its bulk updates fill half of it. Measured best
// (us, with half as many and with half as many again): N = 1500 1024 (1361;
// 1580, -), 2000 1152 (2205; 2550, 2370), 4000 1280 (8660; -, 9255), 8000 2560
// (51955; 54140, 53900), 10000 3584 (94693; 99990, 100100).
int bg_columns(int N) {
    const double c = std::max(std::min(0.68 * N, 1280.0), 0.32 * N);
    return (int)(c / LB + 0.5) * LB;
}
// [a, b) in equal steps of at most about `most` columns, multiples of LB but
// the last: larger ones leave the invert of the step's block and its products
// under-filled longer, smaller ones contract over fewer rows (N = 2000 in
// steps of 512 2.22 ms, 640 2.23, 1280 2.43; N = 10000 640 > 99.8, 896 94.7,
// 1536 98.7).
void split_steps(int a, int b, int most, std::vector<int> &ends) {
    const int n = (b - a + most - 1) / most;
    for (int k = 1; k <= n; ++k)
        ends.push_back(k == n ? b : a + (int)((long long)(b - a) * k / n + LB / 2) / LB * LB);
}

// Column ends of all steps; nbg: how many run beside the factorization (0: one
// block, which needs no steps).
std::vector<int> step_ends(int N, size_t *nbg) {
    std::vector<int> ends;
    *nbg = 0;
    if (N <= 3 * LB) return {N};
    const int bg = bg_columns(N);
    split_steps(0, bg, 896, ends);
    *nbg = ends.size();
    split_steps(bg, N, 960, ends);
    return ends;
}

size_t padded(size_t bytes) { return (bytes + 255) / 256 * 256; }

// A diagonal block [a, b) of Ht = M K M^H, through V = K MH (kept in LH).
hipError_t diag_block(const Gep &g, const double2 *K, double2 *Ht, int a, int b) {
    GEP_TRY(mm(g, K, g.MH, g.LH, a, b, a, b, a, b, MM_QU, OP_STORE));
    return mm(g, g.LH, g.MH, Ht, a, b, a, b, a, b, MM_QU | MM_LOWER, OP_STORE);
}

// One step of the blocked transformation: rows and columns c = [a, b) of Ht
// left of and in the diagonal block, and what the rest R = [b, N) needs of
// them. On entry K (in full) and E (in M, left of the diagonal blocks) hold
// what the blocks before left. With M the inverse of L_cc:
//   Ht[c, :a) = M E[c, :a),   E[R, :a) -= L_Rc Ht[c, :a)
//   W = M^H L_Rc^H,   F = K_cR - K_cc W   (F in MH, right of the diagonal block)
//   E[R, c) = F^H M^H,   K_RR -= F^H W + W^H K_cR
//   Ht_cc = M K_cc M^H
// which is the congruence that eliminates L_Rc from both sides.
template <class Ready>
hipError_t step(const Gep &g, double2 *Ht, int a, int b, Ready ready) {
    const int N = g.N;
    std::vector<std::vector<Node>> lv;
    tree(a, b, 0, lv);
    GEP_TRY(invert(g, lv));
    GEP_TRY(ready());
    GEP_TRY(mm(g, g.MH, g.M, Ht, a, b, 0, a, a, b, MM_PU, OP_STORE));
    GEP_TRY(mm(g, g.LH, Ht, g.M, b, N, 0, a, a, b, 0, OP_SUB));
    GEP_TRY(mm(g, g.M, g.LH, g.W, a, b, b, N, a, b, MM_PL, OP_STORE));
    const Rect f = {a, b, b, N, a, b}, k = {b, N, b, N, a, b};
    GEP_TRY(mm_batch(g, g.K, g.W, g.MH, &f, 1, 0, OP_SUB, nullptr, nullptr, nullptr, 0, g.K));
    GEP_TRY(mm(g, g.MH, g.MH, g.M, b, N, a, b, a, b, MM_QU, OP_STORE));
    return mm_batch(g, g.MH, g.W, g.K, &k, 1, MM_LOWER, OP_SUB, g.W, g.K, g.K, -1);
}

hipError_t enqueue_gep(const double2 *H, const double2 *S, int N, double2 *L, double2 *Ht,
                       int *info, char *ws, hipStream_t st, bool g3) {
    const size_t m = padded(16 * (size_t)N * (size_t)N);
    Gep g;
    g.L = L;
    g.LH = reinterpret_cast<double2 *>(ws);
    g.M = reinterpret_cast<double2 *>(ws + m);
    g.MH = reinterpret_cast<double2 *>(ws + 2 * m);
    g.W = reinterpret_cast<double2 *>(ws + 3 * m);
    g.K = reinterpret_cast<double2 *>(ws + 4 * m);
    g.N = N;
    g.info = info ? info : reinterpret_cast<int *>(ws + 5 * m);
    g.st = st;
    g.g3 = g3;
    const long long nn = (long long)N * N;
    const int np = (N + LB - 1) / LB;
    // With up to three panels the fork costs what it saves (N = 300 305 us in
    // one block, 309 in steps; 400 434 and 405, 600 590 and 535).
    hipStream_t sb = np >= 4 ? aux_stream(1) : nullptr;
    // Ht's upper triangle by conjugation, Im(diag) = 0
    const auto mirror = [&]() -> hipError_t {
        if (g_sched) {
            if (g_sched->fails()) return hipErrorUnknown;
            g_sched->add(g_sched->launch(st, "k_mirror"), Ht, 0, N, 0, N, true);
            return hipSuccess;
        }
        return launch_mirror1(Ht, N, st);
    };
    if (g_sched) {
        const void *b[SB_COUNT] = {H, S, L, Ht, g.LH, g.M, g.MH, g.W, g.K, g.info};
        std::copy(b, b + SB_COUNT, g_sched->base);
        if (g_sched->fails()) return hipErrorUnknown;
        SchedOp &op = g_sched->launch(st, "k_gep_init");
        g_sched->add(op, S, 0, N, 0, N, false);
        for (const void *X : {(const void *)L, (const void *)g.M, (const void *)g.MH})
            g_sched->add(op, X, 0, N, 0, N, true);
        if (sb) {
            g_sched->add(op, H, 0, N, 0, N, false);
            g_sched->add(op, g.K, 0, N, 0, N, true);
        }
        g_sched->add(op, g.info, 0, 1, 0, 1, true);
    } else {
        hipLaunchKernelGGL(k_gep_init, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, st, H, S,
                           L, g.M, g.MH, sb ? g.K : nullptr, N, g.info);
        GEP_TRY(hipGetLastError());
    }
    g.cap = 0;
    if (!sb) {   // few panels: one block
        std::vector<std::vector<Node>> lv;
        tree(0, N, 0, lv);
        GEP_TRY(factor(g, [](int, hipEvent_t, Rect &) { return hipSuccess; }));
        GEP_TRY(invert(g, lv));
        GEP_TRY(diag_block(g, H, Ht, 0, N));
        return mirror();
    }
    // In steps of columns. Once the factorization has passed a step's columns
    // (the leaf and the panel product LH21 of its last panel are enqueued), the
    // step depends on nothing still to come: those of the first `bg` columns run
    // on a second stream, on bg_cap of the compute units, beside the rest of
    // the factorization, which no longer touches LH's columns < t0. The others follow it on all compute units.
    size_t nbg;
    const std::vector<int> ends = step_ends(N, &nbg);
    Gep gb = g;
    gb.st = sb;
    gb.cap = bg_cap(N, g_sched ? 256 : num_cus());
    hipEvent_t e_split = nullptr, e_inv = nullptr, e_v = nullptr;
    hipError_t err = ev_create(&e_split);
    if (err == hipSuccess) err = ev_create(&e_inv);
    if (err == hipSuccess) err = ev_create(&e_v);
    size_t done = 0;   // steps enqueued
    const auto begin = [&](size_t k) { return k ? ends[k - 1] : 0; };
    if (err == hipSuccess)
        err = factor(g, [&](int t0, hipEvent_t e_ahead, Rect &l21) -> hipError_t {
            if (done == nbg || t0 != ends[done]) return hipSuccess;
            GEP_TRY(ev_record(e_split, st));
            GEP_TRY(ev_wait(sb, e_split, WT_FORK));
            // an earlier L21 = LH21^H may still read LH's columns < t0 on the
            // lookahead stream, or is still to come; V overwrites them below
            if (e_ahead) GEP_TRY(ev_wait(sb, e_ahead, WT_FORK_AHEAD));
            const int a = begin(done++);
            GEP_TRY(conj_t_batch(gb, g.LH, L, &l21, 1));
            l21.i1 = l21.i0;
            GEP_TRY(step(gb, Ht, a, t0, [] { return hipSuccess; }));
            GEP_TRY(ev_record(e_inv, sb));
            GEP_TRY(diag_block(gb, g.K, Ht, a, t0));
            return ev_record(e_v, sb);
        });
    const size_t forked = done;
    for (; err == hipSuccess && done < ends.size(); ++done) {
        err = step(g, Ht, begin(done), ends[done], [&] {
            return done == forked ? ev_wait(st, e_inv, WT_END_AFTER_INVERSE) : hipSuccess;
        });
        if (err == hipSuccess) err = diag_block(g, g.K, Ht, begin(done), ends[done]);
    }
    if (err == hipSuccess && forked > 0) err = ev_wait(st, e_v, WT_END_AFTER_BACKGROUND);
    for (hipEvent_t e : {e_split, e_inv, e_v}) ev_destroy(e);
    GEP_TRY(err);
    return mirror();
}

}  // namespace

std::vector<int> gep_steps(int N) {
    size_t nbg;
    return step_ends(N, &nbg);
}

size_t gep_workspace_bytes(int N) {
    return 5 * padded(16 * (size_t)N * (size_t)N) + 256;   // LH, M, MH, W, K, info slot
}

hipError_t launch_gep(const double2 *H, const double2 *S, int N, double2 *L, double2 *Ht,
                      int *info, char *ws, hipStream_t st, bool g3) {
    const hipError_t e = enqueue_gep(H, S, N, L, Ht, info, ws, st, g3);
    if (e != hipSuccess && N > 3 * LB) join_after_error(st);   // only those use other streams
    return e;
}

namespace {
// launch_gep with the recorder installed: distinct stand-in addresses, nothing
// is dereferenced or launched.
hipStream_t sched_stream() { return reinterpret_cast<hipStream_t>((uintptr_t)0x10); }
hipError_t sched_run(Sched &sc, int N, bool g3) {
    auto fake = [](uintptr_t a) { return reinterpret_cast<double2 *>(a << 40); };
    g_sched = &sc;
    const hipError_t e = launch_gep(fake(1), fake(2), N, fake(3), fake(4), nullptr,
                                    reinterpret_cast<char *>((uintptr_t)1 << 44), sched_stream(), g3);
    g_sched = nullptr;
    return e;
}
}  // namespace

int gep_check_schedule(int N, bool g3, int drop_tag, std::string &report) {
    Sched sc;
    sc.drop_tag = drop_tag;
    if (sched_run(sc, N, g3) != hipSuccess) {
        report = "orchestration returned an error";
        return -1;
    }
    return sched_check(sc, N, report);
}

int gep_check_failure(int N, bool g3, int call, std::string &report) {
    Sched sc;
    sc.fail_call = call;
    sched_run(sc, N, g3);
    if (sc.calls < call) return -1;
    int unjoined = 0;
    const int races = sched_check(sc, N, report, sched_stream(), &unjoined);
    if (unjoined) report += std::to_string(unjoined) + " launches are not joined into the caller's stream";
    return races + unjoined;
}

}  // namespace hs
