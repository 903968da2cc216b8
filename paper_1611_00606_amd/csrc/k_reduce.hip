// The large stacked reductions, on complex FP64 MFMA tiles:
//   H = B^H Y + A^H X,   X_a = T^AA_a A_a + T^AB_a B_a,
//                        Y_a = T^BA_a A_a + T^BB_a B_a
//   S = A^H A + B^H |U|^2 B
// Both are Hermitian and only their lower triangles are computed, so neither
// needs a Hermitian rank-k form: the stacked operands [A; B] contract over 2K
// rows with [X; Y], where Alg. 1's terms Z^H B + B^H Z + (Y^H Y or A^H X)
// contract over 3K (its zher2k and zherk save the upper triangle, a choice
// the tiles make by themselves). At N_G = 8000, K = 8100: 125 ms for the two
// outputs against 155 ms in the 3K form, at the same error.
// The U scaling is applied to the right operand as |u|^2 while it is read.
//
// Only lower-triangle tiles are computed; a tile's epilogue also writes its
// conjugate transpose and Im(diagonal) = 0, so the outputs need no further
// pass. Three tile sizes share one launch (8-wave blocks of the same LDS),
// because a 128 x 128 tile takes 0.45 us of a CU per contraction row
// and 16 K N_G^2 operations rarely make a whole number of rounds of them:
//   128 x 128  the tiles strictly below the diagonal, first;
//    64 x  64  the diagonal blocks (3 of 4 quarters), the ragged last rows,
//              and the 128-tiles that would start an unfilled last round;
//    32 x  32  the 64-tiles that would start an unfilled last round.
// make_plan chooses how many of each from their measured costs, and whether
// one block has a compute unit to itself or two share it, each with half the
// LDS and half a 128-tile (128 x 64) at a time. (All in 128-tiles the build of
// 32 atoms of N_L = 49 at N_G = 2000 took 3.17 ms, two rounds for 272 tiles on
// 256 compute units; 1.96 ms in blocks of one per unit, 1.82 ms in two. The
// smallest build, 4 atoms of 16 at N_G = 256: 87 us, 30 us now. N_G = 8000, in
// one: 124.7 ms, 119.7 ms now, of which the mirroring pass was 0.4 ms.) All add
// an output's contraction rows in the same order, so the bits of H and S do not
// depend on the split.
//
// The tiles follow a banded order, of which each XCD walks a contiguous run
// of H's tiles and one of S's, H's first (xcd_item; one run over both outputs,
// half the XCDs at H and half at S: 122.8 against 119.7 ms at N_G = 8000).
//
// With G3 every complex product takes 3 real MFMA products instead of 4 (the
// 3M form, see zmfma_direct.h): three quarters of the matrix-core work, a
// slightly larger rounding bound on the imaginary parts.
//
// k_mirror completes the outputs of the split-precision reductions and of the
// eigenproblem reduction: upper = conj(lower), Im(diag) = 0.
#include "hs_internal.h"
#include "zmfma_direct.h"

namespace hs {

namespace {

// One block per compute unit, or two (2 x 72 KB of LDS, 128 registers a lane).
template <bool TWO>
struct Tiles {
    using T128 = TileCfg<128, 128, 8, 2, 4, 4>;   // 64 x 32 complex outputs per wave
    using T64 = TileCfg<64, 64, 16, 2, 4, 4>;     // 32 x 16
    using T32 = TileCfg<32, 32, 16, 2, 2, 8>;     // 16 x 16, four waves only load
    static constexpr int PARTS = 1;               // blocks per 128-tile
};
template <>
struct Tiles<true> {
    using T128 = TileCfg<128, 64, 8, 4, 2, 3>;    // 32 x 32
    using T64 = TileCfg<64, 64, 8, 2, 4, 4>;
    using T32 = TileCfg<32, 32, 16, 2, 2, 4>;
    static constexpr int PARTS = 2;
};
template <class T>
constexpr int red_lds() {
    static_assert(T::T64::LDS_ELEMS <= T::T128::LDS_ELEMS && T::T32::LDS_ELEMS <= T::T128::LDS_ELEMS,
                  "one LDS ring");
    return T::T128::LDS_ELEMS;
}
constexpr int RED_THREADS = Tiles<false>::T128::NT;
constexpr int BAND = 4;   // tile columns per band of the tile order

struct RedArgs {
    const double2 *A, *B, *X, *Y;
    const double *d;
    int K;
    double2 *H;
    double2 *S;
    int n_g;
    int nf;       // whole 128-tile rows
    int nlow;     // whole 128-tiles strictly below the diagonal, per output
    int nedge;    // diagonal quarters and last rows, in 64-tiles, per output
    int n128;     // of the 2 nlow, computed as 128-tiles
    int n64;      // of the remaining 64-tiles, computed as 64-tiles
    int n32;      // 64-tiles computed as four 32-tiles each
    int b128, b64;   // blocks of the first two ranges
};

// Tile (i, j), j < i, of the t-th position in the banded order: bands of
// BAND tile columns, each band walked row by row from its diagonal down.
__host__ __device__ __forceinline__ void band_tile(int t, int nt, int &ti, int &tj) {
    for (int c0 = 0;; c0 += BAND) {
        const int m = nt - c0;   // rows of the band, its first one empty
        const int w = m < BAND ? m : BAND;
        const int tri = w * (w - 1) / 2;
        const int cnt = tri + (m - w) * w;
        if (t < cnt) {
            if (t < tri) {
                int r = 1;
                while ((r + 1) * r / 2 <= t) ++r;
                ti = c0 + r;
                tj = c0 + (t - r * (r - 1) / 2);
            } else {
                const int u = t - tri;
                ti = c0 + w + u / w;
                tj = c0 + u % w;
            }
            return;
        }
        t -= cnt;
    }
}

// What a block computes: a 128-tile (a 128 / PARTS columns wide part of it), 64-
// or 32-tile at rows m0, columns n0. size 0: nothing.
struct RedPlace {
    bool isH;
    int size, m0, n0;
};
template <int PARTS>
__host__ __device__ __forceinline__ RedPlace red_place(const RedArgs &args, int b) {
    RedPlace r = {false, 0, 0, 0};
    if (b < args.b128) {
        int q = xcd_item(b, PARTS * args.n128, PARTS * args.nlow);
        if (q < 0) return r;
        const int part = q % PARTS;
        q /= PARTS;
        r.isH = q < args.nlow;
        int ti, tj;
        band_tile(r.isH ? q : q - args.nlow, args.nf, ti, tj);
        r.size = 128;
        r.m0 = ti * 128;
        r.n0 = tj * 128 + part * (128 / PARTS);
        return r;
    }
    b -= args.b128;
    const bool whole = b < args.b64;
    int sub = 0, u;
    if (whole) {
        u = xcd_item(b, args.n64, args.n64);
        if (u < 0) return r;
    } else {
        b -= args.b64;
        sub = b & 3;
        u = args.n64 + (b >> 2);
    }
    // 64-tile u: quarters of the 128-tiles after the first n128, then the
    // diagonal quarters and last rows of H, then of S
    int I, J;   // in 64-tiles
    const int nq = 4 * (2 * args.nlow - args.n128);
    if (u < nq) {
        const int q = args.n128 + u / 4;
        r.isH = q < args.nlow;
        band_tile(r.isH ? q : q - args.nlow, args.nf, I, J);
        I = 2 * I + (u >> 1 & 1);
        J = 2 * J + (u & 1);
    } else {
        u -= nq;
        r.isH = u < args.nedge;
        if (!r.isH) u -= args.nedge;
        if (u < 3 * args.nf) {
            const int q = u % 3;   // (0,0), (1,0), (1,1) of the diagonal block
            I = 2 * (u / 3) + (q + 1) / 2;
            J = 2 * (u / 3) + q / 2;
        } else {
            u -= 3 * args.nf;
            I = 2 * args.nf;
            if (u > I) {
                u -= I + 1;
                ++I;
            }
            J = u;
        }
    }
    r.size = whole ? 64 : 32;
    r.m0 = I * 64 + (whole ? 0 : (sub >> 1) * 32);
    r.n0 = J * 64 + (whole ? 0 : (sub & 1) * 32);
    return r;
}

// One C::BM x C::BN tile of H or S at rows m0, columns n0 (multiples of C::BN).
template <class C, bool G3>
__device__ __forceinline__ void reduce_tile(const RedArgs &args, bool isH, int m0, int n0,
                                            double2 *lds) {
    const int n_g = args.n_g;
    if (m0 >= n_g || n0 > m0) return;
    // Segment tables are built from scalar arguments in registers: taking a
    // reference into the by-value kernel argument would copy it to scratch.
    Acc<C> acc;
    if (isH) {
        // B^H Y + A^H X: the larger terms last (T^AA carries most of H), which
        // leaves fewer roundings at the full size of the sum
        Segs<2, false> t;
        t.nseg = 2;
        t.len = args.K;
        t.ldp = t.ldq = n_g;
        t.P[0] = args.B;
        t.Q[0] = args.Y;
        t.P[1] = args.A;
        t.Q[1] = args.X;
        t.qscale = nullptr;
        ztile_direct<C, 2, false, G3>(t, m0, n_g, n0, n_g, acc, lds);
    } else {
        // A^H A + B^H diag(|u|^2) B
        Segs<2, true> t;
        t.nseg = 2;
        t.len = args.K;
        t.ldp = t.ldq = n_g;
        t.P[0] = args.A;
        t.Q[0] = args.A;
        t.P[1] = args.B;
        t.Q[1] = args.B;
        t.qscale = args.d;     // [2K]: 1 on A's rows, |u|^2 on B's rows
        ztile_direct<C, 2, true, G3>(t, m0, n_g, n0, n_g, acc, lds);
    }
    if (!wave_works<C>()) return;
    double2 *out = isH ? args.H : args.S;
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j) {
            const int g = n0 + acc_col<C>(j);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gp = m0 + acc_row<C>(i, v);
                if (gp < n_g && g <= gp) {
                    const double re = acc.re[i][j][v], im = g == gp ? 0.0 : acc.im[i][j][v];
                    out[(long long)gp * n_g + g] = double2{re, im};
                    // lanes l / 16 = 0..3 hold four consecutive rows gp: 64-byte
                    // runs of a transposed row, its other runs follow with v
                    if (g != gp) out[(long long)g * n_g + gp] = double2{re, -im};
                }
            }
        }
}

template <bool G3, bool TWO>
__global__ void __launch_bounds__(RED_THREADS) __attribute__((amdgpu_waves_per_eu(TWO ? 4 : 2)))
k_reduce(RedArgs args) {
    using T = Tiles<TWO>;
    __shared__ double2 lds[red_lds<T>()];

    const RedPlace p = red_place<T::PARTS>(args, blockIdx.x);
    if (p.size == 128) reduce_tile<typename T::T128, G3>(args, p.isH, p.m0, p.n0, lds);
    else if (p.size == 64) reduce_tile<typename T::T64, G3>(args, p.isH, p.m0, p.n0, lds);
    else if (p.size == 32) reduce_tile<typename T::T32, G3>(args, p.isH, p.m0, p.n0, lds);
}

// When n tiles of equal cost have been handed to slots for a block in turn,
// each to the first that is free; level: the busy time of groups of them.
struct Level {
    double t;
    int n;
};
void hand_out(std::vector<Level> &lv, long long n, double cost) {
    while (n > 0) {
        size_t m = 0;
        for (size_t i = 1; i < lv.size(); ++i)
            if (lv[i].t < lv[m].t) m = i;
        const int k = (int)std::min<long long>(n, lv[m].n);
        n -= k;
        if (k < lv[m].n) lv.push_back(Level{lv[m].t, lv[m].n - k});
        lv[m].t += cost;
        lv[m].n = k;
    }
}

// End of the last block. Of two blocks per compute unit, those left when half
// the slots are empty have a unit to themselves and run 1.7 times as fast.
double end_time(std::vector<Level> &lv, int cus, bool two) {
    std::sort(lv.begin(), lv.end(), [](const Level &a, const Level &b) { return a.t < b.t; });
    const double end = lv.back().t;
    if (!two) return end;
    double half = 0.0;
    int n = 0;
    for (const Level &x : lv) {
        half = x.t;
        n += x.n;
        if (n >= cus) break;
    }
    return half + (end - half) / 1.7;
}

// Costs of the tiles, in units of a compute unit's time for a row of a
// 128-tile in blocks of one per unit: per row the 128-tile, and the 64- and
// 32-tiles by area, from a full device at N_G = 8000, K = 8100 (116.0 ms in
// 128-tiles; in two blocks per unit 118.4 in halves of them, 133.0 in 64-tiles,
// 150.6 in 32-tiles); per tile 20 rows (10 us) to fill the ring and to write.
struct Costs {
    double c128, c64, c32;
};
constexpr Costs COSTS_ONE = {1.0, 1.17, 1.45}, COSTS_TWO = {1.02, 1.14, 1.30},
                COSTS_ONE_3M = {1.0, 1.22, 1.61};
constexpr double TILE_ROWS = 20.0;

// How many tiles of each size, and whether in one or two blocks per compute
// unit (true): the split with the earliest end among a few of each kind. Two
// blocks cover each other's first loads and last stores and end more evenly,
// one block loads each operand less often: (ms, one / two) N_G = 600 0.153 /
// 0.140, 2000 1.76 / 1.62, 2500 6.85 / 6.65, 3000 8.62 / 8.96, 8000 116.0 /
// 118.4; the estimates are within 3% of most measured times. The 3M form's
// third accumulator leaves no room for two.
bool make_plan(RedArgs &a, int cus, bool g3) {
    const int n64rows = (a.n_g + 63) / 64;
    a.nf = a.n_g / 128;
    a.nlow = a.nf * (a.nf - 1) / 2;
    a.nedge = 3 * a.nf;
    for (int i = 2 * a.nf; i < n64rows; ++i) a.nedge += i + 1;
    const int all = 2 * a.nlow;
    const double rows = 2.0 * a.K;
    double best = -1.0;
    bool best_two = false;
    std::vector<Level> lv;
    for (int parts = 1; parts <= (g3 ? 1 : 2); ++parts) {
        const bool two = parts == 2;
        const Costs &c = g3 ? COSTS_ONE_3M : two ? COSTS_TWO : COSTS_ONE;
        const double t128 = c.c128 * rows + TILE_ROWS;   // a slot's time
        const double t64 = parts * c.c64 / 4 * rows + TILE_ROWS;
        const double t32 = parts * c.c32 / 16 * rows + TILE_ROWS;
        for (int k = 0; k < 4; ++k) {   // all 128-tiles, the whole rounds of them, one fewer, none
            const int f = k == 0 ? all : k == 3 ? 0 : std::max(0, all / cus - (k - 1)) * cus;
            const int rest = 4 * (all - f) + 2 * a.nedge;
            for (int l = 0; l < 6; ++l) {   // all 64-tiles, up to two rounds fewer, none
                const int h = l == 5 ? 0 : std::max(0, rest - l * cus / 2);
                lv.assign(1, Level{f / cus * t128, parts * cus});
                hand_out(lv, parts * (f % cus), t128);
                hand_out(lv, h, t64);
                hand_out(lv, 4LL * (rest - h), t32);
                const double end = end_time(lv, cus, two);
                if (best < 0.0 || end < best) {
                    best = end;
                    best_two = two;
                    a.n128 = f;
                    a.n64 = h;
                    a.n32 = rest - h;
                }
            }
        }
    }
    a.b128 = xcd_blocks((best_two ? 2 : 1) * a.n128);
    a.b64 = xcd_blocks(a.n64);
    return best_two;
}

// upper := conj(lower) through a 32x32 LDS transpose; Im(diag) := 0.
constexpr int MT = 32;
__global__ void __launch_bounds__(256)
k_mirror(double2 *H, double2 *S, int n_g) {
    const int bx = blockIdx.x, by = blockIdx.y;   // destination tile: rows by, cols bx
    if (bx < by) return;
    double2 *M = blockIdx.z == 0 ? H : S;
    __shared__ double2 tile[MT][MT + 1];
    const int tx = threadIdx.x % MT, ty = threadIdx.x / MT;   // 32 x 8
    // source: lower tile rows bx*32.., cols by*32..
    for (int r = ty; r < MT; r += 8) {
        const int gr = bx * MT + r, gc = by * MT + tx;
        if (gr < n_g && gc < n_g && gc <= gr) tile[r][tx] = M[(long long)gr * n_g + gc];
    }
    __syncthreads();
    for (int r = ty; r < MT; r += 8) {
        const int gr = by * MT + r, gc = bx * MT + tx;   // destination (gr, gc), gr <= gc
        if (gr < n_g && gc < n_g) {
            if (gr < gc) {
                double2 v = tile[tx][r];
                v.y = -v.y;
                M[(long long)gr * n_g + gc] = v;
            } else if (gr == gc) {
                M[(long long)gr * n_g + gc].y = 0.0;
            }
        }
    }
}

}  // namespace

hipError_t launch_reduce(int K, int n_g, const double2 *A, const double2 *B,
                         const double2 *X, const double2 *Y, const double *d,
                         double2 *H, double2 *S, hipStream_t st, bool g3) {
    RedArgs args;
    args.A = A;
    args.B = B;
    args.X = X;
    args.Y = Y;
    args.d = d;
    args.K = K;
    args.H = H;
    args.S = S;
    args.n_g = n_g;
    const bool two = make_plan(args, num_cus(), g3);
    const dim3 grid(args.b128 + args.b64 + 4 * args.n32);
    if (g3)
        hipLaunchKernelGGL((k_reduce<true, false>), grid, dim3(RED_THREADS), 0, st, args);
    else if (two)
        hipLaunchKernelGGL((k_reduce<false, true>), grid, dim3(RED_THREADS), 0, st, args);
    else
        hipLaunchKernelGGL((k_reduce<false, false>), grid, dim3(RED_THREADS), 0, st, args);
    return hipGetLastError();
}

int reduce_check_plan(int K, int n_g, bool g3, int cus, int plan[4]) {
    RedArgs a = {};
    a.K = K;
    a.n_g = n_g;
    const bool two = make_plan(a, cus, g3);
    plan[0] = two ? 2 : 1;
    plan[1] = a.n128;
    plan[2] = a.n64;
    plan[3] = a.n32;
    constexpr int CELL = 32;
    CellCount cells(n_g, CELL, CELL);
    for (int b = 0; b < a.b128 + a.b64 + 4 * a.n32; ++b) {
        const RedPlace p = two ? red_place<2>(a, b) : red_place<1>(a, b);
        if (p.size) cells.add(p.isH, p.m0, p.n0, p.size, p.size == 128 ? 128 / plan[0] : p.size);
    }
    return cells.wrong();
}

hipError_t launch_mirror(double2 *H, double2 *S, int n_g, hipStream_t st) {
    const int mt = (n_g + MT - 1) / MT;
    hipLaunchKernelGGL(k_mirror, dim3(mt, mt, 2), dim3(256), 0, st, H, S, n_g);
    return hipGetLastError();
}

hipError_t launch_mirror1(double2 *M, int n, hipStream_t st) {
    const int mt = (n + MT - 1) / MT;
    hipLaunchKernelGGL(k_mirror, dim3(mt, mt, 1), dim3(256), 0, st, M, M, n);
    return hipGetLastError();
}

}  // namespace hs
