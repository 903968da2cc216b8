// Modular INT8 form of the large reductions (HS_SPLIT_I8_CRT): the four
// stacked products of H = A^H X + B^H Y and S = A^H A + (U B)^H (U B) (see
// k_reduce.hip) computed exactly on integers.
//
// Operands. For each column n of a sliced operand X let s[n] be the exponent
// with which ||X[.][n]|| 2^s lies in (2^41.85, 2^42.85], ||X|| bounded by
// sqrt(K / 64) times the largest norm of 64 rows, and
//     X'[k][n] = rint(X[k][n] 2^s)
// for the real and the imaginary parts. This rounding is the form's only
// error: up to 2^-43.85 .. 2^-42.85 of the column's norm per element, at 8100
// rows of equal size 2^-36.4 .. 2^-35.4 of their size. (Integers of 36 bits at
// the column's maximum, which the bound 2 K 2^70 on their products allows up
// to K = 28000, are 2 to 3 bits coarser for Gaussian columns: H at N_G = 8000,
// K = 8100 was 6.1e-11 off, now 8.8e-12.)
//
// Products. The real part p_re q_re + p_im q_im and the imaginary part
// p_re q_im - p_im q_re of conj(P')^T Q' are each one dot product of 2K
// integers, so |Re|, |Im| <= ||P'|| ||Q'||. Both are computed modulo NMOD
// pairwise coprime odd moduli m_i <= 255: the operands' residues in symmetric
// form (|r| <= (m - 1) / 2 <= 127, so a residue and its negation are int8),
// INT8 MFMA products summed exactly in INT32 and reduced to a symmetric
// residue at the end of the segment. With M = prod m_i, (M - 1) / 2 = 2^85.803
// and ||X'|| <= 2^42.85 + sqrt(2K) / 2 < 2^42.901 (the rounding; K <= 2^28),
// the residues fix each integer uniquely in the symmetric range of M.
//
// Reconstruction (Chinese remainder theorem in Garner's mixed-radix form):
//     X = v_0 + m_0 (v_1 + m_1 (v_2 + ... + m_9 v_10)),
//     v_i = (r_i - sum_{j<i} v_j W_j) W_i^-1  mod m_i,   W_j = m_0 ... m_{j-1},
// with symmetric digits v_i, computed exactly in FP32 (every intermediate is
// an integer below 2^24) and evaluated in FP64 with one rounding. Each
// segment's integer is scaled by 2^-(sP + sQ) and the segments of
// H (two) and of S (two) are added in FP64.
//
// The scheme is the modular-integer emulation of floating-point matrix
// products of Ozaki, Uchino and Imamura ("Ozaki scheme II", 2025). Against
// the INT8 slice pairs of HS_SPLIT_I8 (15 INT8 products per complex product)
// it needs one per modulus (11), and the INT32 sums of a modulus need no
// per-level accumulators, so a wave holds a four times larger output tile.
#include <cmath>

#include "hs_internal.h"
#include "split_common.h"

namespace hs {

namespace {

typedef int i4 __attribute__((ext_vector_type(4)));

constexpr int NMOD = 11;
constexpr int CRT_MOD[NMOD] = {255, 253, 251, 247, 241, 239, 233, 229, 227, 223, 217};
constexpr int NSEG = 4;        // H: (B, Y), (A 2^e, X 2^-e); S: (A, A), (Bs, Bs)
// Segments the work buffer has room for (part of the workspace size callers
// have been given).
constexpr int NSEG_ROOM = 5;

// Garner constants, symmetric: w[i][j] = W_j mod m_i (j < i), u[i] = W_i^-1 mod m_i.
constexpr int sym_mod_c(long long x, int m) {
    long long r = x % m;
    if (r < 0) r += m;
    return r > m / 2 ? (int)(r - m) : (int)r;
}
constexpr int inv_mod_c(long long a, int m) {
    a %= m;
    if (a < 0) a += m;
    for (int x = 1; x < m; ++x)
        if (a * x % m == 1) return x;
    return 0;
}
struct GarnerTab {
    int w[NMOD][NMOD];
    int u[NMOD];
    int wu[NMOD][NMOD];   // w[i][j] u[i] mod m_i, symmetric
};
constexpr GarnerTab make_garner() {
    GarnerTab t{};
    for (int i = 0; i < NMOD; ++i) {
        long long wm = 1;   // W_j mod m_i
        for (int j = 0; j < i; ++j) {
            t.w[i][j] = sym_mod_c(wm, CRT_MOD[i]);
            wm = wm * CRT_MOD[j] % CRT_MOD[i];
        }
        t.u[i] = sym_mod_c(inv_mod_c(wm, CRT_MOD[i]), CRT_MOD[i]);
        for (int j = 0; j < i; ++j) t.wu[i][j] = sym_mod_c((long long)t.w[i][j] * t.u[i], CRT_MOD[i]);
    }
    return t;
}
constexpr GarnerTab GT = make_garner();
static_assert(GT.u[0] == 1 && ((long long)GT.u[1] * 255 % 253 + 253) % 253 == 1, "Garner table");
// a digit's sum r_i u_i - sum_{j<i} wu[i][j] v_j is an integer below 2^24
static_assert(NMOD * 127 * 127 < (1 << 24), "Garner sums exact in FP32");
// three symmetric digits fold into an integer below 2^24 (exact in FP32)
static_assert(255LL * 253 * 251 / 2 < (1 << 24), "digit groups exact in FP32");

// Exponent s of a column from the largest norm of 64 of its rows; cn: crt_norm(K).
__device__ __forceinline__ int crt_shift(const unsigned long long *mx, int n, double cn) {
    const double m = __longlong_as_double((long long)mx[n]);
    int e = 0, d = 0;
    if (m > 0.0) frexp(frexp(m, &e) * cn, &d);
    return 42 - e - d;
}
// 2^-0.85 sqrt(blocks of 64 rows) and the norms' 2^-4, a little more for their
// own rounding
double crt_norm(int K) { return 16.0 * 0.55478473603393 * (1.0 + 1e-12) * std::sqrt((double)((K + 63) / 64)); }

__device__ __forceinline__ int crt_modulus(int mi) {
    int m = CRT_MOD[0];
#pragma unroll
    for (int i = 1; i < NMOD; ++i)
        if (mi == i) m = CRT_MOD[i];
    return m;
}

// ---------------------------------------------------------------------------
// Residues. One thread per (16 complex rows, column): the real and the
// imaginary parts -> integers -> NMOD residues of 16 int8 each, written
// to R[i][g][n][0..15]. A stage of the products is 64 complex rows, eight
// items g of a column: the real parts of rows 16 q .. 16 q + 15 (q = 0..3),
// then the imaginary parts.

__global__ void __launch_bounds__(256)
k_residue(SliceJobs jobs, int K, int n_g, int blocks, double cn) {
    const int z = blockIdx.y;
    const double2 *X = slice_ptr(jobs.M, z);
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    const int n = (int)(idx % n_g);
    const int rb = (int)(idx / n_g);   // block of 16 rows
    if (rb >= blocks) return;
    double2 raw[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int k = 16 * rb + q;
        raw[q] = double2{0.0, 0.0};
        if (k < K) raw[q] = X[(long long)k * n_g + n];
    }
    const auto cut = [&](int op) __attribute__((always_inline)) {
        const int sh = crt_shift(slice_ptr(jobs.mx, op), n, cn);
        double x[2][16];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const double2 v = raw[q];
            x[0][q] = rint(ldexp(v.x, sh));
            x[1][q] = rint(ldexp(v.y, sh));
        }
        const long long plane = 2LL * blocks * n_g;   // 16-byte items per modulus
        uint4 *out = reinterpret_cast<uint4 *>(slice_ptr(jobs.S, op)) + (8LL * (rb >> 2) + (rb & 3)) * n_g + n;
#pragma unroll
        for (int i = 0; i < NMOD; ++i) {
            // x / m is below 2^36 and at least 1 / (2 m) from a half-integer,
            // so rint of the rounded quotient is exact and so is the remainder
            const double m = CRT_MOD[i], inv = 1.0 / CRT_MOD[i];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                unsigned w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const double r = fma(-m, rint(x[c][j] * inv), x[c][j]);
                    w[j >> 2] |= ((unsigned)(int)r & 0xffu) << (8 * (j & 3));
                }
                out[i * plane + 4LL * c * n_g] = uint4{w[0], w[1], w[2], w[3]};
            }
        }
    };
    slice_operands(jobs, z, [&](SliceForm form) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 16; ++q)
            if (16 * rb + q < K) raw[q] = slice_value(jobs, form, raw[q], 16 * rb + q);
    }, cut);
}

// ---------------------------------------------------------------------------
// Products modulo one modulus. One block per (128 x 128 lower-triangle tile,
// segment, modulus): 4 waves of 64 x 64 outputs (4 x 4 MFMA blocks of
// 16 x 16), two blocks per CU (two waves per SIMD). A stage is 64 complex
// rows: 8 items of 16 bytes per column and operand, the real and the
// imaginary parts in items of their own, moved global -> LDS with 16-byte
// direct loads, two 32 KiB buffers (the next stage loads while the current
// one is multiplied). The difference in the imaginary part is taken once, at
// the end: its two sums have accumulators of their own (192 registers in all),
// so the K loop holds no vector arithmetic besides the MFMAs. (With the parts
// interleaved and (q_im, -q_re) formed in registers, three vector operations
// per dword, the kernel took 38.1 ms at N_G = 8000, K = 8100; now 34.7 ms,
// 2.63 POP/s.) The INT32 sums stay exact for CFOLD stages (checked below);
// longer segments reduce them modulo m every CFOLD stages.
//
// Measured at N_G = 8000 (K = 8100): against 8 waves of 64 x 32 outputs in
// 128-row stages (one block per CU) this shape reads a third less from LDS
// per MFMA and was 9% faster; deeper pipelines (3 to 5 buffers, up to four
// stages in flight) are not faster, nor is V_MFMA_I32_32X32X32_I8 (49.4
// against 45.3 ms for the build). Bands of 8 tile columns in the tile order
// (64 tiles resident per XCD share 8 row and 8 column panels) fetch 15% less
// than bands of 4.

constexpr int CB = 128;                    // tile rows (g') and columns (g)
constexpr int CWM = 2, CWN = 2;            // waves
constexpr int CNT = 64 * CWM * CWN;
constexpr int CTM = CB / CWM / 16, CTN = CB / CWN / 16;   // 16 x 16 blocks per wave
constexpr int CITEMS = 8;                  // items per column and stage (64 complex rows)
constexpr int COP = CITEMS * CB;           // items per operand and stage
constexpr int CBUF = 2 * COP;
constexpr int CFOLD = 1024;                // stages between reductions of the sums
constexpr int CBAND = 8;
constexpr int CFRAG = CWM * CWN * CTM * CTN;   // 16 x 16 blocks per tile (64)
constexpr int CWAVES_EU = 2;               // waves per SIMD (at most 256 registers each)
constexpr int CNBUF = 2;                   // LDS stage buffers: CNBUF - 1 stages in flight
constexpr int CHW = CWM * CWN / 2;         // loader waves per operand
constexpr int CLPW = 2 * CITEMS / CHW;     // direct loads per wave and stage
static_assert((long long)CFOLD * CITEMS * 16 * 127 * 127 + 127 < (1LL << 31), "INT32 sums exact");
static_assert(CFRAG == 64, "the residue layout assumes 64 blocks per tile");

struct CrtArgs {
    const uint4 *P[NSEG], *Q[NSEG];   // residue planes of modulus 0 per segment
    const int *scaled;                 // 0: segment 1's P is segment 2's, A
    uint2 *out;                        // [NSEG * NMOD][ntri][CFRAG][64 lanes]
    long long plane;                   // items per modulus plane
    int n_g, groups, nt, ntri, ntri8;
};

// symmetric residue of an INT32 sum (exact: the quotient is below 2^24 and at
// least 1 / (2 m) from a half-integer)
__device__ __forceinline__ int sym_res(int x, double m, double inv) {
    const double d = (double)x;
    return (int)fma(-m, rint(d * inv), d);
}

__global__ void __launch_bounds__(CNT) __attribute__((amdgpu_waves_per_eu(CWAVES_EU)))
k_crt_reduce(CrtArgs args) {
    __shared__ uint4 bufs[CNBUF * CBUF];

    const int job = blockIdx.y;
    const int seg = job / NMOD, mi = job - seg * NMOD;
    const int bx = blockIdx.x;
    const int per_xcd = args.ntri8 / 8;
    const int t = (bx % 8) * per_xcd + bx / 8;
    if (t >= args.ntri) return;
    int ti, tj;
    sband_tile(t, args.nt, ti, tj, CBAND);
    if (ti < 0) return;
    const int n_g = args.n_g;
    const int m0 = ti * CB, n0 = tj * CB;
    // the segment's planes, selected with constant indices (a dynamic index
    // into the argument block would copy it to scratch memory)
    const uint4 *P = args.P[0], *Q = args.Q[0];
#pragma unroll
    for (int s = 1; s < NSEG; ++s)
        if (seg == s) {
            P = args.P[s];
            Q = args.Q[s];
        }
    if (seg == 1 && !*args.scaled) P = args.P[2];
    P += mi * args.plane;
    Q += mi * args.plane;
    const double m = crt_modulus(mi);
    const double minv = 1.0 / m;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % CWM, wn = wave / CWM;

    // loader: the first half of the waves fills P's item rows, the second
    // half Q's; wave w of a half takes rows w, w + CHW, w + 2 CHW, ..., both
    // 64-column halves of each; columns past the edge read the last column
    // (they only feed outputs past N_G, never used)
    static_assert(CB == 128 && CITEMS % CHW == 0, "the loader's split of the stage");
    const int op_w = wave / CHW, row_w = wave % CHW;
    const int cb = (op_w == 0 ? m0 : n0) + lane;
    const unsigned o0 = (unsigned)(cb < n_g ? cb : n_g - 1) * 16u;
    const unsigned o1 = (unsigned)(cb + 64 < n_g ? cb + 64 : n_g - 1) * 16u;
    const uint4 *ldsrc = op_w == 0 ? P : Q;
    auto issue = [&](uint4 *buf, int st) __attribute__((always_inline)) {
        uint4 *dst = buf + op_w * COP + row_w * CB;
        const uint4 *rows = ldsrc + (long long)(st * CITEMS + row_w) * n_g;
#pragma unroll
        for (int i = 0; i < CITEMS / CHW; ++i) {
            const char *r = reinterpret_cast<const char *>(rows + (long long)(CHW * i) * n_g);
            __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint4 *>(r + o0),
                                             dst + CHW * i * CB, 16, 0, 0);
            __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint4 *>(r + o1),
                                             dst + CHW * i * CB + 64, 16, 0, 0);
        }
    };

    // Re = sum pr qr + pi qi; Im = U - V, U = sum pr qi, V = sum pi qr
    i4 accr[CTM][CTN], accu[CTM][CTN], accv[CTM][CTN];
#pragma unroll
    for (int i = 0; i < CTM; ++i)
#pragma unroll
        for (int j = 0; j < CTN; ++j) accr[i][j] = accu[i][j] = accv[i][j] = i4{0, 0, 0, 0};
    const int lg = lane >> 4, lc = lane & 15;
    auto compute = [&](const uint4 *buf) __attribute__((always_inline)) {
        const uint4 *lp = buf;
        const uint4 *lq = buf + COP;
        i4 ar[CTM], ai[CTM];
#pragma unroll
        for (int i = 0; i < CTM; ++i) {
            ar[i] = __builtin_bit_cast(i4, lp[lg * CB + wm * (CB / CWM) + i * 16 + lc]);
            ai[i] = __builtin_bit_cast(i4, lp[(4 + lg) * CB + wm * (CB / CWM) + i * 16 + lc]);
        }
#pragma unroll
        for (int j = 0; j < CTN; ++j) {
            const i4 br = __builtin_bit_cast(i4, lq[lg * CB + wn * (CB / CWN) + j * 16 + lc]);
            const i4 bi = __builtin_bit_cast(i4, lq[(4 + lg) * CB + wn * (CB / CWN) + j * 16 + lc]);
#pragma unroll
            for (int i = 0; i < CTM; ++i) {
                accr[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ar[i], br, accr[i][j], 0, 0, 0);
                accu[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ar[i], bi, accu[i][j], 0, 0, 0);
                accv[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ai[i], br, accv[i][j], 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < CTM; ++i)
                accr[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ai[i], bi, accr[i][j], 0, 0, 0);
        }
    };
    auto fold = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < CTM; ++i)
#pragma unroll
            for (int j = 0; j < CTN; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    accr[i][j][v] = sym_res(accr[i][j][v], m, minv);
                    accu[i][j][v] = sym_res(accu[i][j][v] - accv[i][j][v], m, minv);
                    accv[i][j][v] = 0;
                }
    };

    const int nstage = args.groups / CITEMS;
#pragma unroll
    for (int s = 0; s < CNBUF - 1; ++s)
        if (s < nstage) issue(bufs + s * CBUF, s);
    for (int st = 0; st < nstage; ++st) {
        // this wave's loads of stage st are done (those of up to CNBUF - 2
        // later stages may still be in flight); after the barrier every
        // wave's are, and every wave has finished the stage before, whose
        // buffer is refilled next
        if (st + CNBUF - 2 < nstage)
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((CNBUF - 2) * CLPW) : "memory");
        else
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        // a plain barrier: __syncthreads() would also wait for the later
        // stages' loads (its fence covers every outstanding memory access)
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        // the buffer being computed and the one being loaded are distinct:
        // saying so (restrict) keeps the compiler from waiting for the
        // direct loads before every LDS read of the stage
        auto stage = [&](const uint4 *__restrict__ cur, uint4 *__restrict__ nxt)
                         __attribute__((always_inline)) {
            if (st + CNBUF - 1 < nstage) issue(nxt, st + CNBUF - 1);
            compute(cur);
        };
        stage(bufs + (st % CNBUF) * CBUF, bufs + ((st + CNBUF - 1) % CNBUF) * CBUF);
        if ((st + 1) % CFOLD == 0) fold();
    }
    fold();

    // residues of the 4 rows (4 lg + v) of column lc of every 16 x 16 block:
    // Re in x, Im in y, one byte per row, stored as r + 127 (0 .. 254)
    uint2 *out = args.out + ((long long)job * args.ntri + t) * CFRAG * 64;
#pragma unroll
    for (int i = 0; i < CTM; ++i)
#pragma unroll
        for (int j = 0; j < CTN; ++j) {
            unsigned re = 0u, im = 0u;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                re |= (unsigned)(accr[i][j][v] + 127) << (8 * v);
                im |= (unsigned)(accu[i][j][v] + 127) << (8 * v);
            }
            out[(wave * CTM * CTN + i * CTN + j) * 64 + lane] = uint2{re, im};
        }
}

// ---------------------------------------------------------------------------
// Reconstruction: one thread per (tile, 16 x 16 block, lane) of H or S, i.e.
// 4 outputs (rows 4 lg + v, column lc) as laid out by k_crt_reduce.

struct CrtRecArgs {
    const uint2 *res;
    const unsigned long long *mP[NSEG], *mQ[NSEG];
    const int *scaled;
    double2 *H, *S;
    int n_g, nt, ntri;
    double cn;
};

// The integer with residues rb[i] - 127 (rb: the stored bytes). Digit i is
// (r_i u_i - sum_{j<i} (W_j u_i mod m_i) v_j) mod m_i, one reduction per
// digit; digits are folded three at a time in FP32 and the four groups in
// FP64 in pairs (below 2^40 and 2^48), all exact, then the two pairs.
__device__ __forceinline__ double garner(const float (&rb)[NMOD]) {
    float v[NMOD];
    v[0] = rb[0] - 127.0f;
#pragma unroll
    for (int i = 1; i < NMOD; ++i) {
        const float mf = (float)CRT_MOD[i];
        const float inv = 1.0f / (float)CRT_MOD[i];
        float s = fmaf(rb[i], (float)GT.u[i], -127.0f * (float)GT.u[i]);     // r_i u_i
#pragma unroll
        for (int j = 0; j < i; ++j) s = fmaf(-(float)GT.wu[i][j], v[j], s);  // |s| < 2^24
        v[i] = fmaf(-mf, rintf(s * inv), s);                                  // |v_i| <= 127
    }
    auto fold3 = [&](int i) __attribute__((always_inline)) {   // v_i + m_i (v_i+1 + m_i+1 v_i+2)
        return fmaf((float)CRT_MOD[i], fmaf((float)CRT_MOD[i + 1], v[i + 2], v[i + 1]), v[i]);
    };
    const double g0 = fold3(0), g1 = fold3(3), g2 = fold3(6);
    const double g3 = fmaf((float)CRT_MOD[9], v[10], v[9]);
    constexpr double P3 = (double)CRT_MOD[0] * CRT_MOD[1] * CRT_MOD[2];
    constexpr double P6 = (double)CRT_MOD[3] * CRT_MOD[4] * CRT_MOD[5];
    constexpr double P9 = (double)CRT_MOD[6] * CRT_MOD[7] * CRT_MOD[8];
    static_assert(NMOD == 11, "the digit grouping assumes 11 moduli");
    return fma(fma(g3, P9, g2), P3 * P6, fma(g1, P3, g0));   // one rounding, the last
}

__global__ void __launch_bounds__(256)
k_crt_recon(CrtRecArgs a) {
    const long long id = (long long)blockIdx.x * 256 + threadIdx.x;
    const bool isH = blockIdx.y == 0;
    const int lane = (int)(id & 63);
    const int f = (int)((id >> 6) % CFRAG);
    const int t = (int)(id / (64 * CFRAG));
    if (t >= a.ntri) return;
    int ti, tj;
    sband_tile(t, a.nt, ti, tj, CBAND);
    if (ti < 0) return;
    const int wave = f / (CTM * CTN), i = (f % (CTM * CTN)) / CTN, j = f % CTN;
    const int wm = wave % CWM, wn = wave / CWM;
    const int lg = lane >> 4, lc = lane & 15;
    const int n_g = a.n_g;
    const int g = tj * CB + wn * (CB / CWN) + j * 16 + lc;
    const int gp0 = ti * CB + wm * (CB / CWM) + i * 16 + 4 * lg;
    if (g >= n_g || gp0 >= n_g || g > gp0 + 3) return;   // no output of the lower triangle

    double sr[4] = {0.0, 0.0, 0.0, 0.0}, si[4] = {0.0, 0.0, 0.0, 0.0};
    auto segment = [&](int s, const unsigned long long *mP, const unsigned long long *mQ)
                       __attribute__((always_inline)) {
        uint2 w[NMOD];
#pragma unroll
        for (int mi = 0; mi < NMOD; ++mi)
            w[mi] = a.res[(((long long)(s * NMOD + mi) * a.ntri + t) * CFRAG + f) * 64 + lane];
        const int sq = crt_shift(mQ, g, a.cn);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float rr[NMOD], ri[NMOD];
#pragma unroll
            for (int mi = 0; mi < NMOD; ++mi) {
                rr[mi] = (float)((w[mi].x >> (8 * v)) & 0xffu);
                ri[mi] = (float)((w[mi].y >> (8 * v)) & 0xffu);
            }
            const int gp = gp0 + v < n_g ? gp0 + v : n_g - 1;
            const int sh = -(crt_shift(mP, gp, a.cn) + sq);
            sr[v] += ldexp(garner(rr), sh);
            si[v] += ldexp(garner(ri), sh);
        }
    };
    if (isH) {
        segment(0, a.mP[0], a.mQ[0]);
        segment(1, *a.scaled ? a.mP[1] : a.mP[2], a.mQ[1]);
    } else {
        segment(2, a.mP[2], a.mQ[2]);
        segment(3, a.mP[3], a.mQ[3]);
    }
    double2 *out = isH ? a.H : a.S;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int gp = gp0 + v;
        if (gp < n_g && g <= gp) out[(long long)gp * n_g + g] = double2{sr[v], si[v]};
    }
}

int crt_tiles(int n_g, int *nt) {
    *nt = (n_g + CB - 1) / CB;
    return *nt * (*nt + 1) / 2;
}

}  // namespace

size_t crt_residue_bytes(int K, int n_g) {
    const long long groups = (long long)((K + CITEMS * 8 - 1) / (CITEMS * 8)) * CITEMS;
    return (size_t)NMOD * groups * n_g * 16;
}

size_t crt_work_bytes(int n_g) {
    int nt;
    const long long ntri = crt_tiles(n_g, &nt);
    return (size_t)NSEG_ROOM * NMOD * ntri * CFRAG * 64 * sizeof(uint2);
}

hipError_t launch_residue(const SliceJobs &jobs, int K, int n_g, hipStream_t st) {
    const int blocks = (K + CITEMS * 8 - 1) / (CITEMS * 8) * (CITEMS / 2);   // of 16 rows
    hipError_t e = launch_colmax(jobs, K, n_g, st, true);
    if (e != hipSuccess) return e;
    const long long items = (long long)blocks * n_g;
    hipLaunchKernelGGL(k_residue, dim3((unsigned)((items + 255) / 256), NSLICE_SRC), dim3(256), 0,
                       st, jobs, K, n_g, blocks, crt_norm(K));
    return hipGetLastError();
}

hipError_t launch_crt_reduce(int K, int n_g, const SliceView (&hseg)[2][2],
                             const SliceView (&sseg)[2][2], const int *scaled, void *work,
                             double2 *H, double2 *S, hipStream_t st) {
    auto u4 = [](const _Float16 *p) { return reinterpret_cast<const uint4 *>(p); };
    const SliceView *segs[NSEG] = {hseg[0], hseg[1], sseg[0], sseg[1]};
    CrtArgs a;
    CrtRecArgs r;
    for (int s = 0; s < NSEG; ++s) {
        a.P[s] = u4(segs[s][0].S);
        a.Q[s] = u4(segs[s][1].S);
        r.mP[s] = segs[s][0].mx;
        r.mQ[s] = segs[s][1].mx;
    }
    a.scaled = r.scaled = scaled;
    a.out = reinterpret_cast<uint2 *>(work);
    a.n_g = n_g;
    a.groups = (K + CITEMS * 8 - 1) / (CITEMS * 8) * CITEMS;
    a.plane = (long long)a.groups * n_g;
    a.ntri = crt_tiles(n_g, &a.nt);
    a.ntri8 = (a.ntri + 7) / 8 * 8;
    hipLaunchKernelGGL(k_crt_reduce, dim3(a.ntri8, NSEG * NMOD), dim3(CNT), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    r.res = a.out;
    r.H = H;
    r.S = S;
    r.n_g = n_g;
    r.nt = a.nt;
    r.ntri = a.ntri;
    r.cn = crt_norm(K);
    const long long threads = (long long)a.ntri * CFRAG * 64;
    hipLaunchKernelGGL(k_crt_recon, dim3((unsigned)((threads + 255) / 256), 2), dim3(256), 0, st, r);
    return hipGetLastError();
}

}  // namespace hs
