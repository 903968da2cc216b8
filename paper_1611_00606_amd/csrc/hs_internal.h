// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <string>
#include <vector>

#include "../../include/hs_build.h"

namespace hs {

// Consecutive blocks of a launch go to the 8 XCDs in turn. Of n items (H's
// `first` ones, then S's) XCD x takes a contiguous run of H's and one of S's,
// H's before S's, so that the blocks resident on one XCD share operand panels
// through its L2 and all XCDs work on the same output; every XCD gets n / 8
// items, up to rounding.
__host__ __device__ inline int xcd_blocks(int n) { return (n + 7) / 8 * 8; }
// Item of block b < xcd_blocks(n), or -1. XCD x takes the blocks' range [c0, c1)
// of n; of every prefix c of it H's share is floor(c nf / n), which grows by at
// most one per block, so that the ranges of H and of S fit into the blocks for
// any n and `first`.
__host__ __device__ __forceinline__ int xcd_item(int b, int n, int first) {
    const long long x = b % 8;
    const int i = b / 8;
    const int c0 = (int)(x * n / 8), c1 = (int)((x + 1) * n / 8);
    if (i >= c1 - c0) return -1;
    if (n <= first) return c0 + i;
    const int h0 = (int)((long long)c0 * first / n), h1 = (int)((long long)c1 * first / n);
    return i < h1 - h0 ? h0 + i : first + (c0 - h0) + i - (h1 - h0);
}

// Device-side description of the atoms of one build.
struct Atoms {
    const int *row_off;  // [N_A+1] first row of each atom in A, B, U, X, Y
    const int *t_off;    // [N_A+1] first element of each atom's N_L x N_L block
    int n_atoms;
    int max_nl;
    int K;               // total rows
};

struct AtomPlan;
struct AtomBufs;

// Atom tables and the operand forms of the per-atom products (k_prep.hip):
//   M1_a      T_AA,a as a full Hermitian matrix from its lower triangle
//   M2_a      T_BB,a likewise
//   d[2K]     per contraction row of the S reduction (A rows, then B rows):
//             d[r] = 1, d[K + r] = |U[r]|^2
hipError_t launch_forms(const AtomPlan &p, const AtomBufs &ab, const double2 *T_AA,
                        const double2 *T_BB, const double2 *U, hipStream_t st);
// info[a]: 0 or the 1-based failing pivot of T_AA,a's Cholesky (Alg. 1's try
// step), as a launch of its own; the product launches below run it beside
// the products.
hipError_t launch_chol(const Atoms &at, const double2 *T_AA, int *info, hipStream_t st);

// Per-atom products:
//   X_a = T^AB_a B_a + T^AA_a A_a = T_AB,a B_a + M1_a^H A_a
//   Y_a = T^BA_a A_a + T^BB_a B_a = T_AB,a^H A_a + M2_a^H B_a
// and, when info is not NULL, the Cholesky of T_AA,a into info[a].
hipError_t launch_atom(const Atoms &at, int n_g, const double2 *A, const double2 *B,
                       const double2 *T_AA, const double2 *T_AB, const double2 *M1,
                       const double2 *M2, int *info, double2 *X, double2 *Y, hipStream_t st);

// Large reductions H = A^H X + B^H Y, S = A^H A + B^H |U|^2 B, both triangles
// (complex FP64 MFMA; g3: 3 real products per complex product instead of 4).
hipError_t launch_reduce(int K, int n_g, const double2 *A, const double2 *B,
                         const double2 *X, const double2 *Y, const double *d,
                         double2 *H, double2 *S, hipStream_t st, bool g3);

// Host-only checks of the tiles that a reduction's blocks compute on a device
// of `cus` compute units: the number of cells of the lower triangles of H and S
// that are not computed exactly once. plan: blocks per compute unit, 128-tiles,
// 64-tiles, 64-tiles computed as 32-tiles; 1, whole tiles, half tiles, 0.
int reduce_check_plan(int K, int n_g, bool g3, int cus, int plan[4]);
int split_check_plan(int n_g, int cus, int plan[4]);
// How often each h x w cell on or below the diagonal of H and of S is computed.
struct CellCount {
    int n, h, w, nr, nc;
    std::vector<unsigned char> count;   // saturates at 2
    CellCount(int n_g, int h_, int w_)
        : n(n_g), h(h_), w(w_), nr((n_g + h_ - 1) / h_), nc((n_g + w_ - 1) / w_),
          count(2 * (size_t)nr * nc, 0) {}
    void add(bool isH, int m0, int n0, int rows, int cols) {
        for (int r = m0 / h; r < (m0 + rows) / h && r < nr; ++r)
            for (int c = n0 / w; c < (n0 + cols) / w && c < nc; ++c) {
                unsigned char &x = count[((isH ? 0 : (size_t)nr) + r) * nc + c];
                if (x < 2) ++x;
            }
    }
    int wrong() const {
        int bad = 0;
        for (int r = 0; r < 2 * nr; ++r)
            for (int c = 0; c < nc && c * w < std::min(n, (r % nr + 1) * h); ++c)
                bad += count[(size_t)r * nc + c] != 1;
        return bad;
    }
};

// Error bookkeeping shared by the C entry points (thread-local message).
void set_error(int status, const std::string &msg);
const char *message_for(int status);   // the last message if it explains `status`, else NULL
int hip_fail(hipError_t e, const char *where);   // records the message, returns HS_ERR_HIP
int check_device();                              // HS_OK on gfx950, else an error status
int num_cus();                                   // compute units of the current device
inline bool valid_mode(int mode) {   // HS_FP64 .. HS_SPLIT_I8_CRT
    return mode == HS_FP64 || mode == HS_SPLIT_F16 || mode == HS_SPLIT_I8 || mode == HS_FP64_3M ||
           mode == HS_SPLIT_BF16 || mode == HS_SPLIT_I8_CRT;
}
inline bool split_mode(int mode) {   // the operands are sliced (or cut into residues)
    return mode == HS_SPLIT_F16 || mode == HS_SPLIT_I8 || mode == HS_SPLIT_BF16 ||
           mode == HS_SPLIT_I8_CRT;
}

// Split-precision reductions (k_split.hip). The sliced operands, from the
// matrices M[0..3] = A, B, X, Y [K][N_G]: 0 A, 1 B, 2 X 2^-e, 3 Y, 4 the rows
// of B scaled by sqrt(rscale[k]), 5 A 2^e, with e[k] per row (slice_row_exp;
// where A and X need no balance e = 0 and operand 0 stands for 5, which is not
// written); for each the column maxima mx [N_G] (bit patterns of doubles; block norms in
// the modular form) and the FP16 slices S [4][groups][N_G][8], groups = 4 * ceil(K / 16).
// Every pass takes all of them in one launch and reads each matrix once.
constexpr int NSLICE_SRC = 4;
constexpr int NSPLIT = 6;
struct SliceJobs {
    const double2 *M[NSLICE_SRC];
    const double *rscale;
    unsigned long long *mx[NSPLIT];
    _Float16 *S[NSPLIT];
    // scratch, one entry per rgroup rows: upper halves of the largest |Re| or
    // |Im| of A's rows and of X's
    unsigned *rmx[2];
    int rgroup;
    int *scaled;   // whether rows are scaled (written by launch_colmax)
};
struct SliceView {
    const _Float16 *S;
    const unsigned long long *mx;
};
// The reductions' (A 2^e, X 2^-e) takes hseg[1][0] if *scaled, else sseg[0][0] = A.
size_t split_slice_bytes(int K, int n_g);
// zero every mx and rmx, then A's and X's row maxima and the column maxima
// into them; norm: instead of the maxima the largest Euclidean norm of 64 rows
// of each column
hipError_t launch_colmax(const SliceJobs &jobs, int K, int n_g, hipStream_t st, bool norm);
// column maxima and slices; bf16: the same slices held as BF16 and multiplied
// on BF16 MFMA
hipError_t launch_slice(const SliceJobs &jobs, int K, int n_g, hipStream_t st, bool bf16);
// H segments (B,Y), (A 2^e, X 2^-e); S segments (A,A), (Bs,Bs): [segment][P or Q]
hipError_t launch_split_reduce(int K, int n_g, const SliceView (&hseg)[2][2],
                               const SliceView (&sseg)[2][2], const int *scaled, double2 *H,
                               double2 *S, hipStream_t st, bool bf16);
// INT8 form: slices S8 [5][groups][N_G][16 int8], groups = 4 * ceil(K / 32);
// same column maxima and segments as the FP16 form.
size_t split8_slice_bytes(int K, int n_g);
hipError_t launch_slice8(const SliceJobs &jobs, int K, int n_g, hipStream_t st);
hipError_t launch_split8_reduce(int K, int n_g, const SliceView (&hseg)[2][2],
                                const SliceView (&sseg)[2][2], const int *scaled, double2 *H,
                                double2 *S, hipStream_t st);
// Modular INT8 form (k_crt.hip): residues R [NMOD][groups][N_G][16 int8],
// groups = 8 * ceil(K / 64) (of 64 rows four hold the real parts of 16 rows
// each, four the imaginary parts), of each operand's integers; the
// reduction writes each segment's residues into `work` (crt_work_bytes) and
// rebuilds H and S from them.
size_t crt_residue_bytes(int K, int n_g);
size_t crt_work_bytes(int n_g);
hipError_t launch_residue(const SliceJobs &jobs, int K, int n_g, hipStream_t st);
hipError_t launch_crt_reduce(int K, int n_g, const SliceView (&hseg)[2][2],
                             const SliceView (&sseg)[2][2], const int *scaled, void *work,
                             double2 *H, double2 *S, hipStream_t st);
inline size_t slice_bytes(int mode, int K, int n_g) {
    if (mode == HS_SPLIT_I8_CRT) return crt_residue_bytes(K, n_g);
    return mode == HS_SPLIT_I8 ? split8_slice_bytes(K, n_g) : split_slice_bytes(K, n_g);
}
// upper := conj(lower), Im(diag) := 0 for both outputs (launch_mirror1: one matrix)
hipError_t launch_mirror(double2 *H, double2 *S, int n_g, hipStream_t st);
hipError_t launch_mirror1(double2 *M, int n, hipStream_t st);

// Generalized eigenproblem reduction (k_gep.hip): S = L L^H, Ht = L^-1 H L^-H.
// info: device int or NULL (a workspace slot is used then); g3: the large
// products in the 3M form.
size_t gep_workspace_bytes(int N);
std::vector<int> gep_steps(int N);   // column ends of the steps
hipError_t launch_gep(const double2 *H, const double2 *S, int N, double2 *L, double2 *Ht,
                      int *info, char *ws, hipStream_t st, bool g3);
// Runs launch_gep's orchestration without issuing anything and checks that
// every pair of launches on different streams that touch a common 128 x 128
// cell of a matrix (one writing) is ordered; returns the number of pairs
// that are not (-1 if the orchestration failed), describing a few in report.
int gep_check_schedule(int N, bool g3, int drop_tag, std::string &report);
// The same with the call-th launch or event call (from 1) failing: the pairs,
// and the launches that the caller's stream is not ordered after when
// launch_gep returns; -1 if there is no such call.
int gep_check_failure(int N, bool g3, int call, std::string &report);

// ---------------------------------------------------------------------------
// Host-side plan of one atom set and the enqueue steps shared by the one-shot
// build (hs_build_ex) and the resident context (hs_ctx).

// Atom-side sizes and offsets (host copy).
struct AtomPlan {
    int n_atoms = 0, K = 0, max_nl = 0;
    long long t_total = 0;
    std::vector<int> row_off, t_off;      // [N_A+1] each
    std::vector<unsigned char> nl;        // [N_A]
    // Returns 0, or -8 for an invalid N_L (per-atom entries included).
    int make(int N_A, const int32_t *nl_per_atom, int N_L);
    // Device bytes of the k-independent buffers (AtomBufs).
    size_t atom_bytes() const;
    // Device bytes of the per-k-point buffers for N_G (X, Y; plus the
    // sliced operands in the split-precision mode).
    size_t kpoint_bytes(int n_g, int mode = 0) const;
};

// k-independent device buffers of an atom set, carved from one allocation.
struct AtomBufs {
    int *tables;      // row_off [N_A+1], then t_off [N_A+1]
    int *info;        // [N_A]
    double *d;        // [2K]
    double2 *M1;      // [t_total] Hermitian T_AA
    double2 *M2;      // [t_total] Hermitian T_BB
    void carve(const AtomPlan &p, char *base);
    Atoms atoms(const AtomPlan &p) const;
};

// Batched per-atom stage (k_batch.hip): item tables of one launch.
// Every tile shape has at least ATOM_TILE_MIN_BM rows and ATOM_TILE_MIN_BN
// columns, which bounds the product tiles per atom (and so the tile table).
constexpr int ATOM_TILE_MIN_BM = 32, ATOM_TILE_MIN_BN = 128;
struct BatchBufs {
    int *perm;    // [N_A]
    int *zoff;    // [N_A + 1]
    int *ctrl;    // [2] item counter; after the stage: SliceJobs.scaled
    int *tiles;   // [2 max_tiles(N_A, N_G)] atom, tile within the atom of each product tile
    static long long max_tiles(int n_atoms, int n_g);
    static size_t bytes(int n_atoms, int n_g);
    void carve(int n_atoms, char *base);   // tiles last
};
// Host plan: tile shape per N_L, atom order (N_L descending) and the first
// product tile of each position.
struct BatchPlan {
    unsigned char cfg[HS_MAX_NL + 1];
    std::vector<int> perm, zoff;
    long long nz = 0;   // product tiles per product (Z or W)
    // cfg_table: [HS_MAX_NL + 1] tile id per N_L, or NULL for default_tile
    void make(const AtomPlan &p, int n_g, const unsigned char *cfg_table);
    // every N_L of the plan maps to an existing tile id
    static bool valid(const AtomPlan &p, const unsigned char *cfg_table);
};
struct BatchIO {
    const double2 *T_AA, *T_AB, *A, *B, *M1, *M2;
    int *info;   // NULL: products only
    double2 *X, *Y;
};
int tile_shape(int id, int *bm, int *bn);   // 0, or -1 for an unknown id
int default_tile(int nl);
// Persistent launch of the per-atom stage.
hipError_t launch_batch(const AtomPlan &p, const Atoms &at, const BatchPlan &bp, int n_g,
                        const BatchIO &io, const BatchBufs &bb, hipStream_t st);

// Per-k-point device buffers.
struct KpointBufs {
    double2 *X, *Y;   // [K][N_G] each
    _Float16 *sl[NSPLIT];
    unsigned long long *mx[NSPLIT];
    void *crt;        // segment residues of the modular form (else NULL)
    BatchBufs batch;
    void carve(const AtomPlan &p, int n_g, int mode, char *base);
};

// How the per-atom products of one build run: one launch with a tile shape
// for all atoms (batch = false), or the persistent batched launch with the
// tile table cfg; info: where the Cholesky of T_AA reports, or NULL when it
// has been run already (the resident context).
struct AtomStage {
    bool batch = false;
    const unsigned char *cfg = nullptr;   // [HS_MAX_NL + 1] or NULL
    const double2 *T_AA = nullptr;
    int *info = nullptr;
};

// Per-atom products and the reductions for one k-point. ev: optional phase
// events [1..4] as in hs_options.phase_events (ev[0] is recorded by the caller).
hipError_t enqueue_kpoint(const AtomPlan &p, const AtomBufs &ab, int n_g, int mode,
                          const double2 *A, const double2 *B, const double2 *T_AB,
                          const KpointBufs &kb, double2 *H, double2 *S, hipStream_t st,
                          const hipEvent_t *ev, const AtomStage &stage = AtomStage());

// Argument checks shared by the one-shot entry points (hs_build's argument
// order; per_atom: N_L comes from a per-atom table and is not checked here).
int check_build_args(const hs_complex *A, const hs_complex *B, const hs_complex *T_AA,
                     const hs_complex *T_AB, const hs_complex *T_BB, const hs_complex *U,
                     int N_A, int N_L, int N_G, const hs_complex *H, const hs_complex *S,
                     bool per_atom);
// One-shot build on stream st with the workspace ws (atom part, then
// k-point part; p.atom_bytes() + p.kpoint_bytes(n_g, mode) bytes). Returns
// HS_OK or a status; enqueues only.
int run_build(const AtomPlan &p, int n_g, int mode, const hs_complex *A, const hs_complex *B,
              const hs_complex *T_AA, const hs_complex *T_AB, const hs_complex *T_BB,
              const hs_complex *U, hs_complex *H, hs_complex *S, char *ws, int32_t *info_user,
              hipStream_t st, void **events, bool batch, const hs_tuning *tuning);

}  // namespace hs
