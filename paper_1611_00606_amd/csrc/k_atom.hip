// Per-atom products, as complex MFMA tiles:
//   X_a = T^AB_a B_a + T^AA_a A_a = T_AB,a B_a + M1_a^H A_a
//   Y_a = T^BA_a A_a + T^BB_a B_a = T_AB,a^H A_a + M2_a^H B_a
// with M1, M2 the Hermitian T^AA_a, T^BB_a prepared by k_forms, so that
// H = A^H X + B^H Y. (Alg. 1's Z_a, Y_a and X_a take 20 N_L^2 N_G real
// operations per atom against 32 here, but its H contracts over 3K rows
// instead of 2K: 4 K N_G^2 operations saved for 12 K N_L N_G. That is fewer from
// N_G = 3 N_L on, in FP64; below, and to several times that where the reductions
// run on INT8, it is more. One form serves all sizes nevertheless: it needs no
// factor before the products, and against the 3K form with its separate
// Cholesky no build was slower (us, before and now: 100 atoms of 121, N_G = 128
// FP64 17317 and 1494, modular 868 and 643, N_G = 363 17666 and 1769, 1180 and
// 1016; the least gain, INT8 at N_G = 1000, 3592 and 3557).)
//
// Each block computes a BM x BN tile of one atom's N_L x N_G output (one
// tile covers all of an atom's rows, BM >= N_L); the contraction runs over
// the atom's N_L rows twice. Blocks are ordered so that the X and the Y tile
// of the same columns, which read the same rows of A and B, are neighbours.
// The first n_chol blocks run the Cholesky of T^AA_a (info[a]) instead: a
// serial chain of N_L columns that nothing else waits for, hidden beside the
// products.
#include "hs_internal.h"
#include "prep_atom.h"
#include "zmfma_atom.h"

namespace hs {

namespace {

// Blocks in a row of the grid: a dimension of it holds fewer than 2^32 threads,
// and millions of light atoms, or tens of thousands at a large N_G, make more.
constexpr int GRID_ROW = 1 << 22;

template <class C>
__global__ void __launch_bounds__(C::NT)
k_atom(Atoms at, int n_g, int mtiles, int ctiles, int n_chol, const double2 *__restrict__ A,
       const double2 *__restrict__ B, const double2 *__restrict__ T_AA,
       const double2 *__restrict__ T_AB, const double2 *__restrict__ M1,
       const double2 *__restrict__ M2, int *__restrict__ info, double2 *__restrict__ X,
       double2 *__restrict__ Y) {
    static_assert(C::NT == CHOL_THREADS && C::LDS_ELEMS * 16 >= CHOL_LDS_BYTES, "shared block");
    __shared__ double2 lds[C::LDS_ELEMS];

    int b = blockIdx.y * GRID_ROW + blockIdx.x;
    if (b < n_chol) {
        chol_info(at, b, T_AA, info, reinterpret_cast<char *>(lds));
        return;
    }
    b -= n_chol;
    const int which = b & 1;  // 0: X, 1: Y
    b >>= 1;
    const int ct = b % ctiles;
    b /= ctiles;
    const int a = b / mtiles;
    const int mt = b % mtiles;
    if (a >= at.n_atoms) return;   // the last row of the grid
    const int r0 = at.row_off[a];
    const int n = at.row_off[a + 1] - r0;
    const int m0 = mt * C::BM;
    if (m0 >= n) return;  // atom has fewer rows than this row tile (mixed N_L)
    const int n0 = ct * C::BN;
    const Segs<2, false> tab = atom_segs(which, n, n_g, at.t_off[a], r0, A, B, T_AB, M1, M2);
    Acc<C> acc;
    ztile_atom<C>(tab, m0, n, n0, n_g, which == 0, acc, lds);
    atom_store<C>(acc, m0, n, n0, n_g, (which == 0 ? X : Y) + (long long)r0 * n_g);
}

template <class C>
hipError_t launch_atom_cfg(const Atoms &at, int n_g, const double2 *A, const double2 *B,
                           const double2 *T_AA, const double2 *T_AB, const double2 *M1,
                           const double2 *M2, int *info, double2 *X, double2 *Y, hipStream_t st) {
    const int mtiles = (at.max_nl + C::BM - 1) / C::BM;
    const int ctiles = (n_g + C::BN - 1) / C::BN;
    const int n_chol = info ? at.n_atoms : 0;
    const long long blocks = n_chol + 2LL * ctiles * mtiles * at.n_atoms;
    if (blocks > (1LL << 30)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)std::min<long long>(blocks, GRID_ROW),
                    (unsigned)((blocks + GRID_ROW - 1) / GRID_ROW));
    hipLaunchKernelGGL(k_atom<C>, grid, dim3(C::NT), 0, st, at, n_g, mtiles, ctiles, n_chol, A, B,
                       T_AA, T_AB, M1, M2, info, X, Y);
    return hipGetLastError();
}

}  // namespace

// Row tile of 32, 64, 96 or 128 (the smallest that covers the largest N_L),
// 128 columns (192 for the 96-row tile, as in the batched launch's
// built-in choice).
hipError_t launch_atom(const Atoms &at, int n_g, const double2 *A, const double2 *B,
                       const double2 *T_AA, const double2 *T_AB, const double2 *M1,
                       const double2 *M2, int *info, double2 *X, double2 *Y, hipStream_t st) {
    if (at.max_nl <= 32)
        return launch_atom_cfg<AtomCfg<1, 2, 16>>(at, n_g, A, B, T_AA, T_AB, M1, M2, info, X, Y, st);
    if (at.max_nl <= 64)
        return launch_atom_cfg<AtomCfg<2, 2, 16>>(at, n_g, A, B, T_AA, T_AB, M1, M2, info, X, Y, st);
    if (at.max_nl <= 96)
        return launch_atom_cfg<AtomCfg<3, 3, 8>>(at, n_g, A, B, T_AA, T_AB, M1, M2, info, X, Y, st);
    return launch_atom_cfg<AtomCfg<4, 2, 16>>(at, n_g, A, B, T_AA, T_AB, M1, M2, info, X, Y, st);
}

}  // namespace hs
