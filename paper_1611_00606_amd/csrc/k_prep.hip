// Per-atom preparation: the atom tables and the operand forms that do not
// depend on the k-point (k_forms), and the Cholesky of T^AA_a as a launch of
// its own (k_chol) for the resident context, which builds no products at that
// point.
#include <cstring>

#include "prep_atom.h"

namespace hs {

namespace {

// One block per atom of a chunk of up to FORM_CHUNK atoms, whose N_L values
// travel as kernel arguments: nothing is copied from host memory, so the
// enqueue is fully asynchronous and needs no host buffer to outlive the call.
// Each block sums the N_L before its atom itself (a scan by one block took
// 60 us at 512 atoms), writes its table entries and forms
//   M1_a = T^AA_a, M2_a = T^BB_a   Hermitian, from the lower triangles
//   d[r] = 1, d[K + r] = |u_r|^2   per contraction row of the S reduction
// The blocks are spread in y over an atom's elements, FORM_ELEMS each, and in z
// over the two matrices; bound by latency (with one block per atom 20 us at
// N_A = 32, N_L = 49 and 69 us at N_A = 108, N_L = 121; now 10 and 28).
constexpr int FORM_CHUNK = 1024;
constexpr int FORM_THREADS = 256;
constexpr int FORM_ELEMS = 4 * FORM_THREADS;   // elements of a matrix per block
struct FormChunk {
    unsigned char nl[FORM_CHUNK];
    int a0;         // first atom of the chunk
    int row0;       // row offset of the first atom
    int t0;         // T offset of the first atom
    int n_atoms;    // of the build
};

// Elements [e0, e0 + FORM_ELEMS) of the Hermitian n x n block (row-major,
// element (i,k)) from the lower triangle of the stored block t; Im of the
// diagonal dropped.
__device__ __forceinline__ void hermitian_from_lower(const double2 *__restrict__ t, int n,
                                                     int e0, double2 *__restrict__ m) {
    const int e1 = min(n * n, e0 + FORM_ELEMS);
    for (int e = e0 + threadIdx.x; e < e1; e += FORM_THREADS) {
        const int i = e / n, k = e - (e / n) * n;
        double2 v;
        if (k < i) v = t[i * n + k];
        else if (k > i) {
            v = t[k * n + i];
            v.y = -v.y;
        } else {
            v.x = t[i * n + i].x;
            v.y = 0.0;
        }
        m[e] = v;
    }
}

__global__ void __launch_bounds__(FORM_THREADS)
k_forms(FormChunk c, int K, int *__restrict__ row_off, int *__restrict__ t_off,
        const double2 *__restrict__ T_AA, const double2 *__restrict__ T_BB,
        const double2 *__restrict__ U, double2 *__restrict__ M1, double2 *__restrict__ M2,
        double *__restrict__ d) {
    __shared__ int part[2][FORM_THREADS / 64];
    const int i = blockIdx.x, e0 = blockIdx.y * FORM_ELEMS;
    if (e0 >= c.nl[i] * c.nl[i]) return;
    int r = 0, t = 0;
    for (int j = threadIdx.x; j < i; j += FORM_THREADS) {
        r += c.nl[j];
        t += c.nl[j] * c.nl[j];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        r += __shfl_xor(r, o);
        t += __shfl_xor(t, o);
    }
    if ((threadIdx.x & 63) == 0) {
        part[0][threadIdx.x >> 6] = r;
        part[1][threadIdx.x >> 6] = t;
    }
    __syncthreads();
    r = c.row0;
    t = c.t0;
#pragma unroll
    for (int w = 0; w < FORM_THREADS / 64; ++w) {
        r += part[0][w];
        t += part[1][w];
    }
    const int a = c.a0 + i, n = c.nl[i];
    if (blockIdx.z) {
        hermitian_from_lower(T_BB + t, n, e0, M2 + t);
        return;
    }
    hermitian_from_lower(T_AA + t, n, e0, M1 + t);
    if (e0) return;
    if (threadIdx.x == 0) {
        row_off[a] = r;
        t_off[a] = t;
        if (a + 1 == c.n_atoms) {
            row_off[a + 1] = r + n;
            t_off[a + 1] = t + n * n;
        }
    }
    for (int l = threadIdx.x; l < n; l += FORM_THREADS) {
        const double2 u = U[r + l];
        d[r + l] = 1.0;
        d[K + r + l] = u.x * u.x + u.y * u.y;
    }
}

__global__ void __launch_bounds__(CHOL_THREADS)
k_chol(Atoms at, const double2 *__restrict__ T_AA, int *__restrict__ info) {
    __shared__ __align__(16) char lds[CHOL_LDS_BYTES];
    chol_info(at, blockIdx.x, T_AA, info, lds);
}

}  // namespace

hipError_t launch_forms(const AtomPlan &p, const AtomBufs &ab, const double2 *T_AA,
                        const double2 *T_BB, const double2 *U, hipStream_t st) {
    for (int a0 = 0; a0 < p.n_atoms; a0 += FORM_CHUNK) {
        FormChunk c;
        const int n = std::min(FORM_CHUNK, p.n_atoms - a0);
        std::memcpy(c.nl, p.nl.data() + a0, n);
        c.a0 = a0;
        c.row0 = p.row_off[a0];
        c.t0 = p.t_off[a0];
        c.n_atoms = p.n_atoms;
        const int nl = *std::max_element(c.nl, c.nl + n);
        const int ny = (nl * nl + FORM_ELEMS - 1) / FORM_ELEMS;
        hipLaunchKernelGGL(k_forms, dim3(n, ny, 2), dim3(FORM_THREADS), 0, st, c, p.K, ab.tables,
                           ab.tables + p.n_atoms + 1, T_AA, T_BB, U, ab.M1, ab.M2, ab.d);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_chol(const Atoms &at, const double2 *T_AA, int *info, hipStream_t st) {
    hipLaunchKernelGGL(k_chol, dim3(at.n_atoms), dim3(CHOL_THREADS), 0, st, at, T_AA, info);
    return hipGetLastError();
}

}  // namespace hs
