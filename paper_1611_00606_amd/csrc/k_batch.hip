// Batched form of the per-atom stage for atoms of mixed N_L: one persistent
// launch runs every atom's Cholesky (info[a], prep_atom.h) and every atom's
// products
//   X_a = T_AB,a B_a + M1_a^H A_a,   Y_a = T_AB,a^H A_a + M2_a^H B_a
// with the tile shape of each atom's products chosen per N_L (a table filled
// by the autotuner in hs_tune.hip, or the built-in choice below), on the
// per-atom tile engine of zmfma_atom.h.
//
// Work items, taken in order from one atomic counter by a grid of one
// 8-wave block per CU:
//   [0, n_chol)              Cholesky of atom perm[i] (atoms by N_L, largest
//                            first, so the longest factorizations start first)
//   [n_chol, n_chol + 2 nz)  product tiles, atoms in the same order, the X and
//                            the Y tile of the same columns after one another
//                            (they read the same rows of A and B)
// M1, M2 are prepared by k_forms before the launch and no item waits for
// another.
#include "prep_atom.h"
#include "zmfma_atom.h"

namespace hs {

namespace {

constexpr int BT = 512;   // threads of the persistent block (8 waves)

// Candidate tile shapes (BM rows of the atom's N_L x BN columns of N_G):
// 32, 64, 96 or 128 rows by 128 columns, 64 or 96 rows by 192 columns and
// 32 or 64 rows by 256 columns (the wider ones with stages of 8 rows, so
// that two stages fit the LDS). At most nine 16x16 blocks per wave (144
// accumulator registers).
using Cfg0 = AtomCfg<1, 2, 16>;   //  32 x 128
using Cfg1 = AtomCfg<2, 2, 16>;   //  64 x 128
using Cfg2 = AtomCfg<3, 2, 16>;   //  96 x 128
using Cfg3 = AtomCfg<4, 2, 16>;   // 128 x 128
using Cfg4 = AtomCfg<1, 4, 8>;    //  32 x 256
using Cfg5 = AtomCfg<2, 4, 8>;    //  64 x 256
using Cfg6 = AtomCfg<3, 3, 8>;    //  96 x 192
using Cfg7 = AtomCfg<2, 3, 8>;    //  64 x 192
static_assert(Cfg0::NT == BT && Cfg1::NT == BT && Cfg2::NT == BT && Cfg3::NT == BT &&
                  Cfg4::NT == BT && Cfg5::NT == BT && Cfg6::NT == BT && Cfg7::NT == BT,
              "every tile shape runs on the whole persistent block");
static_assert(HS_NUM_TILE_CONFIGS == 8, "tile table and candidate list agree");
static_assert(Cfg0::BM >= ATOM_TILE_MIN_BM && Cfg1::BM >= ATOM_TILE_MIN_BM &&
                  Cfg2::BM >= ATOM_TILE_MIN_BM && Cfg3::BM >= ATOM_TILE_MIN_BM &&
                  Cfg4::BM >= ATOM_TILE_MIN_BM && Cfg5::BM >= ATOM_TILE_MIN_BM &&
                  Cfg6::BM >= ATOM_TILE_MIN_BM && Cfg7::BM >= ATOM_TILE_MIN_BM &&
                  Cfg0::BN >= ATOM_TILE_MIN_BN && Cfg1::BN >= ATOM_TILE_MIN_BN &&
                  Cfg2::BN >= ATOM_TILE_MIN_BN && Cfg3::BN >= ATOM_TILE_MIN_BN &&
                  Cfg4::BN >= ATOM_TILE_MIN_BN && Cfg5::BN >= ATOM_TILE_MIN_BN &&
                  Cfg6::BN >= ATOM_TILE_MIN_BN && Cfg7::BN >= ATOM_TILE_MIN_BN,
              "the tile-position table is sized for these minima");

constexpr int cmax(int a, int b) { return a > b ? a : b; }
constexpr int TILE_LDS = 16 * cmax(cmax(cmax(Cfg0::LDS_ELEMS, Cfg1::LDS_ELEMS),
                                        cmax(Cfg2::LDS_ELEMS, Cfg3::LDS_ELEMS)),
                                   cmax(cmax(Cfg4::LDS_ELEMS, Cfg5::LDS_ELEMS),
                                        cmax(Cfg6::LDS_ELEMS, Cfg7::LDS_ELEMS)));
constexpr int BATCH_LDS = cmax(TILE_LDS, CHOL_LDS_BYTES);
static_assert(BATCH_LDS <= 160 * 1024, "LDS of one CU");

struct BatchArgs {
    Atoms at;
    const double2 *T_AA, *T_AB, *A, *B, *M1, *M2;
    int *info;
    double2 *X, *Y;
    const int *perm;   // [N_A] atom at each position
    const int *tiles;  // [2 nz] atom and tile index within the atom of each product tile
    int *ctrl;         // [0] item counter
    int n_g, nz, n_chol;
    unsigned char cfg[HS_MAX_NL + 1];
};

template <class C>
__device__ __forceinline__ void product_tile(const BatchArgs &args, int which, int r0, int n,
                                             long long t0, int loc, double2 *lds) {
    const int n_g = args.n_g;
    const int ct = (n_g + C::BN - 1) / C::BN;
    const int m0 = (loc / ct) * C::BM;
    const int n0 = (loc % ct) * C::BN;
    const Segs<2, false> tab =
        atom_segs(which, n, n_g, t0, r0, args.A, args.B, args.T_AB, args.M1, args.M2);
    Acc<C> acc;
    ztile_atom<C>(tab, m0, n, n0, n_g, which == 0, acc, lds);
    atom_store<C>(acc, m0, n, n0, n_g, (which == 0 ? args.X : args.Y) + (long long)r0 * n_g);
}

__global__ void __launch_bounds__(BT)
k_batch(BatchArgs args) {
    __shared__ __align__(16) char lds[BATCH_LDS];
    // kind (-1 done, 0 Cholesky, 1 X, 2 Y), atom, tile, and for tiles the
    // atom's first row, N_L and first element of its blocks
    __shared__ int s_job[6];

    const Atoms at = args.at;
    const int nf = args.n_chol;
    const int total = nf + 2 * args.nz;

    // Thread 0 claims and decodes the next item: the counter, then the tile
    // table, then the atom's offsets, so three dependent memory round trips
    // stand between two items.
    for (;;) {
        __syncthreads();   // the previous item is done with LDS and s_job
        if (threadIdx.x == 0) {
            const int it = atomicAdd(args.ctrl, 1);
            int kind = -1, atom = 0, loc = 0, r0 = 0, n = 0, t0 = 0;
            if (it < nf) {
                kind = 0;
                atom = args.perm[it];
            } else if (it < total) {
                const int j = it - nf;
                kind = 1 + (j & 1);
                atom = args.tiles[2 * (j >> 1)];
                loc = args.tiles[2 * (j >> 1) + 1];
                r0 = at.row_off[atom];
                n = at.row_off[atom + 1] - r0;
                t0 = at.t_off[atom];
            }
            s_job[0] = kind;
            s_job[1] = atom;
            s_job[2] = loc;
            s_job[3] = r0;
            s_job[4] = n;
            s_job[5] = t0;
        }
        __syncthreads();
        const int kind = s_job[0], atom = s_job[1], loc = s_job[2];
        if (kind < 0) break;
        if (kind == 0) {
            chol_info(at, atom, args.T_AA, args.info, lds);
            continue;
        }
        const int r0 = s_job[3];
        const int n = s_job[4];
        const long long t0 = s_job[5];
        const int which = kind - 1;
        double2 *tl = reinterpret_cast<double2 *>(lds);
        switch (args.cfg[n]) {
            case 0: product_tile<Cfg0>(args, which, r0, n, t0, loc, tl); break;
            case 1: product_tile<Cfg1>(args, which, r0, n, t0, loc, tl); break;
            case 2: product_tile<Cfg2>(args, which, r0, n, t0, loc, tl); break;
            case 3: product_tile<Cfg3>(args, which, r0, n, t0, loc, tl); break;
            case 4: product_tile<Cfg4>(args, which, r0, n, t0, loc, tl); break;
            case 5: product_tile<Cfg5>(args, which, r0, n, t0, loc, tl); break;
            case 6: product_tile<Cfg6>(args, which, r0, n, t0, loc, tl); break;
            default: product_tile<Cfg7>(args, which, r0, n, t0, loc, tl); break;
        }
    }
}

// Item tables of one launch, written from kernel arguments (no host copy):
// a chunk of up to BT_CHUNK positions per launch; also clears the counter.
constexpr int BT_CHUNK = 256;
struct BatchChunk {
    int perm[BT_CHUNK];
    int zoff[BT_CHUNK];
    int p0, n, last, n_atoms, nz;
};

__global__ void __launch_bounds__(256)
k_batch_tables(BatchChunk c, int *perm, int *zoff, int *ctrl) {
    for (int i = threadIdx.x; i < c.n; i += blockDim.x) {
        perm[c.p0 + i] = c.perm[i];
        zoff[c.p0 + i] = c.zoff[i];
    }
    if (threadIdx.x == 0 && c.p0 == 0) ctrl[0] = 0;
    if (threadIdx.x == 0 && c.last) zoff[c.n_atoms] = c.nz;
}

// Atom and tile index within the atom of every product tile (one block per
// position): the item loop then decodes a tile with one load instead of a
// search over zoff.
__global__ void __launch_bounds__(256) k_batch_tile_index(const int *perm, const int *zoff,
                                                          int *tiles) {
    const int p = blockIdx.x;
    const int atom = perm[p];
    for (int j = zoff[p] + threadIdx.x; j < zoff[p + 1]; j += 256) {
        tiles[2 * j] = atom;
        tiles[2 * j + 1] = j - zoff[p];
    }
}

}  // namespace

// Compute units of the current device (cached per device).
int num_cus() {
    static int cached[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (!cached[dev]) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            n < 1)
            n = 256;
        cached[dev] = n;
    }
    return cached[dev];
}

int tile_shape(int id, int *bm, int *bn) {
    static const int shapes[HS_NUM_TILE_CONFIGS][2] = {
        {Cfg0::BM, Cfg0::BN}, {Cfg1::BM, Cfg1::BN}, {Cfg2::BM, Cfg2::BN},
        {Cfg3::BM, Cfg3::BN}, {Cfg4::BM, Cfg4::BN}, {Cfg5::BM, Cfg5::BN},
        {Cfg6::BM, Cfg6::BN}, {Cfg7::BM, Cfg7::BN}};
    if (id < 0 || id >= HS_NUM_TILE_CONFIGS) return -1;
    if (bm) *bm = shapes[id][0];
    if (bn) *bn = shapes[id][1];
    return 0;
}

// Built-in choice: the tile with the fewest rows that cover N_L (one row
// tile per atom), 128 columns wide except for 96 rows, where 192 columns
// measured faster (2.40 against 2.50 ms for the stage at N_L = 81,
// N_G = 8000).
int default_tile(int nl) {
    return nl <= 32 ? 0 : nl <= 64 ? 1 : nl <= 96 ? 6 : 3;
}

void BatchPlan::make(const AtomPlan &p, int n_g, const unsigned char *cfg_table) {
    for (int v = 0; v <= HS_MAX_NL; ++v) cfg[v] = cfg_table ? cfg_table[v] : (unsigned char)default_tile(v);
    perm.resize(p.n_atoms);
    for (int a = 0; a < p.n_atoms; ++a) perm[a] = a;
    std::stable_sort(perm.begin(), perm.end(),
                     [&](int x, int y) { return p.nl[x] > p.nl[y]; });
    zoff.assign(p.n_atoms + 1, 0);
    long long acc = 0;
    for (int i = 0; i < p.n_atoms; ++i) {
        zoff[i] = (int)acc;
        const int n = p.nl[perm[i]];
        int bm = 0, bn = 0;
        tile_shape(cfg[n], &bm, &bn);
        acc += (long long)((n + bm - 1) / bm) * ((n_g + bn - 1) / bn);
    }
    zoff[p.n_atoms] = (int)acc;
    nz = acc;
}

bool BatchPlan::valid(const AtomPlan &p, const unsigned char *cfg_table) {
    if (!cfg_table) return true;
    for (int a = 0; a < p.n_atoms; ++a)
        if (cfg_table[p.nl[a]] >= HS_NUM_TILE_CONFIGS) return false;
    return true;
}

hipError_t launch_batch(const AtomPlan &p, const Atoms &at, const BatchPlan &bp, int n_g,
                        const BatchIO &io, const BatchBufs &bb, hipStream_t st) {
    if (bp.nz > (1LL << 30) || bp.nz > BatchBufs::max_tiles(p.n_atoms, n_g))
        return hipErrorInvalidValue;
    for (int p0 = 0; p0 < p.n_atoms; p0 += BT_CHUNK) {
        BatchChunk c;
        c.p0 = p0;
        c.n = std::min(BT_CHUNK, p.n_atoms - p0);
        for (int i = 0; i < c.n; ++i) {
            c.perm[i] = bp.perm[p0 + i];
            c.zoff[i] = bp.zoff[p0 + i];
        }
        c.last = p0 + c.n == p.n_atoms;
        c.n_atoms = p.n_atoms;
        c.nz = (int)bp.nz;
        hipLaunchKernelGGL(k_batch_tables, dim3(1), dim3(256), 0, st, c, bb.perm, bb.zoff, bb.ctrl);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_batch_tile_index, dim3(p.n_atoms), dim3(256), 0, st, bb.perm, bb.zoff,
                       bb.tiles);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    BatchArgs a;
    a.at = at;
    a.T_AA = io.T_AA;
    a.T_AB = io.T_AB;
    a.A = io.A;
    a.B = io.B;
    a.M1 = io.M1;
    a.M2 = io.M2;
    a.info = io.info;
    a.X = io.X;
    a.Y = io.Y;
    a.perm = bb.perm;
    a.tiles = bb.tiles;
    a.ctrl = bb.ctrl;
    a.n_g = n_g;
    a.nz = (int)bp.nz;
    a.n_chol = io.info ? p.n_atoms : 0;
    for (int v = 0; v <= HS_MAX_NL; ++v) a.cfg[v] = bp.cfg[v];
    const long long items = a.n_chol + 2 * bp.nz;
    const int grid = (int)std::min<long long>(num_cus(), items);
    hipLaunchKernelGGL(k_batch, dim3(grid), dim3(BT), 0, st, a);
    return hipGetLastError();
}

}  // namespace hs
