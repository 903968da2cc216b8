"""The reductions at the edges of their tiles and stages.

H and S are computed in 128, 64 and 32-wide tiles chosen by N_G, over stages
of 8 or 16 contraction rows, and the tiles write both triangles. The sizes
here sit on both sides of every tile width (one tile, a ragged last row, a
diagonal block's quarters, 128-tiles below the diagonal) and the atom sets
give 2K on both sides of whole stages, down to two rows. Outputs are filled
with NaN first, so an element that no tile writes shows.

Tolerance: the 1e-12 relative Frobenius bound of the FP64 parity tests (at
most 3 K + 1 < 2^12 roundings of 2^-53 each, i.e. below 5e-13 in the worst
case of the sizes here).
"""

import numpy as np
import pytest

import oracle
from hs_inputs import make_problem

pytestmark = pytest.mark.gpu

TOL = 1e-12


def _check(nl, n_g, mode, seed, batch=0):
    import torch
    from paper_1611_00606_amd import DeviceBuild
    p = make_problem(len(nl), list(nl), n_g, seed=seed)
    print(f"case N_L={list(nl)} N_G={n_g} mode={mode} batch={batch}", flush=True)
    r = DeviceBuild.from_problem(p, mode=mode, batch=batch)
    nan = complex(np.nan, np.nan)
    r.H.fill_(nan)
    r.S.fill_(nan)
    r.run()
    torch.cuda.synchronize()
    H, S, info = r.results()
    Hr = oracle.hamiltonian(p.A, p.B, p.T_AA, p.T_AB, p.T_BB, p.nl)
    Sr = oracle.overlap(p.A, p.B, p.U, p.nl)
    assert np.linalg.norm(H - Hr) <= TOL * np.linalg.norm(Hr)
    assert np.linalg.norm(S - Sr) <= TOL * np.linalg.norm(Sr)
    assert np.array_equal(H, H.conj().T) and np.array_equal(S, S.conj().T)
    assert not info.any()


@pytest.mark.parametrize("mode", [0, 3], ids=["fp64", "3m"])
@pytest.mark.parametrize("n_g", [1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 192, 193, 255, 257,
                                 319, 385, 641, 1000])
def test_tile_edges(n_g, mode):
    _check([5, 16, 2], n_g, mode, seed=n_g)


@pytest.mark.parametrize("mode", [0, 3], ids=["fp64", "3m"])
@pytest.mark.parametrize("K", [1, 2, 3, 4, 7, 8, 9, 12, 15, 16, 17, 31, 33, 64])
def test_stage_edges(K, mode):
    _check([K], 70, mode, seed=K)
    _check([K], 1500, mode, seed=100 + K, batch=1)


@pytest.mark.parametrize("n_g", [1000, 1301, 1501, 2001])
@pytest.mark.parametrize("K", [63, 64, 65])
def test_two_blocks_per_unit(K, n_g):
    """Sizes that take two blocks per compute unit: halves of 128-tiles, 64-
    and 32-tiles in all of their mixtures."""
    _check([K], n_g, 0, seed=K + n_g, batch=1)


@pytest.mark.parametrize("mode", [1, 2, 4, 5], ids=["f16", "i8", "bf16", "crt"])
@pytest.mark.parametrize("n_g", [1, 31, 33, 64, 65, 97, 129, 500, 1501])
def test_split_tile_edges(n_g, mode):
    """The split forms' whole and half tiles, against their bound of 1e-9 (the
    slices keep 2^-35 of the operand column maxima per term)."""
    import torch
    from paper_1611_00606_amd import DeviceBuild
    nl = [5, 16, 2]
    p = make_problem(len(nl), nl, n_g, seed=n_g)
    print(f"case N_G={n_g} mode={mode}", flush=True)
    r = DeviceBuild.from_problem(p, mode=mode)
    nan = complex(np.nan, np.nan)
    r.H.fill_(nan)
    r.S.fill_(nan)
    r.run()
    torch.cuda.synchronize()
    H, S, _ = r.results()
    Hr = oracle.hamiltonian(p.A, p.B, p.T_AA, p.T_AB, p.T_BB, p.nl)
    Sr = oracle.overlap(p.A, p.B, p.U, p.nl)
    assert np.linalg.norm(H - Hr) <= 1e-9 * np.linalg.norm(Hr)
    assert np.linalg.norm(S - Sr) <= 1e-9 * np.linalg.norm(Sr)
    assert np.array_equal(H, H.conj().T) and np.array_equal(S, S.conj().T)
