"""The eigenproblem reduction at the edges of its tile shapes.

Each product launch takes 128, 64 or 32-wide tiles by an estimate of its time,
so these sizes reach every shape, in both result forms (Ht in one block up to
three panels, in steps of columns from four on) and both arithmetics: a last
block of 1, 31, 33, 63, 65 and 127 rows, one block, sizes whose panels and
inverse levels take different shapes, and every pattern of one to three steps
beside and after the factorization. Tolerance: the 1e-12 bound of the
reduction's parity tests (cond(S) u sqrt(N) is about 1e-13 here).
"""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 3], ids=["fp64", "3m"])
@pytest.mark.parametrize("N", [31, 97, 128, 160, 191, 383, 512, 545, 895, 1281, 2499, 2531])
def test_gep_tile_edges(N, mode):
    _check(N, mode)


@pytest.mark.parametrize("N", [384, 385, 513, 641, 896, 897, 1024, 1025, 1411, 1920, 2241, 3295])
def test_gep_steps(N):
    _check(N, 0)


def _check(N, mode):
    import torch
    from paper_1611_00606_amd import hs_gep_reduce
    rng = np.random.default_rng(N)
    X = rng.standard_normal((N, N)) + 1j * rng.standard_normal((N, N))
    S = X @ X.conj().T / (2 * N) + np.eye(N)
    S = (S + S.conj().T) / 2
    H = rng.standard_normal((N, N)) + 1j * rng.standard_normal((N, N))
    H = (H + H.conj().T) / 2
    print(f"case N={N} mode={mode}", flush=True)
    Hd, Sd = (torch.from_numpy(x).to("cuda:0") for x in (H, S))
    L = torch.full_like(Hd, complex(np.nan, np.nan))
    Ht = L.clone()
    info = torch.full((1,), -7, dtype=torch.int32, device="cuda:0")
    hs_gep_reduce(Hd, Sd, L, Ht, info=info, mode=mode)
    torch.cuda.synchronize()
    L0, Ht0, inf0 = oracle.gep_reduce(H, S)
    L, Ht = L.cpu().numpy(), Ht.cpu().numpy()
    assert int(info.item()) == 0 == inf0
    assert np.linalg.norm(L - L0) <= 1e-12 * np.linalg.norm(L0)
    assert np.linalg.norm(Ht - Ht0) <= 1e-12 * np.linalg.norm(Ht0)
    assert np.array_equal(Ht, Ht.conj().T) and not np.triu(L, 1).any()
