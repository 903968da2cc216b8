"""Accuracy of the small reductions' factor: L against extended precision, and
no further off than the plain column Cholesky in binary64 (one rounding at a
pending element's size per column).

The blocked leaf forms every update as a product of its own before it is
subtracted, so it has fewer roundings at that size, not more. The mean over 12
seeds is compared; one factor's error varies by a fifth, the mean by 0.06.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _cholesky(S, dtype):
    A = S.astype(dtype)
    L = np.zeros_like(A)
    for j in range(len(A)):
        L[j, j] = np.sqrt(A[j, j].real)
        L[j + 1:, j] = A[j + 1:, j] / L[j, j].real
        A[j + 1:, j + 1:] -= np.outer(L[j + 1:, j], L[j + 1:, j].conj())
    return L


def _norm(x):
    return float(np.sqrt((abs(x) ** 2).sum()))


@pytest.mark.parametrize("shift", [0.0, 2.0], ids=["gram", "shifted"])
@pytest.mark.parametrize("N", [16, 40, 100, 128, 200])
def test_factor_no_worse_than_columns(N, shift):
    import torch
    from paper_1611_00606_amd import hs_gep_reduce
    logs = []
    for seed in range(12):
        rng = np.random.default_rng(1000 * seed + N)
        M = rng.standard_normal((N, 2 * N)) + 1j * rng.standard_normal((N, 2 * N))
        S = M @ M.conj().T / (2 * N) + shift * np.eye(N)
        S = (S + S.conj().T) / 2
        print(f"case N={N} shift={shift} seed={seed}", flush=True)
        Sd = torch.from_numpy(S).to("cuda:0")
        L, Ht = torch.empty_like(Sd), torch.empty_like(Sd)
        hs_gep_reduce(Sd, Sd, L, Ht)
        torch.cuda.synchronize()
        ref = _cholesky(S, np.clongdouble)
        plain = _norm(_cholesky(S, np.complex128) - ref)
        logs.append(np.log(_norm(L.cpu().numpy() - ref) / plain))
    print(f"  ratio {np.exp(np.mean(logs)):.3f}", flush=True)
    assert np.mean(logs) <= 0.06
