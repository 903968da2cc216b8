"""The per-atom products add their larger term last.

X_0 = T_AA A + T_AB B with T_AA A = 1 and N_L terms of 2^-54 in T_AB B: summed
before the 1 they are exact, after it each would be lost. H = X_0 + B^H Y is
then exactly 1 + 2 N_L 2^-54.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [0, 1])
@pytest.mark.parametrize("mode", [0, 3], ids=["fp64", "3m"])
@pytest.mark.parametrize("nl", [16, 32, 64, 96, 120])
def test_small_terms_are_not_lost(nl, mode, batch):
    import torch
    from paper_1611_00606_amd import DeviceBuild
    print(f"case N_L={nl} mode={mode} batch={batch}", flush=True)
    A = np.zeros((nl, 1), complex)
    A[0] = 1.0
    B = np.full((nl, 1), 2.0 ** -27, complex)
    T_AB = np.zeros((nl, nl), complex)
    T_AB[0] = 2.0 ** -27
    zero = np.zeros(nl * nl, complex)
    r = DeviceBuild(A, B, np.eye(nl).reshape(-1), T_AB.reshape(-1), zero, np.ones(nl), [nl], 1,
                    mode=mode, batch=batch)
    r.run()
    torch.cuda.synchronize()
    H, _, info = r.results()
    assert H[0, 0] == 1.0 + 2 * nl * 2.0 ** -54 and info[0] == 0
