"""Every kind of plan of the FP64 reductions, on the device's own unit count.

One or two blocks per compute unit, with all, some or none of the 128-tiles as
such and the rest in 64-tiles, 32-tiles or both: the plan is asked for first,
so that a change of the cost model cannot move a case to another kind unseen.
Outputs are filled with NaN first. Tolerance: 1e-12, the bound of the FP64
parity tests, far above 3 K + 1 < 2^12 roundings of 2^-53.
"""

import numpy as np
import pytest

import oracle
from hs_inputs import make_problem

pytestmark = pytest.mark.gpu

# (blocks per unit, 128-tiles, 64-tiles, 32-tiles) as computed by 256 units
KINDS = {
    "one_all_64": (1740, [64, 65], (1, "all", True, False)),
    "one_none_32": (38, [128] * 15 + [77], (1, "none", False, True)),
    "one_none_64": (741, [129 - 17, 17], (1, "none", True, False)),
    "one_none_both": (963, [100, 100, 100], (1, "none", True, True)),
    "one_some_64": (2184, [64, 65], (1, "some", True, False)),
    "one_some_both": (2332, [125] * 16, (1, "some", True, True)),
    "one_all_both": (2073, [81] * 100, (1, "all", True, True)),
    "two_all_64": (1037, [7], (2, "all", True, False)),
    "two_all_both": (1481, [64, 65], (2, "all", True, True)),
    "two_all_32": (2147, [125] * 16, (2, "all", False, True)),
    "two_none_32": (1074, [100, 100, 99, 1], (2, "none", False, True)),
    "two_none_64": (593, [7], (2, "none", True, False)),
    "two_none_both": (1000, [64, 65], (2, "none", True, True)),
    "two_some_32": (2258, [100, 100, 99, 1], (2, "some", False, True)),
    "two_some_64": (2221, [7], (2, "some", True, False)),
    "two_some_both": (2295, [64, 65], (2, "some", True, True)),
}


@pytest.mark.parametrize("mode", [0, 3], ids=["fp64", "3m"])
@pytest.mark.parametrize("name", list(KINDS))
def test_plan(name, mode):
    import torch
    import paper_1611_00606_amd as P
    n_g, nl, kind = KINDS[name]
    K, low = sum(nl), (n_g // 128) * (n_g // 128 - 1)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    two, n128, n64, n32 = P.hs_check_reduce_plan(K, n_g, P.HS_FP64, cus)[1]
    got = (two, "none" if n128 == 0 else "all" if n128 == low else "some", n64 > 0, n32 > 0)
    assert cus != 256 or got == kind, (got, kind)
    p = make_problem(len(nl), nl, n_g, seed=n_g)
    print(f"case {name} N_G={n_g} K={K} mode={mode} plan {two} {n128} {n64} {n32}", flush=True)
    r = P.DeviceBuild.from_problem(p, mode=mode, batch=1)
    nan = complex(np.nan, np.nan)
    r.H.fill_(nan)
    r.S.fill_(nan)
    r.run()
    torch.cuda.synchronize()
    H, S, info = r.results()
    Hr = oracle.hamiltonian(p.A, p.B, p.T_AA, p.T_AB, p.T_BB, p.nl)
    Sr = oracle.overlap(p.A, p.B, p.U, p.nl)
    assert np.linalg.norm(H - Hr) <= 1e-12 * np.linalg.norm(Hr)
    assert np.linalg.norm(S - Sr) <= 1e-12 * np.linalg.norm(Sr)
    assert np.array_equal(H, H.conj().T) and np.array_equal(S, S.conj().T)
    assert not info.any()
