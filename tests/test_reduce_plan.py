"""Every tile of H and S is computed exactly once (host only).

The reductions' blocks find their tiles from the launch's plan alone;
hs_check_reduce_plan walks them on the host and counts each cell of the two lower
triangles. The plans depend on the compute-unit count: 256 on an MI355X, 128,
64 or 32 in its partitions; counts that are no multiple of 8 exist on no such
device and must be safe all the same.
"""

import os
import subprocess

import pytest

import paper_1611_00606_amd as P

SIZES = [1, 31, 32, 33, 64, 65, 127, 128, 129, 256, 300, 385, 500, 641, 1000, 1301, 1501, 2000,
         2224, 2251, 2261, 2301, 2500, 3001, 3275, 3893, 4100, 6000]


@pytest.mark.parametrize("cus", [256, 128, 64, 32, 304, 100, 250, 7, 1])
@pytest.mark.parametrize("mode", [P.HS_FP64, P.HS_FP64_3M, P.HS_SPLIT_F16], ids=["fp64", "3m", "f16"])
def test_every_cell_once(mode, cus):
    for n_g in SIZES:
        for K in ((1, 300, 8100) if mode in (P.HS_FP64, P.HS_FP64_3M) else (1,)):
            wrong, plan = P.hs_check_reduce_plan(K, n_g, mode, cus)
            assert wrong == 0, (n_g, K, plan)


def test_every_kind_of_plan_is_seen():
    """FP64: one or two blocks per unit; all, some or none of the 128-tiles as
    such; 64- and 32-tiles, one or both. FP16: whole, halves, both."""
    seen = set()
    for n_g in SIZES + [8000]:
        nf = n_g // 128
        for K in (1, 300, 2000, 8100):
            two, n128, n64, n32 = P.hs_check_reduce_plan(K, n_g)[1]
            low = nf * (nf - 1)
            part = "none" if n128 == 0 else "all" if n128 == low else "some"
            seen.add((two, part, n64 > 0, n32 > 0))
    assert {(t, p) for t, p, _, _ in seen} >= {(1, "all"), (1, "some"), (2, "none"), (2, "some"),
                                               (2, "all")}
    assert {(a, b) for _, _, a, b in seen} >= {(True, False), (False, True), (True, True)}
    kinds = {(w > 0, h > 0) for w, h in
             (P.hs_check_reduce_plan(1, n, P.HS_SPLIT_F16)[1][1:3] for n in SIZES)}
    assert kinds == {(True, False), (False, True), (True, True)}


def test_xcd_order_is_a_permutation(tmp_path):
    """For any number of items and any number of H's among them."""
    clang = "/opt/rocm/llvm/bin/clang++"
    if not os.path.exists(clang):
        pytest.skip("no host compiler with the HIP headers")
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "xcd_item_check.cpp")
    exe = str(tmp_path / "xcd_item_check")
    subprocess.run([clang, "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    src, "-o", exe], check=True)
    assert subprocess.run([exe], capture_output=True, text=True, check=True).stdout == "0\n"


def test_arguments():
    assert P.hs_check_reduce_plan(0, 10)[0] == -1
    assert P.hs_check_reduce_plan(10, 0)[0] == -2
    assert P.hs_check_reduce_plan(10, 10, P.HS_SPLIT_I8)[0] == -3
    assert P.hs_check_reduce_plan(10, 10, P.HS_FP64, 0)[0] == -4
    assert P.hs_check_reduce_plan(10, 2 ** 31 - 1)[0] == -2
    assert P.hs_check_reduce_plan(2 ** 31 - 1, 10)[0] == -1
