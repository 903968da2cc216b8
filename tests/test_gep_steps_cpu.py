"""Steps of the eigenproblem reduction: one source for the library and the
operation counts, and what the launches rely on (host only)."""

import pytest

import paper_1611_00606_amd as P
from paper_1611_00606_amd.flops import gep_executed_flops, gep_steps

SIZES = list(range(1, 3000, 7)) + list(range(3000, 17000, 331))


def test_counts_use_the_librarys_steps():
    for N in SIZES:
        assert gep_steps(N) == P.hs_gep_steps(N)


def test_steps_cover_the_columns_in_few_blocks():
    """Steps end at multiples of 128 columns (the last at N), ascend, and hold at
    most eight blocks of 128: four nodes of one depth of their recursion, as
    many rectangles as a launch takes."""
    for N in SIZES:
        ends = P.hs_gep_steps(N)
        assert ends[-1] == N and all(e % 128 == 0 for e in ends[:-1])
        assert len(ends) == 1 or N > 384
        for a, b in zip([0] + ends, ends):
            assert 0 < b - a <= 1024
    assert all(len(P.hs_gep_steps(N)) >= 2 for N in SIZES if N > 384)


def test_executed_count():
    """One block: N^3/6 + 5/6 N^3 complex multiply-adds; many: towards 16/3 N^3."""
    assert gep_executed_flops(300) == pytest.approx(8 * 300 ** 3)
    assert 16 / 3 < gep_executed_flops(16000) / 16000 ** 3 < 5.6


def test_arguments():
    with pytest.raises(ValueError):
        P.hs_gep_steps(0)
