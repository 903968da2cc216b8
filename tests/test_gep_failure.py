"""A reduction that fails half-way leaves nothing unordered (host only).

Each launch, event creation, record and wait of the schedule fails in turn:
whatever was enqueued before, on any stream, has to be ordered before later
work on the caller's stream, which may free or reuse the workspace.
"""

import pytest

import paper_1611_00606_amd as P


# one block of columns; one, two and three steps beside the factorization
@pytest.mark.parametrize("mode", [P.HS_FP64, P.HS_FP64_3M])
@pytest.mark.parametrize("N", [1, 300, 385, 513, 900, 1500, 2200, 4200])
def test_every_failing_call_is_joined(N, mode):
    call = 1
    while True:
        n, report = P.hs_gep_check_failure(N, call, mode)
        if n == -3:
            break
        assert n == 0, (call, report)
        call += 1
    assert call > 5


def test_arguments():
    assert P.hs_gep_check_failure(0, 1)[0] == -1
    assert P.hs_gep_check_failure(2 ** 31 - 1, 1)[0] == -1
    assert P.hs_gep_check_failure(100, 1, P.HS_SPLIT_F16)[0] == -2
    assert P.hs_gep_check_failure(100, 0)[0] == -3
    assert P.hs_gep_check_failure(100, 100000)[0] == -3
