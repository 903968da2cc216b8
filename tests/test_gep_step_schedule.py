"""Race check of the eigenproblem reduction's schedule over its step patterns
(host only).

From four panels of 128 columns on the first steps of columns run beside the
factorization: one, two or three of them and more, a step's last panel the first
or the second of its pair, the last step ragged, and at N = 2500 the compute units
they may take change. The wait sites are those of hs_gep_check_schedule: 1 the first
S21^H after the preparation, 2 the first panel product after it, 3 the next
column blocks after the previous bulk update, 4 L21 and the bulk update after the
panel product, 5 the factorization's join of the lookahead stream, 7 a background
step after its last panel, 8 the same after the lookahead stream's reads, 9 the
first step after the factorization after the background's last inverse, 10 the
end after the background's products.
"""

import pytest

import paper_1611_00606_amd as P


def _beside(N):
    """Steps beside the factorization: up to max(min(0.68 N, 1280), 0.32 N) columns."""
    bg = int(max(min(0.68 * N, 1280.0), 0.32 * N) / 128 + 0.5) * 128
    return [e for e in P.hs_gep_steps(N) if e <= bg]


def test_no_race_at_any_size():
    sizes = list(range(385, 3400, 7)) + [4095, 4096, 5003, 6000, 8000, 9273, 12000]
    patterns = set()
    for N in sizes:
        for mode in (P.HS_FP64, P.HS_FP64_3M):
            n, report = P.hs_gep_check_schedule(N, mode)
            assert n == 0, (N, report)
        b = _beside(N)
        patterns |= {(len(b), (e // 128) % 2) for e in b}
    # one to three steps, forks after the first and after the second panel of a pair
    assert patterns >= {(k, odd) for k in (1, 2, 3) for odd in (0, 1)}


@pytest.mark.parametrize("N", [513, 700, 1000, 1500, 2499, 2600, 6000])
@pytest.mark.parametrize("site", [1, 2, 3, 4, 5, 7, 8, 9, 10])
def test_each_wait_is_needed(N, site):
    assert P.hs_gep_check_schedule(N, P.HS_FP64, drop_wait=site)[0] > 0
