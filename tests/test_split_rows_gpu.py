"""The split forms' errors against those of Alg. 1's operands, cut.

Operands are cut relative to their columns, so an unbalanced pair of operands
(all of T_AA in X, none in A) loses digits that Alg. 1's Cholesky factors, which
share T_AA evenly, keep: atoms and rows of unlike magnitude in T_AA. The bound
is the error of Alg. 1's own operands cut at a power of two per column. The
library's row exponents are whole numbers, which leaves a row up to 2^(1/2) above
balance in either operand: a factor 2. Over ordinary problems, where nothing is
unbalanced, the geometric mean of the ratio is held to 1.
"""

import numpy as np
import pytest

import oracle as O
from _split_model import alg1_error, overlap_error
from hs_inputs import make_problem

pytestmark = pytest.mark.gpu

BALANCE = 2.0


def _atom_x1000(seed, n_g=100):
    """One atom's T_AA a thousand times the others'."""
    p = make_problem(64, 20, n_g, seed=seed)
    p.set_t_block("T_AA", 5, 1e3 * p.t_block("T_AA", 5))
    return p


def _unlike_rows(seed, fail_atoms=None):
    """T_AA = D T D and A = D^-1 A', D over four decades within each atom."""
    p = make_problem(64, 20, 100, seed=seed, fail_atoms=fail_atoms)
    rng = np.random.default_rng(seed)
    off = p.row_offsets()
    for a in range(p.N_A):
        d = 10.0 ** rng.uniform(-2, 2, int(p.nl[a]))
        p.set_t_block("T_AA", a, d[:, None] * p.t_block("T_AA", a) * d[None, :])
        p.A[off[a]:off[a + 1]] /= d[:, None]
    return p


def _zero_rows(seed):
    """Unlike rows; A is zero on some rows, T_AA and T_AB on others (X zero)."""
    p = _unlike_rows(seed)
    off = p.row_offsets()
    for a in range(0, p.N_A, 3):
        p.A[off[a] + 2] = 0
        for which in ("T_AA", "T_AB"):
            t = p.t_block(which, a).copy()
            t[5] = 0
            if which == "T_AA":
                t[:, 5] = 0
                t[5, 5] = 1e-300
            p.set_t_block(which, a, t)
    return p


CASES = {"atom_x1000": lambda: _atom_x1000(3), "unlike_rows": lambda: _unlike_rows(4),
         # 4 N_G^2 < K: one row maximum for six rows
         "grouped_rows": lambda: _atom_x1000(7, 8),
         "unlike_rows_failing": lambda: _unlike_rows(5, [1, 40]), "zero_rows": lambda: _zero_rows(6)}


def _ratios(p, mode):
    """Errors of H and S over those of Alg. 1's operands."""
    import torch
    from paper_1611_00606_amd import DeviceBuild
    r = DeviceBuild.from_problem(p, mode=mode)
    r.run()
    torch.cuda.synchronize()
    H, S, _ = r.results()
    assert np.array_equal(H, H.conj().T) and np.array_equal(S, S.conj().T)
    Hr = O.hamiltonian(p.A, p.B, p.T_AA, p.T_AB, p.T_BB, p.nl)
    Sr = O.overlap(p.A, p.B, p.U, p.nl)
    eh, es = (np.linalg.norm(x - y) / np.linalg.norm(y) for x, y in ((H, Hr), (S, Sr)))
    rh, rs = alg1_error(p, Hr, mode), overlap_error(p, Sr, mode)
    print(f"  H {eh:.2e} (Alg. 1's operands {rh:.2e}), S {es:.2e} ({rs:.2e})", flush=True)
    return eh / rh, es / rs


@pytest.mark.parametrize("mode", [1, 2, 4, 5])
@pytest.mark.parametrize("name", list(CASES))
def test_error_on_unlike_rows(name, mode):
    print(f"case {name} mode={mode}", flush=True)
    assert max(_ratios(CASES[name](), mode)) <= BALANCE


@pytest.mark.parametrize("mode", [1, 2, 4, 5])
def test_error_on_ordinary_problems(mode):
    """Several sizes and magnitudes: the column scales' luck averages out."""
    logs = []
    for i in range(10):
        rng = np.random.default_rng(i)
        n_a, n_g = int(rng.integers(4, 65)), int(rng.integers(60, 160))
        nl = int(rng.integers(9, 60)) if i % 2 else rng.integers(9, 60, n_a)
        print(f"case {i} N_A={n_a} N_G={n_g} mode={mode}", flush=True)
        p = make_problem(n_a, nl, n_g, seed=i, n_fail=i % 3)
        for k in ("A", "B", "T_AA", "T_AB", "T_BB"):
            setattr(p, k, getattr(p, k) * 2.0 ** rng.uniform(-1, 1))
        logs.append(np.log(_ratios(p, mode)))
    assert np.all(np.mean(logs, axis=0) <= 0.0)


@pytest.mark.parametrize("mode", [1, 2, 4, 5])
@pytest.mark.parametrize("exp", [-505, 505])
def test_values_whose_squares_leave_the_range(exp, mode):
    """A and B at 2^+-505 (block norms of the modular form are then summed at the
    block's own exponent); the forms' bound of 1e-9, relative. The oracle works
    on values at 1 and is scaled by powers of two."""
    import torch
    from paper_1611_00606_amd import DeviceBuild
    print(f"case exp={exp} mode={mode}", flush=True)
    p = make_problem(5, [16, 9, 30, 7, 12], 150, seed=12, fail_atoms=[1])
    Hr = O.hamiltonian(p.A, p.B, p.T_AA, p.T_AB, p.T_BB, p.nl)
    Sr = O.overlap(p.A, p.B, p.U, p.nl)
    p.A *= 2.0 ** exp
    p.B *= 2.0 ** exp
    r = DeviceBuild.from_problem(p, mode=mode)
    r.run()
    torch.cuda.synchronize()
    H, S, _ = r.results()
    for got, want in ((H, Hr), (S, Sr)):
        back = got * 2.0 ** -exp * 2.0 ** -exp
        assert np.linalg.norm(back - want) <= 1e-9 * np.linalg.norm(want)
