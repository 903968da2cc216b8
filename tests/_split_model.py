"""NumPy model of the split forms' operand cuts, for their error bounds.

A product of two operands keeps, per column, the slices of the FP16 or INT8
form (the pairs those forms multiply) or the integers of the modular form.
`alg1_error` is the error of H when Alg. 1's own operands are cut so:
Z^H B + B^H Z + W^H W (A^H W for atoms without a Cholesky factor), Z = T_BA A +
1/2 T_BB B, W = C^H A (T_AA A), every column scaled by a power of two.
"""

import numpy as np

BITS = {"f16": [8, 9, 9, 9], "i8": [7] * 5, "crt": [36]}
FORM = {1: "f16", 2: "i8", 4: "f16", 5: "crt"}   # by HS mode


def _cut(X, form):
    m = np.maximum(abs(X.real), abs(X.imag)).max(axis=0)
    m = m * (128.0 / 127.0) if form == "i8" else m
    e = np.where(m > 0, np.frexp(m)[1], 0)
    r = X * np.ldexp(1.0, -e)
    if form == "crt":
        s = 2.0 ** 35
        return [(np.rint(r.real * s) + 1j * np.rint(r.imag * s)) / s], e
    out, w = [], 1.0
    for b in BITS[form]:
        r, w = r * 2.0 ** b, w * 2.0 ** -b
        s = np.rint(r.real) + 1j * np.rint(r.imag)
        if form == "i8":
            s = np.clip(s.real, -127, 127) + 1j * np.clip(s.imag, -127, 127)
        r = r - s
        out.append(s * w)
    return out, e


def cut_product(P, Q, form):
    """P^H Q from the kept pairs of slices."""
    (p, ep), (q, eq) = _cut(P, form), _cut(Q, form)
    n = len(p)
    acc = sum(p[s].conj().T @ sum(q[:n - s]) for s in range(n))
    return acc * np.ldexp(1.0, ep)[:, None] * np.ldexp(1.0, eq)[None, :]


def alg1_error(p, H, mode):
    """Relative Frobenius distance from H of Alg. 1's grouping, cut."""
    Z, W, V = (np.zeros_like(p.A) for _ in range(3))
    off = p.row_offsets()
    for a in range(p.N_A):
        s = slice(off[a], off[a + 1])
        T, TB, BB = (p.t_block(k, a) for k in ("T_AA", "T_AB", "T_BB"))
        Z[s] = TB.conj().T @ p.A[s] + 0.5 * BB @ p.B[s]
        try:
            W[s] = np.linalg.cholesky(T).conj().T @ p.A[s]
            V[s] = W[s]
        except np.linalg.LinAlgError:
            W[s], V[s] = T @ p.A[s], p.A[s]
    f = FORM[mode]
    G = cut_product(Z, p.B, f) + cut_product(p.B, Z, f) + cut_product(V, W, f)
    return np.linalg.norm(mirrored(G) - H) / np.linalg.norm(H)


def overlap_error(p, S, mode):
    """Relative Frobenius distance from S of A^H A + (U B)^H (U B), cut."""
    f, V = FORM[mode], abs(p.U)[:, None] * p.B
    G = cut_product(p.A, p.A, f) + cut_product(V, V, f)
    return np.linalg.norm(mirrored(G) - S) / np.linalg.norm(S)


def mirrored(G):
    """The lower triangle's Hermitian completion."""
    L = np.tril(G, -1)
    return L + L.conj().T + np.diag(G.diagonal().real)
