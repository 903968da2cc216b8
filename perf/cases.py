"""The work a program has this framework do, as measurable cases.

A FLAPW program builds H and S of one k-point from the matching coefficients
A, B, the per-atom blocks T and the norms U (hs_build_ex), or builds many
k-points of one atom set (hs_ctx_build, the serving loop), and reduces the
generalized eigenproblem of each pair to standard form (hs_gep_reduce). The
cases call those entry points with device tensors, at the sizes of this
repository's workloads (hs_inputs), and draw(rng) gives more of the same
ranges, odd sizes, mixed N_L, failing atoms and every reduction mode among
them.

Inputs follow hs_inputs' distributions, drawn on the device from the seed:
A, B ~ CN(0,1)/sqrt(N_G); T_AA = herm(M M^H / N_L + I), failing atoms shifted
by -2 lambda_max; T_AB ~ CN(0,1)/N_L; T_BB Hermitian; U real in [0.5, 2].
"""

import math

import torch

import paper_1611_00606_amd as hs
from paper_1611_00606_amd.serving import Context, ServingLoop

DEV = "cuda:0"
MODES = {"fp64": hs.HS_FP64, "fp64_3m": hs.HS_FP64_3M, "f16": hs.HS_SPLIT_F16,
         "bf16": hs.HS_SPLIT_BF16, "i8": hs.HS_SPLIT_I8, "crt": hs.HS_SPLIT_I8_CRT}


def listed():
    return [
        # The smallest build: four light atoms, a small basis. A program that
        # tests or sweeps many small systems waits for its latency.
        _build("build_tiny", 4, 16, 256),
        # An ordinary build of a medium system, three atoms on the
        # Cholesky-failure branch.
        _build("build_plain", 32, 49, 2000, n_fail=3),
        # Four atom types with different l_max in one build, the per-atom
        # stage batched, 6 atoms failing.
        _build("build_mixed_batched", 128, [16, 49, 81, 121], 6000, n_fail=6, batch=1),
        # The headline build: 100 atoms, l_max 8, N_G = 8000.
        _build("build_large", 100, 81, 8000, batch=1),
        # The 3M form at the paper's AuAg system, K_max = 2.5.
        _build("build_3m_auag", 108, 121, 3275, mode="fp64_3m"),
        # INT8 slices at the paper's NaCl system, K_max = 3.0: many atoms,
        # a contraction much longer than the outputs are wide.
        _build("build_i8_nacl", 512, 49, 3893, mode="i8", batch=1),
        # The modular form at the headline size: the fastest large build.
        _build("build_crt_large", 100, 81, 8000, mode="crt", batch=1),
        # One k-point of a resident atom set, FP16 slices, the small end of
        # the serving stream, an odd size.
        _ctx("kpoint_f16_small", 64, 64, 1501, mode="f16"),
        # A burst of k-points with host inputs through the serving loop.
        _serve("serve_burst", 64, 64, "1500-2251-3001"),
        # Reduction of the generalized eigenproblem: one small pair, where
        # latency counts, a medium one, and the headline build's.
        _gep("gep_small", 300),
        _gep("gep_medium", 2000),
        _gep("gep_large", 8000),
    ]


def draw(rng):
    kind = rng.choice(["build"] * 4 + ["ctx"] * 2 + ["gep"] * 2)
    if kind == "gep":
        n = _log_int(rng, 65, 8000)
        return _gep(None, n, rng.choice(["fp64", "fp64_3m"]))
    mode = rng.choice(["fp64", "fp64", "fp64", "fp64_3m", "f16", "bf16", "i8", "crt"])
    batch = rng.choice([0, 1])
    while True:
        n_g = _log_int(rng, 256, 9273)
        n_a = _log_int(rng, 4, 512)
        if kind == "build" and rng.random() < 0.3:
            n_l = sorted(rng.randint(9, 121) for _ in range(rng.randint(2, 4)))
        else:
            n_l = rng.randint(9, 121)
        n_fail = min(n_a, rng.choice([0, 0, 1, 3, 6]))
        c = (_ctx if kind == "ctx" else _build)(None, n_a, n_l, n_g, mode=mode, batch=batch,
                                               n_fail=n_fail)
        if sum(_nl(c)) * n_g * n_g <= 8100 * 8000 * 8000 and sum(_nl(c)) * n_g <= 1e8:
            return c


def work(case):
    if case["kind"] == "gep":
        n = case["n"]
        # the standard count of the reduction (zpotrf + zhegst); H and the
        # lower triangle of S read, L and Ht written
        return {"bytes": 16 * 3.5 * n * n, "flops": 16.0 / 3.0 * n ** 3}
    nl = _nl(case)
    K, t = sum(nl), sum(n * n for n in nl)
    total = {"bytes": 0.0, "flops": 0.0}
    for n_g in _sizes(case):
        # A, B, T, U read, H and S written; both Hermitian, so half of each
        # product: H = [A; B]^H (T [A; B]) and S = [A; B]^H (D [A; B]) contract
        # over 2K rows, 8 real operations per complex multiply-add; the
        # per-atom products take at least 20 N_L^2 N_G (Alg. 1).
        total["bytes"] += 16.0 * (2 * K * n_g + 3 * t + K + 2 * n_g * n_g)
        total["flops"] += 16.0 * K * n_g * n_g + 20.0 * t * n_g
    return total


def prepare(case, seed):
    if case["kind"] == "gep":
        H, S = _gep_inputs(case, seed)
        n = case["n"]
        return {"kind": "gep", "H": H, "S": S, "L": torch.empty_like(H),
                "Ht": torch.empty_like(H),
                "info": torch.zeros(1, dtype=torch.int32, device=DEV),
                "workspace": torch.empty(hs.hs_gep_workspace_bytes(n), dtype=torch.uint8,
                                         device=DEV),
                "mode": MODES[case["mode"]]}
    nl = _nl(case)
    T_AA, T_AB, T_BB, U = _atom_inputs(case, seed)
    mode = MODES[case["mode"]]
    if case["kind"] == "serve":
        ctx = Context(*(x.cpu().numpy() for x in (T_AA, T_AB, T_BB, U)), nl)
        reqs, outs, keep = [], {}, []
        for r, n_g in enumerate(_sizes(case)):
            A, B = (x.cpu().pin_memory() for x in _ab(sum(nl), n_g, seed, r))
            keep.append((A, B))
            reqs.append({"id": r, "N_G": n_g, "A_ptr": A.data_ptr(), "B_ptr": B.data_ptr(),
                         "ld": n_g})
            outs[r] = tuple(torch.empty((n_g, n_g), dtype=torch.complex128, device=DEV)
                            for _ in range(2))
        arena = sum(ctx.footprint_bytes(n_g, mode) for n_g in _sizes(case)) + (64 << 20)
        loop = ServingLoop(ctx, case["slots"], arena, mode=mode)
        return {"kind": "serve", "loop": loop, "reqs": reqs, "outs": outs, "keep": keep}
    n_g = case["n_g"]
    A, B = _ab(sum(nl), n_g, seed, 0)
    H = torch.empty((n_g, n_g), dtype=torch.complex128, device=DEV)
    st = {"kind": case["kind"], "A": A, "B": B, "n_g": n_g, "H": H, "S": torch.empty_like(H),
          "mode": mode, "batch": case["batch"]}
    if case["kind"] == "ctx":
        st["ctx"] = Context(*(x.cpu().numpy() for x in (T_AA, T_AB, T_BB, U)), nl)
        nbytes = st["ctx"].workspace_bytes(n_g, mode)
    else:
        uniform = len(set(nl)) == 1
        st.update(T_AA=T_AA, T_AB=T_AB, T_BB=T_BB, U=U, n_a=len(nl), n_l=max(nl),
                  nl=None if uniform else nl,
                  info=torch.empty(len(nl), dtype=torch.int32, device=DEV))
        nbytes = hs.hs_workspace_bytes(len(nl), st["nl"], max(nl), n_g, mode)
    st["workspace"] = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    return st


def run(st):
    if st["kind"] == "gep":
        hs.hs_gep_reduce(st["H"], st["S"], st["L"], st["Ht"], info=st["info"],
                         workspace=st["workspace"], mode=st["mode"])
        return st["L"], st["Ht"], st["info"]
    if st["kind"] == "serve":
        def take(res):   # the result's arena space is reused after this call
            for out, ptr in zip(st["outs"][res["id"]], (res["H"], res["S"])):
                out.copy_(torch.as_tensor(_DeviceMatrix(ptr, res["N_G"]), device=DEV))
            torch.cuda.current_stream().synchronize()
        st["loop"].run(st["reqs"], [0.0] * len(st["reqs"]), on_result=take)
        return [st["outs"][r["id"]] for r in st["reqs"]]
    if st["kind"] == "ctx":
        st["ctx"].build(st["A"], st["B"], st["n_g"], st["H"], st["S"], st["workspace"],
                        mode=st["mode"], batch=st["batch"])
        return st["H"], st["S"]
    hs.hs_build_ex(st["A"], st["B"], st["T_AA"], st["T_AB"], st["T_BB"], st["U"], st["n_a"],
                   st["n_l"], st["n_g"], st["H"], st["S"], workspace=st["workspace"],
                   info=st["info"], mode=st["mode"], nl_per_atom=st["nl"], batch=st["batch"])
    return st["H"], st["S"], st["info"]


def exact(case, seed):
    if case["kind"] == "gep":
        if case["n"] > 3000:
            return None   # the factorization and two full solves take too long on the host
        H, S = (x.cpu() for x in _gep_inputs(case, seed))
        L = torch.linalg.cholesky(S)
        V = torch.linalg.solve_triangular(L, H, upper=False)
        Ht = torch.linalg.solve_triangular(L, V.mH, upper=False)
        return L, (Ht + Ht.mH) * 0.5, None
    T_AA, T_AB, T_BB, U = _atom_inputs(case, seed)
    nl = _nl(case)
    out = []
    for r, n_g in enumerate(_sizes(case)):
        A, B = _ab(sum(nl), n_g, seed, r)
        X, Y = torch.empty_like(A), torch.empty_like(B)
        r0 = t0 = 0
        for n in nl:
            rows, blk = slice(r0, r0 + n), slice(t0, t0 + n * n)
            aa, ab, bb = (t[blk].view(n, n) for t in (T_AA, T_AB, T_BB))
            torch.matmul(aa, A[rows], out=X[rows])
            X[rows] += ab @ B[rows]
            torch.matmul(ab.mH.contiguous(), A[rows], out=Y[rows])
            Y[rows] += bb @ B[rows]
            r0, t0 = r0 + n, t0 + n * n
        H = A.mH @ X
        H += B.mH @ Y
        del X, Y
        S = A.mH @ A
        S += B.mH @ (B * U.abs().square()[:, None])
        out.append((H, S))
    if case["kind"] == "serve":
        return out
    return out[0] + ((None,) if case["kind"] == "build" else ())


# ---------------------------------------------------------------------------


def _build(name, n_a, n_l, n_g, mode="fp64", batch=0, n_fail=0, kind="build"):
    c = {"kind": kind, "n_a": n_a, "n_g": n_g, "mode": mode, "batch": batch, "n_fail": n_fail,
         # one value, or the types' values, atoms shared out in order
         "n_l": "-".join(str(x) for x in n_l) if isinstance(n_l, list) else str(n_l)}
    if name:
        c["name"] = name
    return c


def _ctx(name, *args, **kw):
    return _build(name, *args, kind="ctx", **kw)


def _serve(name, n_a, n_l, sizes, slots=3):
    c = _build(name, n_a, n_l, sizes, kind="serve")
    c["slots"] = slots
    return c


def _gep(name, n, mode="fp64"):
    c = {"kind": "gep", "n": n, "mode": mode}
    if name:
        c["name"] = name
    return c


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sizes(case):
    """N_G of each k-point of the case (a served burst has several)."""
    return [int(x) for x in str(case["n_g"]).split("-")]


def _nl(case):
    """N_L of each atom: n_a atoms in equal runs of the case's types."""
    types = [int(x) for x in case["n_l"].split("-")]
    return [types[a * len(types) // case["n_a"]] for a in range(case["n_a"])]


def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + stream) % (1 << 63))
    return g


def _cn(g, *shape, scale=1.0):
    x = torch.randn(*shape, 2, generator=g, device=DEV, dtype=torch.float64)
    return torch.view_as_complex(x.mul_(scale * math.sqrt(0.5)))


def _ab(K, n_g, seed, request):
    s = 1.0 / math.sqrt(n_g)
    return (_cn(_gen(seed, 16 + 2 * request), K, n_g, scale=s),
            _cn(_gen(seed, 17 + 2 * request), K, n_g, scale=s))


def _herm(t):
    return (t + t.mH) * 0.5


def _atom_inputs(case, seed):
    """T_AA, T_AB, T_BB (concatenated row-major blocks) and U."""
    g = _gen(seed, 1)
    nl = _nl(case)
    failing = set(torch.randperm(len(nl), generator=torch.Generator().manual_seed(int(seed)))
                  [:case["n_fail"]].tolist())
    aa, ab, bb = [], [], []
    a = 0
    while a < len(nl):   # a run of atoms of one N_L
        n = nl[a]
        m = sum(1 for x in nl[a:] if x == n)
        X = _cn(g, m, n, n)
        T = _herm(torch.stack([x @ x.mH.contiguous() for x in X]) / n
                  + torch.eye(n, device=DEV, dtype=torch.complex128))
        for i in range(m):
            if a + i in failing:
                lam = float(torch.linalg.eigvalsh(T[i].cpu()).max())
                T[i].diagonal().sub_(2.0 * lam)
        aa.append(T.reshape(-1))
        ab.append(_cn(g, m, n, n, scale=1.0 / n).reshape(-1))
        bb.append((_herm(_cn(g, m, n, n)) / n).reshape(-1))
        a += m
    u = torch.rand(sum(nl), generator=g, device=DEV, dtype=torch.float64) * 1.5 + 0.5
    return torch.cat(aa), torch.cat(ab), torch.cat(bb), u.to(torch.complex128)


def _gep_inputs(case, seed):
    """H and S as a build gives them: S = A^H A + B^H |U|^2 B of full rank,
    H Hermitian of the same size, both exactly Hermitian."""
    n = case["n"]
    K = n + 64
    A, B = _ab(K, n, seed, 0)
    u2 = (torch.rand(K, 1, generator=_gen(seed, 2), device=DEV, dtype=torch.float64) * 1.5
          + 0.5).square()
    S = A.mH @ A
    S += B.mH @ (B * u2)
    H = A.mH @ B
    return (H + H.mH) * 0.5, (S + S.mH) * 0.5


class _DeviceMatrix:
    """A served result (device pointer) as an array that torch can view."""

    def __init__(self, ptr, n):
        self.__cuda_array_interface__ = {"data": (int(ptr), False), "shape": (n, n),
                                         "typestr": "<c16", "version": 3}
