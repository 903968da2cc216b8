"""The eigenproblem reduction reads nothing of its workspace that it has not
written: with the workspace full of NaN and of zeros L and Ht are the same bits.

Sizes: one block, its last panel ragged; one to three steps beside the
factorization, forks after first and second panels of a pair, steps of up to
eight panels.
"""

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 3], ids=["fp64", "3m"])
@pytest.mark.parametrize("N", [100, 300, 384, 385, 700, 1000, 1500, 2100, 2600, 4200])
def test_workspace_contents_do_not_matter(N, mode):
    import torch
    import paper_1611_00606_amd as P
    print(f"case N={N} mode={mode}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(N)
    X = torch.randn(N, N, dtype=torch.complex128, device="cuda:0", generator=g)
    S = X @ X.conj().T.contiguous() / (2 * N) + torch.eye(N, dtype=X.dtype, device="cuda:0")
    S = (S + S.conj().T) / 2
    H = X + X.conj().T
    out = []
    for fill in (float("nan"), 0.0):
        ws = torch.full((P.hs_gep_workspace_bytes(N) // 8,), fill, dtype=torch.float64, device="cuda:0")
        L, Ht = torch.empty_like(H), torch.empty_like(H)
        info = torch.full((1,), -7, dtype=torch.int32, device="cuda:0")
        P.hs_gep_reduce(H, S, L, Ht, info=info, workspace=ws.view(torch.uint8), mode=mode)
        torch.cuda.synchronize()
        assert int(info.item()) == 0
        out.append((L, Ht))
    for a, b in zip(*out):
        assert torch.isfinite(torch.view_as_real(a)).all() and torch.equal(a, b)
