"""A captured split build decides about its rows anew on every replay.

Whether rows of A and X are scaled is found on the device, so one graph serves
inputs of both kinds: replays with balanced and with unlike rows, in turn and with
eager builds between them, give bitwise what an eager build gives.
"""

import numpy as np
import pytest

from hs_inputs import make_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [0, 1])
@pytest.mark.parametrize("mode", [1, 2, 4, 5])
def test_replays_equal_eager_builds(mode, batch):
    import torch
    from paper_1611_00606_amd import DeviceBuild
    print(f"case mode={mode} batch={batch}", flush=True)
    plain = make_problem(12, 20, 200, seed=1)
    unlike = plain.copy()
    off = unlike.row_offsets()
    rng = np.random.default_rng(2)
    for a in range(unlike.N_A):
        d = 10.0 ** rng.uniform(-2, 2, 20)
        unlike.set_t_block("T_AA", a, d[:, None] * unlike.t_block("T_AA", a) * d[None, :])
        unlike.A[off[a]:off[a + 1]] /= d[:, None]
    want, inputs = [], []
    for p in (plain, unlike):
        r = DeviceBuild.from_problem(p, mode=mode, batch=batch)
        r.run()
        torch.cuda.synchronize()
        want.append((r.H.clone(), r.S.clone()))
        inputs.append((r.A, r.T_AA))
    g = DeviceBuild.from_problem(plain, mode=mode, batch=batch)
    g.run()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.run()
    for i in (0, 1, 1, 0, 1, 0):
        g.A.copy_(inputs[i][0])
        g.T_AA.copy_(inputs[i][1])
        g.H.fill_(float("nan"))
        g.S.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(g.H, want[i][0]) and torch.equal(g.S, want[i][1]), i
        r.run()   # an eager build of its own between the replays
        torch.cuda.synchronize()
