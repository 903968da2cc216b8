"""Shares of the peak in bench.py's record count what a build executes."""

import numpy as np

import bench
import hs_inputs
import paper_1611_00606_amd
from paper_1611_00606_amd import tuning
from paper_1611_00606_amd.flops import algorithmic_flops, executed_flops


def test_paper_shape_share_of_the_peak(monkeypatch):
    """A build that runs its own operations at exactly the peak is at 100%,
    though Alg. 1's count of them is larger."""
    p = hs_inputs.make_problem(8, 8, 512, seed=0)
    assert algorithmic_flops(p.nl, p.N_G, np.zeros(8)) > executed_flops(p.nl, p.N_G)
    ms = executed_flops(p.nl, p.N_G) / (bench.FP64_MFMA_PEAK_TFLOPS * 1e12) * 1e3

    class Run:
        info = type("Info", (), {"cpu": staticmethod(lambda: np.zeros(8)),
                                 "numpy": staticmethod(lambda: np.zeros(8))})

        @classmethod
        def from_problem(cls, *a, **kw):
            return cls()

    Run.info.cpu = staticmethod(lambda: Run.info)
    monkeypatch.setattr(hs_inputs, "make_config", lambda name, seed: p)
    monkeypatch.setattr(paper_1611_00606_amd, "DeviceBuild", Run)
    monkeypatch.setattr(tuning, "autotune", lambda *a, **kw: (None, None))
    monkeypatch.setattr(bench, "timed_builds", lambda *a, **kw: (np.full(4, ms / 4), ms))
    out = bench.paper_shape_bench("nacl_kmax4", 0, 1, None)
    assert out["pct_of_fp64_mfma_peak"] <= 100.0
    assert abs(out["pct_of_fp64_mfma_peak"] - 100.0) < 2.0   # ms is rounded to 1e-3
