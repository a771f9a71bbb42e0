"""bench.py's roofline records name the kernels that a solve launched, on sampled spans
(kernel_ms, count, event_ms, event count, bytes) of made-up launches."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

FAMILIES = {"fp32_inner": "FP32 passes", "fp64_truth": "FP64 passes"}
NONE = (0.0, 0, 0.0, 0, 0.0)


def test_only_launched_families():
    import bench
    some = (1.0, 10, 2.0, 10, 4e9)
    r = bench.rooflines([NONE, NONE, some, NONE, NONE], FAMILIES, 12, 4096)
    assert list(r) == ["resident"]
    assert r["resident"]["achieved"] == 4e9 / 2e-3 / 1e9
    r = bench.rooflines([some, some, NONE, NONE, NONE], FAMILIES, 12, 4096)
    assert list(r) == ["fp32_inner"] and r["fp32_inner"]["launches_per_solve"] == 20
    assert set(bench.rooflines([NONE] * 5, FAMILIES, 12, 4096)) == {*FAMILIES, "resident"}


def test_batched_record_has_the_resident_kernel(monkeypatch):
    """The batched workload's record, with stand-ins for the device."""
    import numpy as np
    import bench

    class Lat:
        def __init__(self, *a, **k):
            pass

        def solve(self, b, p):
            return b, [dict(true_rel_res=1e-11, outer_iters=3)] * 12

    class Cuda:
        synchronize = staticmethod(lambda: None)

    class T:
        cuda = Cuda
        from_numpy = staticmethod(lambda a: type("A", (), {"cuda": lambda self: a})())

    class Inputs:
        config_seed = staticmethod(int)
        draw = staticmethod(lambda *a, **k: (np.zeros(1), np.zeros(1)))

    monkeypatch.setattr(bench, "sampled_spans",
                        lambda lat, run: [NONE, NONE, (0.0, 0, 5.0, 7, 1e9), NONE, NONE])
    out, _, _ = bench.batched_config3(T, Lat, Inputs)
    assert list(out["pass_rooflines"]) == ["resident"]
    assert out["pass_rooflines"]["resident"]["launches_per_solve"] == 7
