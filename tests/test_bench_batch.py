"""The batch benchmark's two sides run the same work: the same number of steps in
calls of the same length (inside a call the state has another form than between
calls)."""
import argparse
import json

import bench
from paper_1906_03065_amd import autotune, lbib
from paper_1906_03065_amd import workloads as W


def test_both_sides_call_alike(monkeypatch, capsys):
    import torch

    calls = {"batch": [], "sims": []}

    class Stub:
        def __init__(self, side):
            self.calls = calls[side]

        def step(self, n=1):
            self.calls.append(n)

        def synchronize(self):
            pass

        close = synchronize

        def graph(self):
            return 1

        def check(self):
            return 0

        def get_launch(self, c):
            return {}

    ws = W.c4(count=3)
    monkeypatch.setattr(W, "c4", lambda: ws)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    monkeypatch.setattr(autotune, "tune", lambda ws, steps=20: {})
    monkeypatch.setattr(lbib.Batch, "from_workloads", classmethod(lambda cls, ws: Stub("batch")))
    monkeypatch.setattr(lbib, "from_workload", lambda w: Stub("sims"))
    bench.bench_batch(argparse.Namespace(steps=20, warmup=5, no_cpu=True, cpu_seconds=1.0))
    assert calls["batch"] == [5, 20]
    assert sorted(calls["sims"]) == sorted(3 * calls["batch"])
    assert json.loads(capsys.readouterr().out.splitlines()[-1])["speedup_vs_sequential"] > 0
