"""The autotuner's host logic, on a stand-in batch: which cached shapes it takes,
and what runs before its timer starts."""
import json

import pytest

from paper_1906_03065_amd import autotune, lbib

ARCH = "gfx950"
W = [dict(params=dict(nx=100, ny=90)), dict(params=dict(nx=300, ny=90))]


class Batch:
    """Records its calls; a shape is faster the closer its rows are to 12."""

    def __init__(self, log, clock):
        self.log, self.clock, self.seg = log, clock, {}

    def set_launch(self, cls, bx, seg, ring):
        self.seg[cls] = seg
        self.log.append(("set", cls, seg))

    def step(self, n):
        self.log.append(("step", n))
        self.clock[0] += n * (1.0 + sum(abs(s - 12) for s in self.seg.values()))

    def synchronize(self):
        pass

    def close(self):
        pass


@pytest.fixture
def log(monkeypatch):
    log, clock = [], [0.0]

    def counter():
        log.append(("clock",))
        return clock[0]

    monkeypatch.setattr(autotune, "arch", lambda device="cuda:0": ARCH)
    monkeypatch.setattr(autotune.time, "perf_counter", counter)
    monkeypatch.setattr(lbib.Batch, "from_workloads", classmethod(lambda cls, ws, device=None: Batch(log, clock)))
    return log


def test_tunes_and_reuses(log, tmp_path):
    path = str(tmp_path / "c" / "tune.json")
    got = autotune.tune(W, cache_path=path)
    assert {c: v["seg"] for c, v in got.items()} == {0: 12, 2: 12}
    log.clear()
    assert autotune.tune(W, cache_path=path) == got
    assert log == []


def test_shapes_of_another_kernel_are_timed_again(log, tmp_path):
    path = tmp_path / "tune.json"
    old = dict(block_x=256, seg=48, ring=4, ms_per_step=0.1)
    path.write_text(json.dumps({f"{ARCH}|D2Q9|fp32|class{c}": old for c in range(3)}))
    got = autotune.tune(W, cache_path=str(path))
    assert {c: v["seg"] for c, v in got.items()} == {0: 12, 2: 12}
    assert json.loads(path.read_text())[f"{ARCH}|D2Q9|fp32|class0"] == old  # left for the program that wrote it


def test_timer_starts_after_the_graphs_of_inner_steps(log, tmp_path):
    """The steps inside a call have graphs of their own, which a call of two steps
    never uses: every timed call follows one of four steps or more."""
    autotune.tune(W, cache_path=str(tmp_path / "t.json"))
    warm = 0
    for e in log:
        if e[0] == "set":
            warm = 0
        elif e[0] == "step":
            warm = max(warm, e[1])
        else:
            assert warm >= 4
