"""The autotuner's search and its stored results (CPU: a context that only
keeps what it is told)."""

import json

import numpy as np

import paper_1204_6630_amd as tp
from paper_1204_6630_amd import autotune as at


class Recorder:
    def __init__(self):
        self.tunings, self.counts = [], 0

    def set_tuning(self, **t):
        self.tunings.append(t)

    def set_timing(self, on):
        pass

    def kernel_time(self, reset=False):
        return 1.0, 1

    def count(self, *a, **k):
        self.counts += 1


def test_results_of_earlier_kernels_are_not_applied(tmp_path, monkeypatch):
    """A shape that was stored for the kernels of an earlier version (their
    key, their widest units) is searched for again; one stored now is used."""
    path = tmp_path / "autotune.json"
    monkeypatch.setenv("TPCF_AUTOTUNE_CACHE", str(path))
    key = at._device_key(tp.FP32_CHORD, 20)
    old = {"rows_per_lane": 4, "hist_copies": 32, "max_cols": 16384, "blocks_per_cu": 0, "lut_direct": 1, "lut_bytes": 0}
    path.write_text(json.dumps({"v4|" + key.split("|", 1)[1]: {"tuning": old, "timings_ms": {}}}))
    edges, sample = np.linspace(1.0, 9.0, 21), [(tp.DD, 0, -1, -1, -1)]
    ctx = Recorder()
    res = at.autotune(ctx, sample, edges)
    assert not res["cached"] and ctx.counts > 0
    assert old not in ctx.tunings and res["tuning"] == {k: 0 for k in at.CANDIDATES}
    again = Recorder()
    res = at.autotune(again, sample, edges)
    assert res["cached"] and again.counts == 0 and again.tunings == [res["tuning"]]


def test_every_knob_has_an_effect():
    """The table layout field is accepted but reaches no launch: the search
    would store which of two equal launches happened to be faster."""
    assert "lut_direct" not in at.CANDIDATES
    assert set(at.CANDIDATES) <= {name for name, _ in tp.Tuning._fields_}
