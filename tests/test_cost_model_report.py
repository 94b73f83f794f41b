"""The committed cost model's report: how and on what it was made stands in it,
and a report that learn writes says the same."""
import json
import os
import types

import numpy as np

from paper_2602_08190_amd import learn as Lr

PKG = os.path.dirname(os.path.abspath(Lr.__file__))


def test_committed_report_says_how_it_was_made():
    with open(os.path.join(PKG, "cost_model_gfx950.json")) as f:
        rep = json.load(f)
    assert "learn collect" in rep["command"] and "learn train" in rep["command"]
    assert rep["train_chunks"] + rep["test_chunks"] == Lr.N_COLS * Lr.CHUNKS_PER_COL
    assert f"{Lr.N_COLS} synthetic columns" in rep["data"] and f"{Lr.CHUNKS_PER_COL} chunks of 8 MiB" in rep["data"]


def test_reports_name_their_data():
    a = types.SimpleNamespace(data=["/x/d0.npz", "d128.npz"], weights="/y/w.bin", report="r.json", epochs=7)
    assert Lr.provenance(a).endswith("learn train --data d0.npz d128.npz --weights w.bin --report r.json --epochs 7")
    T = np.full((4, 24), np.nan)
    T[:, :5] = 1.0
    d = {"ids": np.array([[0, 0], [0, 1], [9, 0], [9, 1]], np.int32), "T": T, "X": np.zeros((4, 32), np.float32)}
    s = Lr.describe(d)
    assert s.startswith("2 synthetic columns") and "2 chunks of 8 MiB" in s and s.endswith(": 20 timings")
