"""Host logic of the autotuner (no GPU): it times no build twice, and a tile kept in the cache file is
used for the library it was timed on only."""
import json

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1002_1050_amd import _binding as B  # noqa: E402
from paper_1002_1050_amd import autotune  # noqa: E402


def test_forward_candidates_are_distinct_builds():
    """TB shapes the adjoint's kernels only: the forward has one build per R."""
    for op in (B.TC_OP_FWD, B.TC_OP_FWD_POL):
        R = [t[0] for t in autotune.CANDIDATES[op]]
        assert len(R) == len(set(R)), op
    assert len(set(autotune.CANDIDATES[B.TC_OP_ADJ])) == 6


def test_cached_tiles_belong_to_one_library(monkeypatch, tmp_path):
    path, so = tmp_path / "tiles.json", tmp_path / "lib.so"
    monkeypatch.setenv("TC_TUNE_CACHE", str(path))
    monkeypatch.setattr(B, "LIB_PATH", str(so))
    monkeypatch.setattr(autotune, "_gpu_name", lambda: "cpu-test")
    state = {}
    monkeypatch.setattr(B, "set_tile_ex", lambda op, R, TB, TR: state.update(R=R))
    monkeypatch.setattr(B, "get_tile_ex", lambda op, lmax: (8, 64, 4))
    monkeypatch.setattr(B, "totalconv_fwd_x", lambda *a, **k: None)
    ms = {}

    def timed(fn, reps=2):
        fn()
        return ms[state["R"]]

    monkeypatch.setattr(autotune, "_time", timed)

    def tune():
        return autotune.tune_plain(B.TC_OP_FWD, 100, 4, np.zeros(8), None, None, reps=1)[0]

    class Plan:
        def execute(self):
            pass

        def close(self):
            pass

    so.write_bytes(b"one build")
    ms.update({2: 3.0, 4: 1.0, 8: 2.0})
    assert tune() == 4 and autotune.tune_plan(B.TC_OP_FWD, Plan, reps=1)[0][0] == 4
    ms.update({2: 3.0, 4: 2.0, 8: 1.0})
    assert tune() == 4 and autotune.tune_plan(B.TC_OP_FWD, Plan, reps=1)[0][0] == 4     # from the file
    so.write_bytes(b"another build")
    assert tune() == 8 and autotune.tune_plan(B.TC_OP_FWD, Plan, reps=1)[0][0] == 8     # timed again
    assert len(json.loads(path.read_text())) == 4
