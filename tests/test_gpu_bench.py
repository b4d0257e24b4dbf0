"""bench.py's modes run to the end and print one line of JSON, on reduced workloads."""
import json
import sys

import pytest

import bench
from paper_2602_03152_amd import workload as W

pytestmark = pytest.mark.gpu

SMALL = {0: dict(), 1: dict(n_ctx=9024, budget=700), 2: dict(batch=16, n_ctx=8256, budget=128), 3: dict(batch=1, n_ctx=4096, budget=774)}


@pytest.mark.parametrize("argv,kernel", [
    (["--config", "0"], "fasa_step"), (["--config", "1"], "fasa_list"), (["--config", "2"], "fasa_list"),
    (["--config", "1", "--pairing", "interleaved"], "fasa_list"), (["--config", "3"], "fasa_list"),
    (["--config", "1", "--offload"], "fasa_offload_attend"), (["--config", "0", "--offload"], "fasa_offload_gather"),
    (["--config", "1", "--calibrate", "2"], "fasa_calib_fc"), (["--config", "1", "--paged", "16"], None),
    (["--config", "2", "--ragged", "8"], None), (["--config", "3", "--growing", "8"], None),
    (["--config", "1", "--recall-table"], None),
], ids=str)
def test_mode_runs(monkeypatch, capsys, argv, kernel):
    for cid, kw in SMALL.items():
        monkeypatch.setitem(W.WORKLOADS, cid, W.WORKLOADS[cid].scaled(**kw))
    print("bench", argv, flush=True)
    monkeypatch.setattr(sys, "argv", ["bench.py", *argv, "--steps", "8", "--warmup", "2", "--sets", "4", "--no-cpu-baseline",
                                      "--other-workloads", ""])
    bench.main()
    lines = [l for l in capsys.readouterr().out.splitlines() if l.startswith("{")]
    assert len(lines) == 1
    out = json.loads(lines[0])
    assert out.get("graph_replays_match_eager") in (None, True)
    if kernel:
        assert kernel in out["kernels"]
        if out.get("roofline"):
            assert out["roofline"]["achieved"] > 0
