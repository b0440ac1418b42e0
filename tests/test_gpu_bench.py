"""bench.py on short workloads of its own options: a grid whose time loop launches none of the timed
kernel classes, and one whose headline solve recomputes segments."""

import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,classes", [(32, False), (64, False), (128, True)])
def test_short_run_prints_its_line(N, classes):
    print("CASE bench", N, flush=True)
    cmd = [sys.executable, os.path.join(ROOT, "bench.py"), "--N", str(N), "--members", "2", "--horizon", "8",
           "--ckpt-every", "3", "--ckpt-leg", "4", "--steps", "1", "--warmup", "1", "--plain-solves", "1",
           "--graph-replays", "1", "--serving-requests", "0", "--no-cpu-baseline"]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=110)
    assert r.returncode == 0, r.stderr[-2000:]
    line = json.loads(r.stdout.strip().splitlines()[-1])
    assert line["value"] > 0 and line["checkpointed"]["value"] > 0
    assert (line["roofline"] is not None) == classes
    if classes:
        assert line["roofline"]["timed_launches"] > 0 and line["roofline"]["achieved"] > 0
