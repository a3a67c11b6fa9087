"""The benchmark on its smallest workload, whose iterations run in one launch: the
timed mode records them, and the line is complete."""
import json
import os
import subprocess
import sys

import pytest

from tests.gpu_common import say

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("n,name", [(16, "iterations_small"), (32, "operator")])
def test_timed_mode_records_the_iterations(n, name):
    torch = pytest.importorskip("torch")
    import paper_1712_06758_amd as P
    say(f"timing mode 2 n={n}")
    box = P.Box(n, 10.0, max_batch=2)
    xi = torch.randn(2, n ** 3, device="cuda", dtype=torch.float64)
    base = box.sample(xi, u_box=True)["u_box"]
    box.timing(2)
    box.timing(-1)
    out = box.sample(xi, u_box=True)
    box.timing(0)
    rep = box.timing_report()
    assert set(rep) == {name}
    assert rep[name]["total_ms"] > 0 and rep[name]["launches"] > 0 and rep[name]["bytes_per_launch"] > 0
    assert torch.equal(out["u_box"], base)


def test_smallest_workload():
    say("bench.py --workload box16")
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--workload", "box16", "--no-cpu", "--no-other",
                        "--serve-seconds", "0", "--steps", "2", "--warmup", "1"], cwd=ROOT, capture_output=True,
                       text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    line = json.loads(r.stdout.strip().splitlines()[-1])
    assert line["value"] > 0 and line["steps"] == 2 and line["config"]["n"] == 16
    assert line["roofline"]["kernel"] == line["roofline_fp64"]["kernel"] == "iterations_small"
