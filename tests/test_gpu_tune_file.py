"""The file of tile choices: those of the present kernels are taken over by a later
process, those that were timed with other kernels are not."""
import json
import os
import subprocess
import sys

import pytest

from tests.gpu_common import say

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHILD = """
import json, torch
import paper_1712_06758_amd as P
box = P.Box(32, 10.0, precision="fp64")
print(json.dumps(box.sample(torch.ones(1, 32 ** 3, dtype=torch.float64, device="cuda"))["tiles"]))
"""


def _tiles(path):
    r = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, env={**os.environ, "SPDE_TUNE_CACHE": str(path)},
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout.strip().splitlines()[-1])


def test_choices_of_other_kernels_are_timed_again(tmp_path):
    say("tile choices of an older file")
    path = tmp_path / "tiles.txt"
    old = "gfx950:n32:fp64:b1:t2 0 7 7\n"     # columns of 32 planes: one block in z, far from the fastest
    path.write_text(old)
    first = _tiles(path)
    assert first != [[7, 7]]
    lines = path.read_text()
    assert lines.startswith(old) and len(lines.splitlines()) == 2
    key = lines.splitlines()[1].split()[0]
    # a line of the present key is taken as it stands, and nothing is timed again
    path.write_text(f"{old}{key} 0 7 7\n")
    assert _tiles(path) == [[7, 7]]
    assert path.read_text() == f"{old}{key} 0 7 7\n"
