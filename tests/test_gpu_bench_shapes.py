"""What the bench line says about the launches of a run whose shapes the library chose by size: the
shape and the kernel that ran, also where a graph no longer than the timed steps was asked for."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def line(*args):
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--no-tune", "--no-cpu",
                        "--no-served", "--warmup", "9", *args],
                       capture_output=True, text=True, timeout=300, cwd=ROOT)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads([ln for ln in r.stdout.splitlines() if ln.strip()][-1])


@pytest.mark.parametrize("steps", [20, 60])
def test_untuned_line_names_the_default_shape(steps):
    d = line("--steps", str(steps))
    launch = d["config"]["launch"]
    assert (launch["threads"], launch["ppt"], launch["steps_per_launch"]) == (512, 4, 1)
    assert d["config"]["timed_launches"] == "graph replays"
    assert d["roofline"]["kernel"] == "k_fused" and d["roofline"]["steps_per_launch"] == 1
