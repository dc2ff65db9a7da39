"""The benchmark's large spaces under per-backend pressure: the run ends with its
line, and the choices are the oracle's stored selections."""
import json
import os
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
BENCH = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "bench.py")


@pytest.mark.parametrize("workload", ["forkjoin8", "layered10"])
def test_per_class_workloads(workload):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    res = subprocess.run([sys.executable, BENCH, "--workload", workload, "--pressure", "per-class", "--steps", "2",
                          "--warmup", "1", "--no-cpu-baseline"], capture_output=True, text=True, timeout=100)
    assert res.returncode == 0, res.stderr[-2000:]
    line = json.loads([x for x in res.stdout.splitlines() if x.startswith("{")][-1])
    assert line["golden_check"].startswith("every choice equals")
    assert line["roofline"]["kernel"] in ("k_solve", "dy_sweep") and 0 < line["roofline"]["frac"] < 1
