"""The tuner keeps what it timed apart: a quadratic-state solve times the V-cycle
of its linear hierarchy alone, a linear-state solve of the same mesh, columns
and precision a refinement pass.  Neither takes the other's launch shape, in
memory or from the file.
"""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

pytest.importorskip("torch")
pytest.importorskip("paper_1909_03948_amd.hinv")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import json, sys
import torch
sys.path.insert(0, sys.argv[1])
import synth
from paper_1909_03948_amd import hinv as hv
ctx = hv.Context(0)
for degree in map(int, sys.argv[2]):
    N, nc = 64, int(sys.argv[3])
    ns = (degree * N + 1) ** 2
    gp = hv.Problem(ctx, N, 0.1, 0.5, precision=hv.PREC_FP64, state_degree=degree)
    zero = torch.zeros(ns, dtype=torch.float64, device="cuda")
    gp.linearize(torch.as_tensor(-2.0 + 0.4 * synth.smooth_field(N), device="cuda"), zero, zero)
    b = torch.as_tensor(synth.test_vectors(ns, nc, seed=9), device="cuda")
    assert gp.state_solve(b, torch.zeros_like(b))["rc"] == 0
print(json.dumps(hv.tuner_counts()))
"""


def child(cache, degrees, nc=9):
    env = dict(os.environ, HINV_TUNE_CACHE=cache)
    env.pop("HINV_AUTOTUNE", None)
    env.pop("HINV_SHAPE", None)
    r = subprocess.run([sys.executable, "-c", CHILD, ROOT, degrees, str(nc)], env=env, capture_output=True, text=True,
                       timeout=240)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout.strip().splitlines()[-1])


@pytest.mark.parametrize("order", ["21", "12"])
def test_shapes_of_passes_and_of_cycles_are_kept_apart(tmp_path, order):
    print(f"[gpu-tune-keys] {order}", flush=True)
    cache = str(tmp_path / "tune.jsonl")
    assert child(cache, order) == [2, 0]
    lines = [json.loads(l) for l in open(cache)]
    assert sorted(l["pass"] for l in lines) == [0, 1]
    assert {(l["kind"], l["N"], l["columns"], l["fp32"]) for l in lines} == {(lines[0]["kind"], 64, 9, 0)}
    assert child(cache, order[::-1]) == [0, 2]


def test_a_line_with_more_partials_than_there_is_room_for_is_skipped(tmp_path):
    """A cache line edited to chunks of 64 nodes (67 partial sums a column, where
    the buffers hold 25) is not taken: the shape is chosen anew."""
    cache = str(tmp_path / "tune.jsonl")
    assert child(cache, "1", 3) == [1, 0]
    line = json.loads(open(cache).read())
    assert line["N"] == 64 and line["columns"] == 3
    line.update(per=1, chunk=64)
    with open(cache, "w") as f:
        f.write(json.dumps(line) + "\n")
    assert child(cache, "1", 3) == [1, 0]
    line.update(chunk=256)
    with open(cache, "w") as f:
        f.write(json.dumps(line) + "\n")
    assert child(cache, "1", 3) == [0, 1]
