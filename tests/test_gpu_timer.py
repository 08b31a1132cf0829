"""GPU: what the kernel timer reports.  Meshes N <= 32: the launch of a whole
refinement pass counts and is timed as the bottom levels.
"""
import numpy as np
import pytest

import synth
from cases import instance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hv = pytest.importorskip("paper_1909_03948_amd.hinv")


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


def problem(ctx, N, precision):
    prob, _, obs = instance(16, 10)
    gp = hv.Problem(ctx, N, prob.gamma, prob.delta, obs_xy=obs, d_obs=prob.d, sigma=prob.sigma, beta=prob.beta,
                    precision=precision, rtol=1e-10)
    zero = dev(np.zeros((N + 1) ** 2))
    gp.linearize(dev(-2.0 + 0.4 * synth.smooth_field(N)), zero, zero)
    return gp


@pytest.mark.parametrize("N,precision", [(8, hv.PREC_FP64), (32, hv.PREC_FP64), (32, hv.PREC_FP32_IR)])
def test_small_meshes_are_timed(N, precision):
    print(f"[gpu-timer] N={N} precision={precision}", flush=True)
    ctx = hv.Context(0)
    gp = problem(ctx, N, precision)
    b = dev(synth.test_vectors((N + 1) ** 2, 3, seed=7))
    ctx.kernel_timer("mg_bottom", True, 1)
    passes = 0
    for _ in range(3):
        info = gp.state_solve(b, torch.zeros_like(b))
        assert info["rc"] == hv.HINV_OK
        passes += info["refinements"]
    r = ctx.kernel_timer_read("mg_bottom")
    ctx.kernel_timer("mg_bottom", False, 1)
    print(f"[gpu-timer] {r}", flush=True)
    assert r["launches"] == r["timed"] == passes and r["ms"] > 0 and r["work"] > 0
