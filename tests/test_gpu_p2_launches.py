"""GPU: the iterations a quadratic-state solve enqueues before the host first
looks follow the last solve of the same columns and tolerance that met it.  A
solve that ran into its iteration cap, one of other columns or one to another
tolerance does not make the next one enqueue its count.

Counted through the timer of the bottom kernel, one launch a V-cycle: the
first cycle, one an iteration, at most two iterations past the last one
needed, and never fewer than the eight of a first look.
"""
import numpy as np
import pytest

import synth
from cases import instance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hv = pytest.importorskip("paper_1909_03948_amd.hinv")


def test_iterations_enqueued():
    print("[gpu-p2l]", flush=True)
    prob, _, obs = instance(16, 10, state_degree=2)
    N = 32
    ctx = hv.Context(0)
    gp = hv.Problem(ctx, N, prob.gamma, prob.delta, obs_xy=obs, d_obs=prob.d, sigma=prob.sigma, beta=prob.beta,
                    precision=hv.PREC_FP64, rtol=1e-10, state_degree=2)
    ns = (2 * N + 1) ** 2
    dev = lambda x: torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")
    zero = dev(np.zeros(ns))
    gp.linearize(dev(0.4 * synth.smooth_field(N)), zero, zero)
    B = synth.test_vectors(ns, 3, seed=93).reshape(3, ns)

    def solve(nc, rtol, max_iter, scale=1.0):
        gp.set_solver(hv.PREC_FP64, rtol, max_iter)
        ctx.kernel_timer("mg_bottom", True, 1 << 20)
        info = gp.state_solve(dev(scale * B[:nc]), dev(np.zeros((nc, ns))))
        n = ctx.kernel_timer_read("mg_bottom")["launches"]
        ctx.kernel_timer("mg_bottom", False, 1)
        print(f"[gpu-p2l] nc={nc} rtol={rtol} cap={max_iter}: {info['iterations']} iterations, {n} cycles", flush=True)
        return info, n

    def bounded(info, n):
        assert info["rc"] == hv.HINV_OK
        assert n <= 1 + max(8, info["iterations"] + 2)

    for _ in range(2):
        bounded(*solve(1, 1e-10, 200))
    info, n = solve(1, 1e-100, 60)   # out of reach
    assert info["rc"] == hv.HINV_ENOCONV and info["iterations"] == 60 and n == 61
    bounded(*solve(1, 1e-10, 200))
    bounded(*solve(1, 1e-2, 200))
    bounded(*solve(3, 1e-2, 200))
    bounded(*solve(1, 1e-100, 60, scale=0.0))  # a zero column after the failed solve
