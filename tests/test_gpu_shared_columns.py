"""GPU: kernels that read the operator or the linearization point once for
four columns (from eight columns on): a batch's Hessian action equals the
columns' own, at column counts around the group of four, in FP64.

Both sides solve to 1e-10; the bar is the batch tests' 1e-8.
"""
import numpy as np
import pytest

import synth
from cases import col_rel, instance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hv = pytest.importorskip("paper_1909_03948_amd.hinv")


@pytest.mark.parametrize("mode", [hv.HESS_FULL, hv.HESS_GN_MISFIT])
@pytest.mark.parametrize("nc", [7, 8, 9, 11, 13])
def test_batch_matches_columns(mode, nc):
    print(f"[gpu-share] nc={nc} mode={mode}", flush=True)
    N = 64
    prob, _, obs = instance(N, 60)
    dev = lambda x: torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")
    m = prob.m_pr + 0.5 * synth.smooth_field(N)
    u = prob.forward(m)
    gp = hv.Problem(hv.Context(0), N, prob.gamma, prob.delta, obs_xy=obs, d_obs=prob.d, sigma=prob.sigma,
                    m_prior=prob.m_pr[0], beta=prob.beta, precision=hv.PREC_FP64, rtol=1e-10)
    gp.linearize(dev(m), dev(u), dev(prob.adjoint(m, u)))
    X = synth.test_vectors(prob.n, nc, seed=63)
    Y = dev(np.zeros_like(X))
    assert gp.hessian_apply(mode, dev(X), Y)["rc"] == 0
    Z = np.zeros_like(X)
    for c in range(nc):
        z = dev(np.zeros((1, prob.n)))
        assert gp.hessian_apply(mode, dev(X[c:c + 1]), z)["rc"] == 0
        torch.cuda.synchronize()
        Z[c] = z.cpu().numpy()
    e = col_rel(Y.cpu().numpy(), Z)
    print(f"[gpu-share] {e:.1e}", flush=True)
    assert e <= 1e-8
