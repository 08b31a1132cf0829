"""GPU: eigenproblems of large stacked batches, on both sides of the line between
the one-workgroup and the blocked sweeps (32 matrices up to s = 72, 49 up to 80):
a batch's eigenvalues and eigenvectors equal those of its members' own double
passes, where s > 56 always takes the blocked sweeps.

Bars of the double-pass tests: eigenvalues to 1e-8 lambda_1, R-orthonormal
vectors to 1e-8, and V spanning the members' (cosines of leading vectors).
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


@pytest.mark.parametrize("nb,s", [(31, 72), (32, 65), (32, 72), (48, 73), (49, 73), (49, 80), (40, 64)])
def test_stacked_eigenproblems(nb, s):
    print(f"[gpu-eigb] nb={nb} s={s}", flush=True)
    N, q, k = 16, 150, 12
    prob, _, obs = instance(N, q)
    n = prob.n
    ctx = hv.Context(0)
    zero, gps = dev(np.zeros(n)), []
    for j in range(nb):
        gp = hv.Problem(ctx, N, prob.gamma, prob.delta, obs_xy=obs, d_obs=prob.d, sigma=prob.sigma, beta=prob.beta,
                        m_prior=prob.m_pr[0], precision=hv.PREC_FP64, rtol=1e-10)
        m, u, p = dev(prob.m_pr + 0.3 * synth.smooth_field(N, seed=50 + j)), dev(np.zeros(n)), dev(np.zeros(n))
        gp.forward(m, u)
        gp.gradient(m, u, p, dev(np.zeros(n)))
        gp.linearize(m, u, p)
        gps.append(gp)
    oms = [dev(synth.omega(n, s, seed=200 + j)) for j in range(nb)]
    Vs = [dev(np.zeros((k, n))) for _ in range(nb)]
    lam, info = hv.Batch(ctx, gps).lowrank_eig(oms, k, Vs, mode=hv.HESS_GN_MISFIT)
    assert info["rc"] == 0, info
    for j in (0, 1, nb // 2, nb - 1):
        V = dev(np.zeros((k, n)))
        own, info = gps[j].lowrank_eig(oms[j], k, V, mode=hv.HESS_GN_MISFIT)
        assert info["rc"] == 0, info
        W = dev(np.zeros((k, n)))
        gps[j].prior_apply(Vs[j], W)
        torch.cuda.synchronize()
        e = np.max(np.abs(lam[j] - own)) / own[0]
        o = (Vs[j] @ W.T.contiguous()).cpu().numpy()
        c = (V[:1] @ W[:1].T.contiguous()).cpu().numpy()
        print(f"[gpu-eigb] member {j}: {e:.1e} orth {np.abs(o - np.eye(k)).max():.1e} cos {abs(c[0, 0]):.12f}", flush=True)
        assert e <= 1e-8 and np.abs(o - np.eye(k)).max() <= 1e-8 and abs(abs(c[0, 0]) - 1.0) <= 1e-8
