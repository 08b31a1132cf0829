"""GPU: probe blocks with more columns than the Gauss-Newton Hessian has rank
(q observations), beyond the one-workgroup eigenproblems.  The block then spans
the whole range, so the double pass is exact whatever the probes: its
eigenvalues are the pencil's, to the parity bar 1e-8 lambda_1, and its vectors
R-orthonormal to 1e-8.  Rounding noise of the Gram matrix may look like a
direction; no draw of the probes may make the call break down.
"""
import functools

import numpy as np
import pytest
import scipy.linalg

import synth
from cases import instance
from oracle import model

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hv = pytest.importorskip("paper_1909_03948_amd.hinv")


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


@functools.lru_cache(maxsize=None)
def exact(N, q):
    """The pencil's eigenvalues from H = J^T J: H R^-1 has the nonzero eigenvalues
    of the q x q matrix J R^-1 J^T, J from the Hessian's action on a basis."""
    prob, _, obs = instance(N, q)
    m = prob.m_pr + 0.4 * synth.smooth_field(N)
    u = prob.forward(m)
    p = prob.adjoint(m, u)
    rng = np.random.default_rng(5)
    X = rng.standard_normal((q + 20, prob.n))
    HX = np.array([prob.hessian_apply(m, u, p, x, model.HESS_GN_MISFIT) for x in X])  # spans the range
    Q = scipy.linalg.qr(HX.T, mode="economic", pivoting=True)[0][:, :q]
    RQ = np.array([prob.R_solve(v) for v in Q.T])           # R^-1 of a basis of the range
    A = np.array([prob.hessian_apply(m, u, p, v, model.HESS_GN_MISFIT) for v in RQ])
    T = RQ @ A.T                                            # (R^-1 Q)^T H (R^-1 Q)
    B = RQ @ Q                                              # (R^-1 Q)^T R (R^-1 Q)
    return prob, obs, m, u, p, scipy.linalg.eigh(0.5 * (T + T.T), 0.5 * (B + B.T), eigvals_only=True)[::-1]


@pytest.mark.parametrize("q,s", [(50, 72), (50, 150), (70, 100), (70, 250)])
def test_blocks_wider_than_the_rank(q, s):
    N, k = 32, q // 2
    prob, obs, m, u, p, ref = exact(N, q)
    gp = hv.Problem(hv.Context(0), N, prob.gamma, prob.delta, obs_xy=obs, d_obs=prob.d, sigma=prob.sigma,
                    m_prior=prob.m_pr[0], beta=prob.beta, precision=hv.PREC_AUTO, rtol=1e-10)
    gp.linearize(dev(m), dev(u), dev(p))
    for seed in range(1, 9):
        V, W = dev(np.zeros((k, prob.n))), dev(np.zeros((k, prob.n)))
        lam, info = gp.lowrank_eig(dev(synth.omega(prob.n, s, seed=seed)), k, V, mode=hv.HESS_GN_MISFIT)
        assert info["rc"] == hv.HINV_OK, info
        gp.prior_apply(V, W)
        torch.cuda.synchronize()
        o = np.abs((V @ W.T.contiguous()).cpu().numpy() - np.eye(k)).max()
        e = np.max(np.abs(lam - ref[:k])) / ref[0]
        print(f"[gpu-rank] q={q} s={s} seed={seed}: {e:.1e}, orthonormal to {o:.1e}", flush=True)
        assert e <= 1e-8 and o <= 1e-8
