"""GPU: the s x s factorizations of the randomized algorithms at the edges of
their block sizes, against the FP64 oracle.

The prior's pointwise variance with the same s probes runs Cholesky factors,
triangular inverses and a symmetric eigenproblem of size s.  Tolerances: the
solves leave 1e-10 relative residuals and the factorizations work in FP64, so
the diagonal is held to 1e-8 relative and the eigenvalues to 1e-8 of the
largest, the bounds of the pointwise-variance test at smaller s.
"""
import numpy as np
import pytest

import synth
from cases import instance, rel
from oracle import lowrank

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hv = pytest.importorskip("paper_1909_03948_amd.hinv")


# 56 | 57: one-workgroup eigensolver | blocked; 64 | 65, 96 | 97, 128 | 129: its
# padding; 5, 31, 32, 33, 160: tiles of 32 and 16
@pytest.mark.parametrize("s", [5, 31, 32, 33, 56, 57, 64, 65, 72, 73, 96, 97, 129, 160])
def test_factorizations_at_block_edges(s):
    print(f"[gpu-dense] s={s}", flush=True)
    prob, _, obs = instance(32, 10)
    Om = synth.omega(prob.n, s, seed=23)
    dg_o, mu_o = lowrank.prior_variance(prob.R_solve, Om.T)
    gp = hv.Problem(hv.Context(0), prob.N, prob.gamma, prob.delta, obs_xy=obs, d_obs=prob.d,
                    sigma=prob.sigma, precision=hv.PREC_AUTO, rtol=1e-10, max_iter=400)
    diag = torch.zeros(prob.n, dtype=torch.float64, device="cuda")
    mu, info = gp.prior_variance(torch.as_tensor(Om, device="cuda"), diag)
    torch.cuda.synchronize()
    e_d, e_mu = rel(diag.cpu().numpy(), dg_o), np.max(np.abs(mu - mu_o)) / mu_o[0]
    print(f"[gpu-dense] s={s}: diag rel {e_d:.2e}, mu {e_mu:.2e}", flush=True)
    assert info["rc"] == 0 and np.all(np.diff(mu) <= 0.0)
    assert e_d <= 1e-8 and e_mu <= 1e-8
