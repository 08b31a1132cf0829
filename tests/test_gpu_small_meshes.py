"""GPU: meshes whose whole hierarchy runs in one workgroup (N <= 32; N = 64 for
the other path beside it): state and prior solves against the FP64 oracle for
one column, few columns and FP32 refinement, with a zero column, and the
iteration cap.

Tolerance: the solver's bar of 1e-8 against direct solves at 1e-10 relative
residual.  The cap stops at 1 + 2 floor(max_iter / 2) iterations (they come in
pairs after the first) with HINV_ENOCONV.
"""
import numpy as np
import pytest

import synth
from cases import col_rel, instance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hv = pytest.importorskip("paper_1909_03948_amd.hinv")


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


def setup(N):
    prob, _, obs = instance(N, 10)
    m = prob.m_pr + 0.5 * synth.smooth_field(N)
    gp = hv.Problem(hv.Context(0), N, prob.gamma, prob.delta, obs_xy=obs, d_obs=prob.d, sigma=prob.sigma,
                    m_prior=prob.m_pr[0], beta=prob.beta, precision=hv.PREC_AUTO, rtol=1e-10)
    zero = dev(np.zeros(prob.n))
    gp.linearize(dev(m), zero, zero)
    return prob, m, gp


@pytest.mark.parametrize("N", [4, 8, 16, 32, 64])
@pytest.mark.parametrize("nc", [1, 3, 9])
def test_small_mesh_solves(N, nc):
    print(f"[gpu-small] N={N} nc={nc}", flush=True)
    prob, m, gp = setup(N)
    B = synth.test_vectors(prob.n, nc, seed=71)
    if nc > 1:
        B[1] = 0.0
    Bs = B * prob.free
    X, Y = dev(np.zeros_like(B)), dev(np.zeros_like(B))
    i1, i2 = gp.state_solve(dev(Bs), X), gp.prior_solve(dev(B), Y)
    torch.cuda.synchronize()
    ref = np.zeros_like(B)
    for c in range(nc):
        ref[c, prob.free] = prob._solve_free(m, Bs[c, prob.free])
    es = col_rel(X.cpu().numpy(), ref)
    ep = col_rel(Y.cpu().numpy(), np.array([prob.R_solve(b) for b in B]))
    print(f"[gpu-small] state {es:.1e} ({i1['iterations']} iterations), prior {ep:.1e}", flush=True)
    assert i1["rc"] == 0 and i2["rc"] == 0 and es <= 1e-8 and ep <= 1e-8


@pytest.mark.parametrize("max_iter,taken", [(1, 1), (2, 3), (3, 3)])
def test_small_mesh_iteration_cap(max_iter, taken):
    prob, _, gp = setup(32)
    b = dev(synth.test_vectors(prob.n, 1, seed=72) * prob.free)
    x = torch.zeros_like(b)
    gp.set_solver(hv.PREC_FP64, 1e-10, max_iter)
    info = gp.state_solve(b, x)
    print(f"[gpu-small] cap {max_iter}: {info}", flush=True)
    assert info["rc"] == hv.HINV_ENOCONV and info["iterations"] == taken
    gp.set_solver(hv.PREC_FP64, 1e-10, 0)
    info = gp.state_solve(b, x)
    assert info["rc"] == 0 and info["max_relres"] <= 1e-10
