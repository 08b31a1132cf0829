"""GPU: the quadratic state's solver at the sizes where its tiles and partial
sums change: meshes below, at and past a tile of 8 x 8 vertices, and past the
number of partial sums that a workgroup still adds up itself (N >= 184).

The solution is put back through the operator.  Its residual is the solver's
(1e-10 relative, recursively updated) plus the rounding of at most 25 updates,
each bounded by 2.2e-16 |A| |x| with |A| <= 16 max c_T (the largest absolute
row sum of the quadratic stiffness).
"""
import numpy as np
import pytest

import synth
from cases import instance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hv = pytest.importorskip("paper_1909_03948_amd.hinv")


@pytest.mark.parametrize("N,nc", [(4, 1), (4, 3), (32, 2), (64, 9), (128, 1), (256, 2)])
def test_p2_solves_across_tiles(N, nc):
    print(f"[gpu-p2t] N={N} nc={nc}", flush=True)
    m = 0.4 * synth.smooth_field(N)
    prob, _, obs = instance(16, 10, state_degree=2)
    gp = hv.Problem(hv.Context(0), N, prob.gamma, prob.delta, obs_xy=obs, d_obs=prob.d, sigma=prob.sigma,
                    beta=prob.beta, precision=hv.PREC_AUTO, rtol=1e-10, state_degree=2)
    dev = lambda x: torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")
    S = 2 * N + 1
    zero = dev(np.zeros(S * S))
    gp.linearize(dev(m), zero, zero)
    B = synth.test_vectors(S * S, nc, seed=90).reshape(nc, S, S)
    B[:, [0, -1]] = 0.0
    B[nc - 1] *= 0.0 if nc > 1 else 1.0   # a zero column among others
    B = B.reshape(nc, -1)
    X, R = dev(np.zeros_like(B)), dev(np.zeros_like(B))
    info = gp.state_solve(dev(B), X)
    gp.state_apply(X, R)
    torch.cuda.synchronize()
    X, R = X.cpu().numpy(), B - R.cpu().numpy()
    assert info["rc"] == hv.HINV_OK and info["iterations"] <= 25, info
    for c in range(nc):
        b, x = np.linalg.norm(B[c]), np.linalg.norm(X[c])
        tol = 1e-10 * b + 25 * 2.2e-16 * 16 * np.exp(m.max()) * x
        print(f"[gpu-p2t] column {c}: residual {np.linalg.norm(R[c]):.1e}, allowed {tol:.1e}", flush=True)
        assert np.linalg.norm(R[c]) <= tol
        assert b > 0 or not X[c].any()
