"""GPU: columns of a quadratic-state solve do not depend on each other.  Columns
that end at different iterations (zero, an eigenvector-like smooth mode, rough
ones, one with a NaN) come out as in a call of their own, bit for bit: the sums
of a column are taken by its own workgroups in a fixed order.
"""
import numpy as np
import pytest

import synth
from cases import instance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hv = pytest.importorskip("paper_1909_03948_amd.hinv")


@pytest.mark.parametrize("N", [16, 64])
def test_columns_end_on_their_own(N):
    print(f"[gpu-p2c] N={N}", flush=True)
    prob, _, obs = instance(16, 10, state_degree=2)
    gp = hv.Problem(hv.Context(0), N, prob.gamma, prob.delta, obs_xy=obs, d_obs=prob.d, sigma=prob.sigma,
                    beta=prob.beta, precision=hv.PREC_AUTO, rtol=1e-10, state_degree=2)
    dev = lambda x: torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")
    S = 2 * N + 1
    zero = dev(np.zeros(S * S))
    gp.linearize(dev(0.4 * synth.smooth_field(N)), zero, zero)
    y = np.linspace(0, 1, S)
    B = np.zeros((6, S, S))
    B[1] = np.sin(np.pi * y)[:, None]
    B[2] = np.sin(7 * np.pi * y)[:, None]
    B[3:] = synth.test_vectors(S * S, 3, seed=92).reshape(3, S, S)
    B[5, S // 2, 3] = np.nan
    B = B.reshape(6, -1)
    X = dev(np.ones_like(B))
    assert gp.state_solve(dev(B), X)["rc"] == hv.HINV_ENOCONV  # the column with a NaN
    its = set()
    for c in range(5):
        x = dev(np.ones_like(B[c:c + 1]))
        info = gp.state_solve(dev(B[c:c + 1]), x)
        assert info["rc"] == hv.HINV_OK
        its.add(info["iterations"])
        torch.cuda.synchronize()
        assert np.array_equal(X[c].cpu().numpy(), x[0].cpu().numpy()), c
    print(f"[gpu-p2c] iterations {sorted(its)}", flush=True)
    assert len(its) > 1 and 0 in its
