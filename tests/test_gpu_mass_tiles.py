"""GPU: the prior operator R = K M^-1 K (its mass solve runs on tiles of 64
columns by 32 or 64 rows with a halo of 12) at the edges of those tiles and on
both sides of the rule that picks them, against the FP64 oracle.

Tolerance: 24 Chebyshev steps leave 2 (1/3)^24 = 7.1e-12 of M^-1's result; K
amplifies it by at most its condition number on what the vectors hold, for
the random vectors used here (all frequencies alike) by a factor of order one;
FP64 rounding is below.  2e-11.
"""
import numpy as np
import pytest

import synth
from cases import instance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hv = pytest.importorskip("paper_1909_03948_amd.hinv")


# owned columns 40 a tile: 33, 65, 129 nodes = 1, 2, 4 strips; owned rows 8 or 40:
# 64 x 39 and 64 x 40 columns lie on both sides of 160 workgroups
@pytest.mark.parametrize("N,nc", [(4, 1), (8, 3), (32, 2), (64, 39), (64, 40), (128, 1)])
def test_prior_apply_across_tiles(N, nc):
    print(f"[gpu-mass] N={N} nc={nc}", flush=True)
    prob, _, obs = instance(N, 10)
    gp = hv.Problem(hv.Context(0), N, prob.gamma, prob.delta, obs_xy=obs, d_obs=prob.d, sigma=prob.sigma,
                    precision=hv.PREC_AUTO, rtol=1e-10)
    X = synth.test_vectors(prob.n, nc, seed=61)
    dev = lambda x: torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")
    Y = dev(np.zeros_like(X))
    gp.prior_apply(dev(X), Y)
    torch.cuda.synchronize()
    Y = Y.cpu().numpy()
    for c in {0, nc // 2, nc - 1}:
        ref = prob.R_apply(X[c])
        e = np.linalg.norm(Y[c] - ref) / np.linalg.norm(ref)
        print(f"[gpu-mass] column {c}: {e:.1e}", flush=True)
        assert e <= 2e-11
