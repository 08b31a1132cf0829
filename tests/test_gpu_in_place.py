"""GPU: state solves whose right-hand sides and solutions share memory, in place
(x = b) or shifted against each other, equal the solve with separate vectors.

Linear state: the same FP64 solve, to the parity bar of the Hessian tests.
Quadratic state: the same kernels on the same numbers, so bit for bit.
"""
import numpy as np
import pytest

import synth
from cases import col_rel, instance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hv = pytest.importorskip("paper_1909_03948_amd.hinv")


@pytest.mark.parametrize("shift", [0, 1, 77, -40])
@pytest.mark.parametrize("degree,N,nc", [(1, 32, 1), (1, 64, 9), (2, 4, 2), (2, 32, 1), (2, 32, 9), (2, 64, 1),
                                         (2, 64, 9)])
def test_state_solve_with_overlapping_vectors(degree, N, nc, shift):
    print(f"[gpu-inplace] degree={degree} N={N} nc={nc} shift={shift}", flush=True)
    prob, _, obs = instance(16, 10, state_degree=degree)
    gp = hv.Problem(hv.Context(0), N, prob.gamma, prob.delta, obs_xy=obs, d_obs=prob.d, sigma=prob.sigma,
                    beta=prob.beta, precision=hv.PREC_FP64, rtol=1e-10, state_degree=degree)
    dev = lambda x: torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")
    ns = (degree * N + 1) ** 2
    zero = dev(np.zeros(ns))
    gp.linearize(dev(-2.0 + 0.4 * synth.smooth_field(N)), zero, zero)
    B = synth.test_vectors(ns, nc, seed=91).reshape(nc, ns)
    ref = dev(np.zeros_like(B))
    assert gp.state_solve(dev(B), ref)["rc"] == hv.HINV_OK
    buf = torch.zeros(nc * ns + abs(shift), dtype=torch.float64, device="cuda")
    at = lambda o: buf[o:o + nc * ns].view(nc, ns)
    b, x = at(max(-shift, 0)), at(max(shift, 0))
    b.copy_(dev(B))
    assert gp.state_solve(b, x)["rc"] == hv.HINV_OK
    torch.cuda.synchronize()
    x, ref = x.cpu().numpy(), ref.cpu().numpy()
    if degree == 2:
        assert np.array_equal(x, ref)
    else:
        assert col_rel(x, ref) <= 1e-8
