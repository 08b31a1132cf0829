"""GPU: batches under every segment length the tuner may pick (and lengths that
leave a remainder), with one and two columns a wave and an odd number of
columns (the last wave's second column repeats the last one), on one problem
and on two stacked ones.  Every column of the Hessian actions and of the prior
solves against the oracle, to the parity bar of the Hessian tests.
"""
import functools

import numpy as np
import pytest

import synth
from cases import col_rel, instance
from oracle import model

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hv = pytest.importorskip("paper_1909_03948_amd.hinv")

SHAPES = [f"l1c{c}r{r}" for r in (1, 2, 5, 13, 29) for c in (1, 2)] + ["s1c3r13"]
NC = 9


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


@functools.lru_cache(maxsize=None)
def reference(N, seed):
    prob, _, obs = instance(N, 100, seed=seed)
    m = prob.m_pr + 0.5 * synth.smooth_field(N, seed=seed)
    u = prob.forward(m)
    p = prob.adjoint(m, u)
    X = synth.test_vectors(prob.n, NC, seed=seed)
    return (prob, obs, m, u, p, X, np.array([prob.hessian_apply(m, u, p, v, model.HESS_GN_MISFIT) for v in X]),
            np.array([prob.R_solve(v) for v in X]))


def problem(ctx, N, seed):  # a new one: it captures its graphs under the forced shape
    prob, obs, m, u, p, *_ = reference(N, seed)
    gp = hv.Problem(ctx, N, prob.gamma, prob.delta, obs_xy=obs, d_obs=prob.d, sigma=prob.sigma,
                    m_prior=prob.m_pr[0], beta=prob.beta, precision=hv.PREC_AUTO, rtol=1e-10)
    gp.linearize(dev(m), dev(u), dev(p))
    return gp


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("N", [64, 256])
def test_segments_and_columns_a_wave(N, shape, monkeypatch):
    print(f"[gpu-seg] N={N} {shape}", flush=True)
    monkeypatch.setenv("HINV_SHAPE", shape)
    gp = problem(hv.Context(0), N, 41)
    X, H, R = reference(N, 41)[5:]
    Y, Z = dev(np.zeros_like(X)), dev(np.zeros_like(X))
    for info in (gp.hessian_apply(hv.HESS_GN_MISFIT, dev(X), Y), gp.prior_solve(dev(X), Z)):
        assert info["rc"] == 0 and info["max_relres"] <= 1e-10, info
    torch.cuda.synchronize()
    e = col_rel(Y.cpu().numpy(), H), col_rel(Z.cpu().numpy(), R)
    print(f"[gpu-seg] {e[0]:.1e} {e[1]:.1e}", flush=True)
    assert max(e) <= 1e-8


@pytest.mark.parametrize("shape", SHAPES)
def test_stacked_segments_and_columns_a_wave(shape, monkeypatch):
    print(f"[gpu-seg] stacked {shape}", flush=True)
    monkeypatch.setenv("HINV_SHAPE", shape)
    ctx = hv.Context(0)
    gps = [problem(ctx, 64, s) for s in (41, 42)]
    refs = [reference(64, s) for s in (41, 42)]
    outs = [dev(np.zeros_like(r[5])) for r in refs]
    info = hv.Batch(ctx, gps).hessian_apply(hv.HESS_GN_MISFIT, [dev(r[5]) for r in refs], outs)
    assert info["rc"] == 0 and info["max_relres"] <= 1e-10, info
    torch.cuda.synchronize()
    for o, r in zip(outs, refs):
        e = col_rel(o.cpu().numpy(), r[6])
        print(f"[gpu-seg] {e:.1e}", flush=True)
        assert e <= 1e-8


@pytest.mark.parametrize("shape", ["s1", "s2", "s3", "s4", "s16", "s1k320", "s2k960", "s3k704", "s4k4032", "l3"])
@pytest.mark.parametrize("nc", [1, 7])
def test_partitions_of_few_columns(nc, shape, monkeypatch):
    """The linear apply kernel of few columns: one or two virtual threads a
    thread, whole blocks and chunks that end inside one."""
    print(f"[gpu-seg] few nc={nc} {shape}", flush=True)
    N = 256
    monkeypatch.setenv("HINV_SHAPE", shape)
    gp = problem(hv.Context(0), N, 41)
    X, H, R = (a[:nc] for a in reference(N, 41)[5:])
    Y, Z = dev(np.zeros_like(X)), dev(np.zeros_like(X))
    for info in (gp.hessian_apply(hv.HESS_GN_MISFIT, dev(X), Y), gp.prior_solve(dev(X), Z)):
        assert info["rc"] == 0 and info["max_relres"] <= 1e-10, info
    torch.cuda.synchronize()
    e = col_rel(Y.cpu().numpy(), H), col_rel(Z.cpu().numpy(), R)
    print(f"[gpu-seg] {e[0]:.1e} {e[1]:.1e}", flush=True)
    assert max(e) <= 1e-8
