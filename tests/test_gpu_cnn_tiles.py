"""GPU: the network's gradient at the edges of its 16 x 16 pixel tiles, and on
both sides of the batch size from which the layers' partial sums share one
buffer (2400 tiles).

Tile edges: against the oracle on the BF16-rounded values, 1e-3 per layer, the
bar of the gradient test at other sizes.  Batch size: a batch of 4096 copies of
an image has the image's own loss and gradient (its 1/B is a power of two, so
every rounding of the device is the same); the sums over tiles are FP64 and the
result FP32, so they agree to 1e-6.
"""
import numpy as np
import pytest

from cases import rel
from oracle import cnn as ocnn
from test_gpu_cnn import f32, layer_slices, random_net

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hv = pytest.importorskip("paper_1909_03948_amd.hinv")


@pytest.mark.parametrize("B,S", [(3, 15), (2, 16), (2, 17)])
def test_gradient_at_tile_edges(B, S):
    print(f"[gpu-cnnt] B={B} S={S}", flush=True)
    theta, g = random_net(11), np.random.default_rng(12)
    x = g.standard_normal((B, 3, S, S)).astype(np.float32).astype(np.float64)
    t = g.standard_normal((B, 1, S, S)).astype(np.float32).astype(np.float64)
    net = hv.Cnn(hv.Context(0))
    net.set_params(theta)
    L, grad = net.gradient(f32(x), f32(t[:, 0]))
    L_o, grad_o = ocnn.gradient(theta, x, t, round_bf16=True)
    worst = max(rel(grad[sl].astype(np.float64), grad_o[sl]) for sl in layer_slices())
    print(f"[gpu-cnnt] loss {abs(L - L_o) / L_o:.1e}, worst layer {worst:.1e}", flush=True)
    assert abs(L - L_o) <= 1e-3 * L_o and worst < 1e-3


def test_gradient_of_many_copies():
    theta, g = random_net(13), np.random.default_rng(14)
    x, t = g.standard_normal((1, 3, 9, 9)), g.standard_normal((1, 9, 9))
    net = hv.Cnn(hv.Context(0))
    net.set_params(theta)
    L4, g4 = net.gradient(f32(np.repeat(x, 4096, 0)), f32(np.repeat(t, 4096, 0)))
    L1, g1 = net.gradient(f32(x), f32(t))
    e = rel(g4.astype(np.float64), g1.astype(np.float64))
    print(f"[gpu-cnnt] 4096 copies: loss {abs(L4 - L1) / L1:.1e}, gradient {e:.1e}", flush=True)
    assert abs(L4 - L1) <= 1e-6 * L1 and e <= 1e-6
