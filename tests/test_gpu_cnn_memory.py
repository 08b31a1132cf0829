"""GPU: the network's forward pass holds no memory of the backward pass: the
per-tile partials of the weight gradients (9 x 32 x 32 + 32 floats a tile and
layer) come with the first gradient.
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hv = pytest.importorskip("paper_1909_03948_amd.hinv")


@pytest.mark.parametrize("S", [129, 513])
def test_partials_come_with_the_gradient(S):
    print(f"[gpu-cnnmem] S={S}", flush=True)
    alloc = hv.TorchAllocator(0)
    net = hv.Cnn(hv.Context(0, allocator=alloc))
    net.he_init(1)
    f32 = lambda *s: torch.ones(*s, dtype=torch.float32, device="cuda")
    out = f32(1, S, S)
    net.forward(f32(1, 3, S, S), out)
    torch.cuda.synchronize()
    forward = alloc.live_bytes
    net.gradient(f32(1, 3, S, S), out)
    grown = alloc.live_bytes - forward
    partials = 6 * ((S + 15) // 16) ** 2 * (9 * 32 * 32 + 32) * 4
    print(f"[gpu-cnnmem] forward {forward / 2**20:.1f} MiB, gradient {grown / 2**20:.1f} MiB more, partials "
          f"{partials / 2**20:.1f} MiB", flush=True)
    assert grown >= partials
    net.gradient(f32(1, 3, S, S), out)
    assert alloc.live_bytes == forward + grown
