"""The network's products at the edges of their tiles, chunks and K splits: one row,
one unit, sizes that are no multiple of four (scalar loads), partial tiles and
chunks, and an output layer long enough to be split.  Against the FP64 reference at
the bars of the network's other tests: sums of up to n FP32 products."""
import numpy as np
import pytest
import torch

from oracle import mlp_oracle as M
from paper_2311_08050_amd import binding

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    return binding.Library()


@pytest.mark.parametrize("I,H,O,B", [(1, 1, 1, 1), (4, 32, 100, 16), (3, 33, 257, 17), (4, 100, 515, 65), (2, 64, 1023, 3),
                                     (4, 128, 2052, 64), (4, 256, 4099, 100), (5, 260, 640, 129)])
def test_forward_and_gradient(lib, I, H, O, B):
    rng = np.random.default_rng(H + O)
    p = np.concatenate([a.reshape(-1) for a in (
        rng.uniform(-1, 1, (H, I)) * np.sqrt(6 / I), rng.normal(0, 0.1, H), rng.uniform(-1, 1, (H, H)) * np.sqrt(6 / H),
        rng.normal(0, 0.1, H), rng.uniform(-1, 1, (O, H)) * np.sqrt(3 / H), rng.normal(0, 0.1, O))]).astype(np.float32)
    u, t = rng.normal(size=(B, I)).astype(np.float32), rng.normal(size=(B, O))
    net = binding.Mlp(lib, I, H, O)
    net.set_params(torch.tensor(p))
    ref, _ = M.forward(p.astype(np.float64), u.astype(np.float64), I, H, O)
    y = net.forward(torch.tensor(u)).cpu().numpy()
    assert np.max(np.abs(y - ref)) <= 1e-5 * max(1.0, np.max(np.abs(ref)))
    loss, g = net.grad(torch.tensor(u), torch.tensor(t))
    ref_loss, ref_g = M.grad(p.astype(np.float64), u.astype(np.float64), t, I, H, O)
    assert abs(loss - ref_loss) <= 1e-5 * ref_loss
    g, off = g.cpu().numpy().astype(np.float64), 0
    for _, shape in M.sizes(I, H, O):
        c = int(np.prod(shape))
        a, b = g[off:off + c], ref_g[off:off + c]
        assert np.max(np.abs(a - b)) <= 1e-4 * np.max(np.abs(b)), (shape, np.max(np.abs(a - b)))
        off += c
