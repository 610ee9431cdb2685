"""The network's entry points at the edges of their tiles and grids, against the FP64
oracle: inference on a partial tile and past one pass of its blocks, and the gradient
of batches that fill one wave, some blocks, or every wave several times."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import mlp as omlp

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1409_5574_amd import api
    api.lib()
    return api


def _net(sr, seed):
    flat = omlp.bf16_round(omlp.init(seed))
    return flat, sr.Mlp(flat.astype(np.float32))


@pytest.mark.parametrize("M", [1, 15, 16, 17, 64, 65, 4097, 32768 + 5, 70001])
def test_forward_sizes(sr, M):
    print(f"[gpu-case] mlp forward {M}", flush=True)
    flat, net = _net(sr, 11)
    f = np.random.default_rng(M).uniform(-1.3, 1.3, (M, 2)).astype(np.float32)
    y = net.forward(torch.from_numpy(f)).cpu().numpy().astype(np.float64)
    ref = omlp.forward(flat, f.astype(np.float64))
    # an activation keeps 16 bits or more (2^-17 of it lost), and of three layers of 64
    # such the errors add like their random signs: 3 * 8 * 2^-17 of a layer's scale
    assert np.abs(y - ref).max() <= 3 * 8 * 2.0 ** -17 * max(1.0, np.abs(ref).max())


@pytest.mark.parametrize("M", [1, 16, 63, 65, 1000, 16384, 16385, 20000])
def test_gradient_sizes(sr, M):
    print(f"[gpu-case] mlp gradient {M}", flush=True)
    flat, net = _net(sr, 12)
    rng = np.random.default_rng(M + 1)
    f = rng.uniform(-1.3, 1.3, (M, 2)).astype(np.float32)
    d = rng.uniform(-1.0, 1.0, M).astype(np.float32)
    ft, dt = torch.from_numpy(f).cuda(), torch.from_numpy(d).cuda()
    g = net.backward(ft, dt).cpu().numpy().astype(np.float64)
    # the batch in pieces of whole tiles, each through the same call: every tile's products
    # are the same (a sample's dout is not scaled by the batch), so only the sums differ
    parts = np.zeros_like(g)
    step = max(16, -(-M // 16 // 40) * 16)
    for i in range(0, M, step):
        parts += net.backward(ft[i:i + step], dt[i:i + step]).cpu().numpy().astype(np.float64)
    # 1024 rows at most are added one after another: 2^-24 of the largest partial sum each
    # in the worst case, their square root in the usual one; 4 times that, of the norm
    assert np.linalg.norm(g - parts) <= 4 * 32 * 2.0 ** -24 * np.linalg.norm(parts) + 1e-30


@pytest.mark.parametrize("M", [1, 16, 63, 65, 129])
def test_gradient_of_small_batches_matches_oracle(sr, M):
    """Partial tiles and batches of a few waves against the FP64 gradient itself."""
    print(f"[gpu-case] mlp gradient oracle {M}", flush=True)
    flat, net = _net(sr, 13)
    rng = np.random.default_rng(M + 2)
    f = rng.uniform(-1.2, 1.2, (M, 2)).astype(np.float32)
    d = rng.uniform(0.5, 1.0, M).astype(np.float32)
    g = net.backward(torch.from_numpy(f).cuda(), torch.from_numpy(d).cuda()).cpu().numpy().astype(np.float64)
    ref = omlp.backward(flat, f.astype(np.float64), d.astype(np.float64))
    # a value that enters a product in bfloat16 is 2^-9 off; a gradient passes four such at
    # most (dz3, dz2, an activation, dz1): 4 * 2^-9 of the largest of its array, 2.5 times
    at = 0
    for name, shape in omlp.SIZES:
        k = int(np.prod(shape))
        assert np.abs(g[at:at + k] - ref[at:at + k]).max() <= 2e-2 * np.abs(ref[at:at + k]).max() + 1e-12, name
        at += k
