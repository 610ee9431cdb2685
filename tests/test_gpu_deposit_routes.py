"""The charge deposit on both sides of the sizes at which it changes its way, against the
64-bit oracle: added directly, in a box and in slabs."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import pic
from test_gpu_deposit import _case, _touching

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1409_5574_amd import api
    api.lib()
    return api


@pytest.mark.parametrize("dim, n, count, weights, order", [
    (3, (32, 32, 32), 24575, "wide", "sorted"),          # one add short of the box
    (3, (32, 32, 32), 24577, "wide", "sorted"),
    (3, (32, 32, 32), 24577, "equal", "unsorted"),       # no box: every block direct
    (3, (48, 48, 48), 40000, "wide", "sorted"),          # sparse: direct
    (3, (256, 128, 64), 262144, "equal", "sorted"),      # sparse, and large enough to look
    (2, (384, 384, 1), 49151, "zeros", "sorted"),
    (2, (384, 384, 1), 49153, "zeros", "sorted"),
    (2, (384, 384, 1), 49153, "wide", "unsorted"),
    (2, (5000, 3000, 1), 524288, "wide", "sorted"),
])
def test_charge_on_both_sides_of_the_rule(sr, dim, n, count, weights, order):
    print(f"[gpu-case] rho route {dim}D {n} {count} {weights} {order}", flush=True)
    rng = np.random.default_rng(count + dim)
    dx, pos, w = _case(dim, n, count, weights, order, rng)
    st = {"x": pos[:, 0].copy(), "y": pos[:, 1].copy(), "z": pos[:, 2].copy() if dim == 3 else None,
          "px": np.zeros(count), "py": np.zeros(count), "pz": np.zeros(count), "w": w,
          "id": np.arange(count, dtype=np.uint32)}
    rho = torch.zeros(int(np.prod(n)), device="cuda", dtype=torch.float32)
    sr.deposit_rho(sr.Particles.from_numpy(st, dim=dim), sr.grid_struct(dim, n=n, dx=dx), -1.0, rho)
    ref = pic.deposit_rho(pos.astype(np.float64), w.astype(np.float64), -1.0, dim, n, dx).ravel()
    # a contribution within 12 units of 2^-24 of the particle's q w / dV, and a rounding of
    # the running sum for each add to the node
    adds = _touching(pos, np.ones(count), dim, n, dx)
    tol = (16 + adds) * 2.0 ** -24 * _touching(pos, w, dim, n, dx) / np.prod(dx[:dim])
    assert np.all(np.abs(rho.cpu().numpy() - ref) <= tol + 1e-300)
