"""The charge deposit's block sums in LDS against the oracle: tile-sorted and
unsorted ensembles, ragged last blocks, grids the box wraps around, weights many
orders of magnitude apart, and a weight that is not finite."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import pic

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1409_5574_amd import api
    api.lib()
    return api


def _case(dim, n_grid, count, weights, order, rng):
    dx = (0.3, 0.25, 0.35)
    box = np.array([n_grid[a] * dx[a] for a in range(dim)])
    pos = (rng.uniform(0, 1, (count, dim)) * box).astype(np.float32)
    pos = np.where(pos >= box.astype(np.float32), 0.0, pos).astype(np.float32)
    if order == "sorted":
        cell = np.floor(pos.astype(np.float64) / np.array(dx[:dim])).astype(np.int64)
        pos = pos[np.lexsort([cell[:, a] // 4 for a in range(dim)])]
    w = {"equal": np.ones(count), "wide": 10.0 ** rng.uniform(-6, 6, count),
         "zeros": np.where(rng.uniform(size=count) < 0.5, 0.0, 1.0)}[weights].astype(np.float32)
    return dx, pos, w


def _touching(pos, w, dim, n, dx):
    """Sum of |w| over the particles that have each node in their stencil."""
    out = np.zeros(int(np.prod(n)))
    u = [pos[:, a].astype(np.float64) / dx[a] for a in range(dim)]
    # a fraction within rounding of a cell face may put a particle on either side of it
    for corner in np.ndindex(*(4,) * dim):
        idx, mul = 0, 1
        for a in range(dim):
            idx = idx + np.mod(np.floor(u[a]).astype(np.int64) - 1 + corner[a], n[a]) * mul
            mul *= n[a]
        np.add.at(out, idx, np.abs(w.astype(np.float64)))
    return out


@pytest.mark.parametrize("dim, n, count, weights, order", [
    (3, (32, 24, 20), 6001, "equal", "sorted"),
    (3, (32, 24, 20), 6001, "wide", "sorted"),
    (3, (64, 64, 64), 4000, "equal", "unsorted"),       # boxes over the window: direct adds
    (3, (2, 3, 2), 1500, "wide", "unsorted"),           # boxes that wrap round the grid
    (3, (16, 16, 16), 1, "equal", "unsorted"),
    (3, (16, 16, 16), 513, "zeros", "sorted"),          # one past a full block
    (2, (96, 80, 1), 7000, "wide", "sorted"),
    (2, (96, 80, 1), 7000, "zeros", "unsorted"),
    (2, (2, 2, 1), 512, "equal", "unsorted"),
])
def test_charge_box_matches_oracle(sr, dim, n, count, weights, order):
    print(f"[gpu-case] rho {dim}D {n} {count} {weights} {order}", flush=True)
    rng = np.random.default_rng(7 * count + dim)
    dx, pos, w = _case(dim, n, count, weights, order, rng)
    st = {"x": pos[:, 0].copy(), "y": pos[:, 1].copy(), "z": pos[:, 2].copy() if dim == 3 else None,
          "px": np.zeros(count), "py": np.zeros(count), "pz": np.zeros(count), "w": w,
          "id": np.arange(count, dtype=np.uint32)}
    parts = sr.Particles.from_numpy(st, dim=dim)
    grid = sr.grid_struct(dim, n=n, dx=dx)
    rho = torch.zeros(int(np.prod(n)), device="cuda", dtype=torch.float32)
    sr.deposit_rho(parts, grid, -1.0, rho)
    got = rho.cpu().numpy().astype(np.float64)
    ref = pic.deposit_rho(pos.astype(np.float64), w.astype(np.float64), -1.0, dim, n, dx).ravel()
    # a fraction is within 2^-23 (two roundings), a weight of up to three of them and
    # its product with q w / dV within 12 units of 2^-24 of the particle's q w / dV, and
    # the sums of a node's few blocks round within 4 more
    tol = 16 * 2.0 ** -24 * _touching(pos, w, dim, n, dx) / np.prod(dx[:dim])
    assert np.all(np.abs(got - ref) <= tol + 1e-300)


def test_charge_of_a_nonfinite_weight_stays_on_its_nodes(sr):
    n, dx, count = (24, 24, 24), (0.3, 0.25, 0.35), 1000
    rng = np.random.default_rng(5)
    _, pos, w = _case(3, n, count, "equal", "sorted", rng)
    pos[300] = np.array([3.5 * dx[0], 4.5 * dx[1], 5.5 * dx[2]], np.float32)
    w[300] = np.nan
    st = {"x": pos[:, 0].copy(), "y": pos[:, 1].copy(), "z": pos[:, 2].copy(), "px": np.zeros(count),
          "py": np.zeros(count), "pz": np.zeros(count), "w": w, "id": np.arange(count, dtype=np.uint32)}
    print("[gpu-case] rho nan weight", flush=True)
    rho = torch.zeros(n[0] * n[1] * n[2], device="cuda", dtype=torch.float32)
    sr.deposit_rho(sr.Particles.from_numpy(st), sr.grid_struct(3, n=n, dx=dx), -1.0, rho)
    bad = np.isnan(rho.cpu().numpy().reshape(n[2], n[1], n[0]))
    assert bad[5:7, 4:6, 3:5].all() and bad.sum() == 8
