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


@pytest.mark.parametrize("dim, n, drift, far", [
    (3, (64, 48, 40), 0.0, 0.05),      # one box a block, a few crossings a wave
    (3, (64, 48, 40), 0.0, 1.0),
    (3, (256, 16, 16), 60.0, 0.3),     # x alone is wide: slabs, some round the grid
    (3, (48, 48, 48), 2.0, 0.3),
    (3, (48, 48, 48), 9.0, 0.3),       # over the slabs: window and direct adds
    (2, (700, 96, 1), 0.0, 0.05),
    (2, (700, 96, 1), 90.0, 0.3),
    (2, (3000, 2500, 1), 700.0, 1.0),
])
def test_current_and_charge_of_drifted_blocks_match_oracle(sr, dim, n, drift, far):
    """Particles in the order of the tiles they were in before a drift along x (and a
    tenth of it along the others); a share `far` of the moves up to 0.95 cell, the
    others 0.02 cell."""
    print(f"[gpu-case] current {dim}D {n} {drift} {far}", flush=True)
    count, dx, dt = 6001, np.array([0.3, 0.25, 0.35]), 0.11
    rng = np.random.default_rng(int(1000 * far + drift) + n[0])
    box = np.array(n[:dim]) * dx[:dim]

    def wrap(x):
        x = np.mod(x, box).astype(np.float32)
        return np.where(x >= box.astype(np.float32), 0.0, x).astype(np.float32)

    home = rng.uniform(0, 1, (count, dim)) * box
    cell = np.floor(home / dx[:dim]).astype(np.int64)
    home = home[np.lexsort([cell[:, a] // 4 for a in range(dim)])]
    p0 = wrap(home + rng.normal(0, 1, (count, dim)) * drift * np.array([1, 0.1, 0.1])[:dim] * dx[:dim])
    step = np.where(rng.uniform(size=(count, 1)) < far, 0.95, 0.02) * rng.uniform(-1, 1, (count, dim))
    p1 = wrap(p0.astype(np.float64) + step * dx[:dim])
    w = rng.uniform(0.5, 2.0, count).astype(np.float32)
    p = rng.normal(0, 1, (count, 3)).astype(np.float32)
    st = {"x": p1[:, 0].copy(), "y": p1[:, 1].copy(), "z": p1[:, 2].copy() if dim == 3 else None,
          "px": p[:, 0].copy(), "py": p[:, 1].copy(), "pz": p[:, 2].copy(), "w": w,
          "id": np.arange(count, dtype=np.uint32)}
    parts = sr.Particles.from_numpy(st, dim=dim)
    grid = sr.grid_struct(dim, n=n, dx=tuple(dx))
    old = [torch.from_numpy(p0[:, a].copy()).cuda() for a in range(dim)] + [None] * (3 - dim)
    J = [torch.zeros(int(np.prod(n)), device="cuda") for _ in range(3)]
    rho = torch.zeros(int(np.prod(n)), device="cuda")
    status = torch.zeros(1, device="cuda", dtype=torch.int32)
    sr.deposit_current(parts, old, grid, dt, -1.0, J, status)
    sr.deposit_rho(parts, grid, -1.0, rho)
    assert int(status.item()) == 0
    pd = p.astype(np.float64)
    vz = pd[:, 2] / np.sqrt(1 + (pd * pd).sum(1))
    ref = pic.deposit_current(p0.astype(np.float64), p1.astype(np.float64), vz, w, -1.0, dt, dim, n, tuple(dx))
    ones = _touching(p0, np.ones(count), dim, n, dx)
    dV = np.prod(dx[:dim])
    # a move across the periodic boundary takes off the box length in float: two roundings
    # of n cells, on the nodes it reaches
    wrapped = np.zeros(n[::-1])
    for a in range(dim):
        at = [slice(None)] * 3
        at[2 - a] = np.array([-3, -2, -1, 0, 1, 2]) % n[a]
        wrapped[tuple(at)] += n[a] * 2.0 ** -23
    for a in range(3):
        # a contribution is at most q w dx / (dt dV) times a move of 0.95 cell (2D Jz: q w v
        # / dV); rounded to 2^-21 of that and, with its fractions, factors and products,
        # within 16 units of 2^-24 of it; the sums of a node's few blocks add 2^-21
        top = 2.0 * (dx[a] / dt if a < dim else 1.0) / dV
        tol = (2.0 ** -19 + wrapped.ravel()) * top * ones
        assert np.all(np.abs(J[a].cpu().numpy() - ref[a].ravel()) <= tol + 1e-300), a
    ref = pic.deposit_rho(p1.astype(np.float64), w.astype(np.float64), -1.0, dim, n, tuple(dx)).ravel()
    tol = 16 * 2.0 ** -24 * _touching(p1, w, dim, n, dx) / dV
    assert np.all(np.abs(rho.cpu().numpy() - ref) <= tol + 1e-300)
