"""The deposits on both sides of the sizes at which they change their way, against the
64-bit oracle: the charge added directly, in a box and in slabs; the current in up to two
slabs and up to eight, and the accuracy of light particles beside a heavy one there."""
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
    (3, (32, 32, 32), 32767, "wide", "sorted"),          # one electron short of the box
    (3, (32, 32, 32), 32769, "wide", "sorted"),
    (3, (32, 32, 32), 32769, "equal", "unsorted"),       # no box: every block direct
    (3, (48, 48, 48), 40000, "wide", "sorted"),
    (3, (128, 128, 96), 40000, "wide", "sorted"),        # sparse: direct
    (3, (256, 128, 64), 262144, "equal", "sorted"),      # sparse, and large enough to look
    (2, (384, 384, 1), 65535, "zeros", "sorted"),
    (2, (384, 384, 1), 65537, "zeros", "sorted"),
    (2, (384, 384, 1), 65537, "wide", "unsorted"),
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


@pytest.mark.parametrize("dim, n, count, drift, heavy", [
    (3, (256, 64, 4), 24575, 60.0, 1.0),        # two slabs at most: windows
    (3, (256, 64, 4), 40959, 20.0, 1.0),        # up to four
    (3, (256, 64, 4), 40960, 60.0, 1.0),        # up to eight
    (2, (2000, 64, 1), 65535, 300.0, 1.0),
    (2, (2000, 64, 1), 196607, 90.0, 1.0),
    (2, (2000, 64, 1), 196608, 300.0, 1.0),
    (3, (256, 64, 4), 200000, 60.0, 1e6),       # one heavy particle a block, and light ones
    (2, (2000, 64, 1), 200000, 300.0, 1e6),
])
def test_current_of_drifted_slabs(sr, dim, n, count, drift, heavy):
    """Blocks drifted along x: boxes of some 20 000 nodes, taken in five to eight slabs."""
    print(f"[gpu-case] current slabs {dim}D {n} {count} {drift} {heavy}", flush=True)
    dx, dt = np.array([0.3, 0.25, 0.35]), 0.11
    rng = np.random.default_rng(count + n[0])
    box = np.array(n[:dim]) * dx[:dim]

    def wrap(x):
        x = np.mod(x, box).astype(np.float32)
        return np.where(x >= box.astype(np.float32), 0.0, x).astype(np.float32)

    home = rng.uniform(0, 1, (count, dim)) * box
    cell = np.floor(home / dx[:dim]).astype(np.int64)
    home = home[np.lexsort([cell[:, a] // 4 for a in range(dim)])]
    home[:, 0] += rng.normal(0, 1, count) * drift * dx[0]
    p0 = wrap(home)
    step = np.where(rng.uniform(size=(count, 1)) < 0.2, 0.95, 0.05) * rng.uniform(-1, 1, (count, dim))
    p1 = wrap(p0.astype(np.float64) + step * dx[:dim])
    w = rng.uniform(0.5, 2.0, count).astype(np.float32)
    w[256::512] *= np.float32(heavy)
    p = rng.normal(0, 1, (count, 3)).astype(np.float32)
    st = {"x": p1[:, 0].copy(), "y": p1[:, 1].copy(), "z": p1[:, 2].copy() if dim == 3 else None,
          "px": p[:, 0].copy(), "py": p[:, 1].copy(), "pz": p[:, 2].copy(), "w": w,
          "id": np.arange(count, dtype=np.uint32)}
    old = [torch.from_numpy(p0[:, a].copy()).cuda() for a in range(dim)] + [None] * (3 - dim)
    J = [torch.zeros(int(np.prod(n)), device="cuda") for _ in range(3)]
    status = torch.zeros(1, device="cuda", dtype=torch.int32)
    sr.deposit_current(sr.Particles.from_numpy(st, dim=dim), old, sr.grid_struct(dim, n=n, dx=tuple(dx)),
                       dt, -1.0, J, status)
    assert int(status.item()) == 0
    pd = p.astype(np.float64)
    vz = pd[:, 2] / np.sqrt(1 + (pd * pd).sum(1))
    ref = pic.deposit_current(p0.astype(np.float64), p1.astype(np.float64), vz, w, -1.0, dt, dim, n, tuple(dx))
    weight, adds = _touching(p0, w, dim, n, dx), _touching(p0, np.ones(count), dim, n, dx)
    wrapped = np.zeros(n[::-1])       # box length taken off in float: two roundings of n cells
    for a in range(dim):
        at = [slice(None)] * 3
        at[2 - a] = np.array([-3, -2, -1, 0, 1, 2]) % n[a]
        wrapped[tuple(at)] += n[a] * 2.0 ** -23
    for a in range(3):
        # a contribution is at most q w dx / (dt dV) times a move of 0.95 cell (2D Jz: q w v
        # / dV) and, with its fractions, factors and products, within 32 units of 2^-24 of
        # it; a particle whose bound is above 2^-12 of its slab's sum is rounded to 2^-31 of
        # that sum, 2^-19 of its own bound; each add rounds the running sum.  Nothing
        # depends on the weights of particles that do not touch the node.
        top = 2.0 * (dx[a] / dt if a < dim else 1.0) / np.prod(dx[:dim])
        tol = (2.0 ** -18 + adds * 2.0 ** -24 + wrapped.ravel()) * top * weight
        assert np.all(np.abs(J[a].cpu().numpy() - ref[a].ravel()) <= tol + 1e-300), a
