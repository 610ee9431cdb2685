"""The angular map's blocks and its reduction, and the validity sums, against the host:
photon counts around the lanes that share a chunk, segments that are full, more chunks
than the blocks take at once, explicit chunks, and more blocks than one turn of the sums."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1409_5574_amd import api
    api.lib()
    return api


@pytest.mark.parametrize("n, pp, most, nt, nph, explicit", [
    (1, 4, 4, 3, 5, False),
    (64 * 37 + 5, 4, 40, 32, 64, False),
    (64 * 9000, 1, 33, 5, 7, False),          # over 256 blocks of 16 chunks: a second turn
    (64 * 300, 2, 300, 1, 1, False),          # counts past the segments' ends
    (64 * 500 + 11, 2, 70, 64, 64, True),
])
def test_angular_map_matches_host(sr, n, pp, most, nt, nph, explicit):
    print(f"[gpu-case] angular n={n} pp={pp} most={most} {nt}x{nph}", flush=True)
    rng = np.random.default_rng(n + most)
    start = np.arange(0, n + 64, 64)
    start[-1] = n
    if explicit:
        start = np.concatenate([[0, 0], np.sort(rng.integers(0, n, 331)), [n]])
    nc = len(start) - 1
    cap = np.diff(start) * pp
    count = rng.integers(0, most + 1, nc)
    held = np.minimum(count, cap)
    ph = sr.PhotonBuffer(n, pp, n_chunks=nc if explicit else None, dim=3)
    ph.seg_count.copy_(torch.from_numpy(count.astype(np.int32)))
    for t in (ph.eps, ph.w, *ph.dir):
        t.fill_(float("nan"))                 # slots past a chunk's photons are not read
    slot = np.concatenate([b * pp + np.arange(h) for b, h in zip(start, held)])
    # directions at the middle of a bin, or backwards
    it, ip = rng.integers(0, nt, len(slot)), rng.integers(0, nph, len(slot))
    back = rng.uniform(size=len(slot)) < 0.1
    th, phi = (it + 0.5) * (np.pi / 2 / nt), (ip + 0.5) * (2 * np.pi / nph)
    d = np.stack([np.where(back, -0.5, np.cos(th)), np.sin(th) * np.cos(phi), np.sin(th) * np.sin(phi)])
    eps, w = 10.0 ** rng.uniform(-6, 2, len(slot)), rng.uniform(0.1, 2, len(slot))
    at = torch.from_numpy(slot).cuda()
    for t, v in ((ph.eps, eps), (ph.w, w), *zip(ph.dir, d)):
        t[at] = torch.from_numpy(v.astype(np.float32)).cuda()
    hist = torch.ones(nt * nph + 1, device="cuda", dtype=torch.float64)
    dev = torch.from_numpy(start.astype(np.int64)).cuda() if explicit else None
    sr.angular_histogram(ph, n, (1.0, 0.0, 0.0), (0.0, 1.0, 0.0), nt, nph, hist, sr.angular_work(nt, nph), start=dev)
    e = (eps.astype(np.float32) * w.astype(np.float32)).astype(np.float64)
    ref = 1.0 + np.bincount(np.where(back, nt * nph, it * nph + ip), weights=e, minlength=nt * nph + 1)
    # the same 64-bit terms in another order: under 2^-53 a term, of at most len(slot) terms
    np.testing.assert_allclose(hist.cpu().numpy(), ref, rtol=max(len(slot), 8) * 2.0 ** -53, atol=0)


@pytest.mark.parametrize("n", [1, 257, 256 * 2048 + 1, 256 * 4096 + 300])
def test_validity_sums_add_up_their_flags(sr, n):
    print(f"[gpu-case] validity sums n={n}", flush=True)
    rng = np.random.default_rng(n)
    g = 10.0 ** rng.uniform(0, 5, n)
    w = rng.uniform(0.5, 2.0, n).astype(np.float32)
    st = {"x": np.zeros(n), "y": np.zeros(n), "z": np.zeros(n), "px": g * 10.0 ** rng.uniform(-4, 0, n),
          "py": np.zeros(n), "pz": g, "w": w, "id": np.arange(n, dtype=np.uint32)}
    st = {k: v if k == "id" else v.astype(np.float32) for k, v in st.items()}
    parts = sr.Particles.from_numpy(st, dim=3)
    grid = sr.grid_struct(0, b0=(0.0, 0.0, 800.0))
    flags, sums = sr.validity(parts, None, grid, 0.01, 5e-6, 1 / 137.0, 0.02)
    f = flags.cpu().numpy()[:n]
    got = np.asarray(sums)
    wd = w.astype(np.float64)
    if n > 1:
        assert (f & 1).any() and (f & 2).any() and not (f & 1).all() and not (f & 2).all()
    tol = 64 * 2.0 ** -53            # sums of a few dozen levels and turns
    np.testing.assert_allclose(got[:3], [wd.sum(), wd[(f & 1) != 0].sum(), wd[(f & 2) != 0].sum()],
                               rtol=max(tol, n / 1024 * 2.0 ** -53), atol=0)
