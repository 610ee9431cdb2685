"""The angular map of sparse and mixed segments against the host: chunks of no or a few
photons that a lane takes each, beside waves whose chunks are walked by groups of lanes, more
chunks than the waves take at once, and explicit chunks of very uneven length."""
from __future__ import annotations

import numpy as np
import pytest

import test_gpu_diagnostics as diagnostics

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
    (64 * 8300 + 9, 1, 1, 4, 4, False),       # nine chunks a wave
    (64 * 66000 + 1, 1, 2, 32, 64, False),    # sixty-four a wave, and a second turn
    (64 * 8192, 1, 3, 60, 68, False),         # on both sides of the rule
    (64 * 8193, 1, 3, 60, 68, False),
    (64 * 9000, 1, 3, 64, 63, True),          # a few long chunks
    (64 * 20000, 2, 60, 1, 1, False),
    (15, 1, 40, 2, 3, True),
])
def test_sparse_angular_map_matches_host(sr, n, pp, most, nt, nph, explicit):
    diagnostics.test_angular_map_matches_host(sr, n, pp, most, nt, nph, explicit)


@pytest.mark.parametrize("explicit", [False, True])
def test_full_chunks_among_sparse_ones(sr, explicit):
    """Waves in which a chunk or two hold nearly all the photons, and ones with none."""
    rng = np.random.default_rng(3)
    chunks, pp = 40000, 4
    n = 64 * chunks
    start = np.arange(0, n + 64, 64)
    if explicit:
        start = np.concatenate([[0], np.sort(rng.integers(0, n, chunks - 1)), [n]])
    count = np.where(np.arange(chunks) % 37 == 5, 300, rng.integers(0, 2, chunks))
    count[1000:1100] = 0
    held = np.minimum(count, np.diff(start) * pp)
    print(f"[gpu-case] angular full chunks among sparse ones, explicit={explicit}", flush=True)
    ph = sr.PhotonBuffer(n, pp, n_chunks=chunks if explicit else None, dim=3)
    ph.seg_count.copy_(torch.from_numpy(count.astype(np.int32)))
    for t in (ph.eps, ph.w, *ph.dir):
        t.fill_(float("nan"))
    slot = np.concatenate([pp * b + np.arange(m) for b, m in zip(start, held)])
    at = torch.from_numpy(slot).cuda()
    eps = rng.uniform(0.1, 2.0, len(slot)).astype(np.float32)
    phi = (rng.integers(0, 8, len(slot)) + 0.5) * (2 * np.pi / 8)
    d = [np.full(len(slot), 0.6), 0.8 * np.cos(phi), 0.8 * np.sin(phi)]
    for t, v in ((ph.eps, eps), (ph.w, np.ones(len(slot))), *zip(ph.dir, d)):
        t[at] = torch.from_numpy(np.asarray(v, np.float32)).cuda()
    hist = torch.zeros(9, device="cuda", dtype=torch.float64)
    dev = torch.from_numpy(start.astype(np.int64)).cuda() if explicit else None
    sr.angular_histogram(ph, n, (1.0, 0.0, 0.0), (0.0, 1.0, 0.0), 1, 8, hist, sr.angular_work(1, 8), start=dev)
    ref = np.bincount((phi / (2 * np.pi / 8)).astype(int), weights=eps.astype(np.float64), minlength=9)
    # the same 64-bit terms in another order
    np.testing.assert_allclose(hist.cpu().numpy(), ref, rtol=len(slot) * 2.0 ** -53, atol=0)
