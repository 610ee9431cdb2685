"""Explicit chunks on both sides of the sizes at which the emission step changes its way
(rounds dealt to a block's waves, or one wave a chunk), in blocks that deal and blocks that
need not, and with bounds that decrease, against uniform chunks bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from test_gpu_chunks import _run

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = 64 * 61 + 17          # the last round is short


@pytest.fixture(scope="module")
def sr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1409_5574_amd import api
    api.lib()
    return api


@pytest.fixture(scope="module")
def table(sr):
    return sr.Table()


def _with_empty_chunks(cuts, chunks, seed):
    """The bounds `cuts` (in rounds) with empty chunks between them, `chunks` in all."""
    rng = np.random.default_rng(seed)
    start = np.array([64 * c for c in cuts] + [N])
    more = rng.choice(start, chunks + 1 - len(start))
    return np.sort(np.concatenate([start, more])).tolist()


def _check(sr, table, dim, K, sampler, pp, floor, start):
    cfg = synth.config("c3", grid=(24, 20, 16), slab=None) if dim == 3 else synth.config("c2", grid=(64, 64, 1))
    pu, _, phu, lu, su = _run(sr, table, cfg, N, K, sampler, K, None, 0, floor, np.float32)
    pr, buf, phr, lr, sr_ = _run(sr, table, cfg, N, K, sampler, pp, start, 0, floor, np.float32)
    for k in ("x", "y", "z", "px", "py", "pz"):
        if pu[k] is not None:
            np.testing.assert_array_equal(pu[k], pr[k], err_msg=k)
    assert phu["count"] == phr["count"] > 100
    count = buf.seg_count.cpu().numpy().view(np.uint32).astype(np.int64)
    cap = np.maximum(np.diff(start), 0) * pp
    assert np.all(count[np.diff(start) <= 0] == 0)
    keep = np.concatenate([np.arange(c) < m for c, m in zip(count, cap)])
    for k in ("eps", "w", "dir", "pos", "parent", "k"):
        np.testing.assert_array_equal(phu[k][keep], phr[k], err_msg=k)
    e = phu["eps"].astype(np.float64) * phu["w"].astype(np.float64)
    assert (sr_ & 1) == int(not keep.all())
    # sums of 64-bit terms in another order: a few thousand roundings of 2^-53
    np.testing.assert_allclose(lr[4], e[~keep].sum(), rtol=4e-13, atol=0)
    np.testing.assert_allclose(lr[[0, 1, 2, 3, 5, 7]], lu[[0, 1, 2, 3, 5, 7]], rtol=4e-13, atol=0)
    np.testing.assert_allclose(lr[6], lu[6], rtol=1e-6)     # a sum of 32-bit weights


CUTS = [0, 1, 1, 2, 21, 22, 24, 27, 31, 31, 60]


@pytest.mark.parametrize("dim, K, sampler, pp, floor, chunks", [
    (3, 1, 0, 1, 0.0, 8192), (3, 1, 0, 1, 0.0, 8193),
    (2, 8, 0, 8, 0.0, 8192), (3, 8, 0, 8, 0.0, 8193),
    (3, 4, 3, 4, 30.0, 8193), (2, 4, 3, 4, 0.0, 9000),
    (2, 2, 1, 2, 0.0, 8193), (3, 2, 1, 2, 30.0, 8193),
    (3, 8, 0, 1, 0.0, 8193),                           # segments that overflow
    (3, 16, 0, 16, 0.0, 2048), (3, 16, 0, 16, 0.0, 2049), (2, 16, 3, 16, 0.0, 2049),
])
def test_many_explicit_chunks(sr, table, dim, K, sampler, pp, floor, chunks):
    print(f"[gpu-case] {chunks} explicit chunks {dim}D K={K} sampler={sampler} pp={pp}", flush=True)
    _check(sr, table, dim, K, sampler, pp, floor, _with_empty_chunks(CUTS, chunks, K + chunks))


@pytest.mark.parametrize("dim, K, sampler, pp", [(3, 1, 0, 1), (3, 8, 3, 8), (2, 4, 1, 1), (2, 16, 0, 16)])
@pytest.mark.parametrize("cuts", [
    list(range(0, 61, 3)),                             # three rounds each: no block deals
    [0, 3, 6, 9, 12, 13, 13, 13, 14, 30, 31, 32, 33],  # a block that does not, two that do
    [0, 5, 6, 7, 8, 9, 14, 19, 24, 29],                # a longest chunk of just over its share
])
def test_blocks_that_deal_and_blocks_that_do_not(sr, table, dim, K, sampler, pp, cuts):
    print(f"[gpu-case] chunks at {cuts[:6]} {dim}D K={K} sampler={sampler} pp={pp}", flush=True)
    _check(sr, table, dim, K, sampler, pp, 0.0, [64 * c for c in cuts] + [N])


@pytest.mark.parametrize("chunks", [15, 8193])
@pytest.mark.parametrize("dim, K, sampler", [(3, 4, 0), (2, 1, 3)])
def test_bounds_that_decrease_hold_nothing(sr, table, dim, K, sampler, chunks):
    print(f"[gpu-case] decreasing bounds {chunks} {dim}D K={K}", flush=True)
    start = _with_empty_chunks(CUTS, chunks - 4, chunks) + [N - 64, N - 200, 640, 5]
    _check(sr, table, dim, K, sampler, K, 0.0, start)


@pytest.mark.parametrize("dim, K", [(3, 1), (3, 8), (2, 4)])
def test_waves_at_the_periodic_boundary(sr, table, dim, K):
    """Every particle in the last cell along x, whose right neighbours are the first cells,
    in dealt rounds: the same state and photons as in uniform chunks."""
    print(f"[gpu-case] last cell along x {dim}D K={K}", flush=True)
    cfg = synth.config("c3", grid=(24, 20, 16), slab=None) if dim == 3 else synth.config("c2", grid=(64, 64, 1))
    start = [64 * c for c in CUTS] + [N]
    out = []
    real = synth.gen_particles
    try:
        def shifted(c, n=None):
            st = real(c, n=n)
            edge = np.float32((cfg.grid[0] - 1) * cfg.dx)
            st["x"] = (edge + np.float32(0.9 * cfg.dx) * (st["x"] / st["x"].max())).astype(np.float32)
            return st
        synth.gen_particles = shifted
        for s in (None, start):
            out.append(_run(sr, table, cfg, N, K, 0, K, s, 0, 0.0, np.float32))
    finally:
        synth.gen_particles = real
    for k in ("x", "y", "z", "px", "py", "pz"):
        if out[0][0][k] is not None:
            np.testing.assert_array_equal(out[0][0][k], out[1][0][k], err_msg=k)
    for k in ("eps", "w", "dir", "pos", "parent", "k"):
        np.testing.assert_array_equal(out[0][2][k], out[1][2][k], err_msg=k)
