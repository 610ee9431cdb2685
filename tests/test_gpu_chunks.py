"""Explicit chunks against uniform ones: a chunk of m 64-particle rounds holds the photons
of m uniform chunks in their order, whichever waves of its block took the rounds."""
from __future__ import annotations

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


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


def _run(sr, table, cfg, n, K, sampler, pp, start, dn_policy, floor, dtype):
    st = synth.gen_particles(cfg, n=n)
    scale = 3000.0 if cfg.dim == 3 else 2000.0
    for k in ("px", "py", "pz"):
        st[k] = (st[k] * scale).astype(np.float32)
    st = {k: (v if k == "id" else v.astype(dtype)) for k, v in st.items()}
    E, B = synth.standing_wave_grid(cfg, 0.4)
    parts = sr.Particles.from_numpy(st, dim=cfg.dim,
                                    dtype=torch.float64 if dtype == np.float64 else torch.float32)
    nc = sr.n_chunks_uniform(n) if start is None else len(start) - 1
    dev = None if start is None else torch.tensor(start, dtype=torch.int64, device="cuda")
    photons = sr.PhotonBuffer(n, pp, n_chunks=None if start is None else nc, dim=cfg.dim)
    ledger = sr.LedgerBuf(1, nc)
    prm = sr.params_struct(cfg.hbar_n, cfg.alpha, K, sampler, cfg.recoil, dn_policy, sampler == 0,
                           omega_grid=floor)
    sr.gather_push_emit(parts, sr.Fields(E, B), sr.grid_struct(cfg.dim, n=cfg.grid, dx=(cfg.dx,) * 3), cfg.dt,
                        5, 3, prm, table, photons, ledger, 0, start=dev)
    torch.cuda.synchronize()
    return parts.to_numpy(), photons, photons.gather(n, dev), ledger.row(0), ledger.read_status()


@pytest.mark.parametrize("dim, K, sampler, pp, dn_policy, floor, dtype", [
    (3, 4, 3, 4, 0, 0.0, np.float32),
    (3, 8, 0, 8, 1, 0.0, np.float32),
    (3, 16, 0, 16, 0, 30.0, np.float32),
    (2, 1, 0, 1, 0, 0.0, np.float32),
    (2, 2, 1, 2, 0, 0.0, np.float32),
    (2, 2, 1, 2, 0, 30.0, np.float32),
    (3, 3, 0, 1, 0, 0.0, np.float32),       # segments that overflow
    (3, 2, 0, 2, 0, 0.0, np.float64),
])
def test_explicit_chunks_hold_the_uniform_chunks_photons(sr, table, dim, K, sampler, pp, dn_policy, floor, dtype):
    cfg = synth.config("c3", grid=(24, 20, 16), slab=None) if dim == 3 else synth.config("c2", grid=(64, 64, 1))
    n = 64 * 61 + 17                        # the last round is short
    # one round, none, many (a chunk of several turns of the waves), a last short one
    cuts = [0, 1, 1, 2, 21, 22, 24, 27, 31, 31, 60]
    start = [64 * c for c in cuts] + [n]
    print(f"[gpu-case] explicit chunks {dim}D K={K} sampler={sampler} pp={pp}", flush=True)
    pu, _, phu, lu, su = _run(sr, table, cfg, n, K, sampler, K, None, dn_policy, floor, dtype)
    pr, buf, phr, lr, sr_ = _run(sr, table, cfg, n, K, sampler, pp, start, dn_policy, floor, dtype)
    for k in ("x", "y", "z", "px", "py", "pz"):
        if pu[k] is not None:
            np.testing.assert_array_equal(pu[k], pr[k], err_msg=k)
    assert phu["count"] == phr["count"] > 100
    # what fits of each chunk's photons, in the uniform order
    count = buf.seg_count.cpu().numpy().view(np.uint32).astype(np.int64)
    cap = np.diff(start) * pp
    keep = np.concatenate([np.arange(c) < m for c, m in zip(count, cap)])
    for k in ("eps", "w", "dir", "pos", "parent", "k"):
        np.testing.assert_array_equal(phu[k][keep], phr[k], err_msg=k)
    e = phu["eps"].astype(np.float64) * phu["w"].astype(np.float64)
    assert (sr_ & 1) == int(not keep.all())
    # sums of 64-bit terms in another order: a few thousand roundings of 2^-53
    np.testing.assert_allclose(lr[4], e[~keep].sum(), rtol=4e-13, atol=0)
    np.testing.assert_allclose(lr[[0, 1, 2, 3, 5, 7]], lu[[0, 1, 2, 3, 5, 7]], rtol=4e-13, atol=0)
    np.testing.assert_allclose(lr[6], lu[6], rtol=1e-6)     # a sum of 32-bit weights
