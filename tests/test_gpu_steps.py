"""The multi-step launch at the edges of its batches and chunks: one launch of n
steps leaves, bit for bit, what n launches of one step leave, for step counts
around a batch, partial chunks, every sampler, segments that overflow, and a
momentum that is not finite."""
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


def _run(sr, table, st, splits, prm, pp):
    """Launches of the given numbers of steps; final state, ledger rows, photon counts."""
    cfg = synth.config("c1")
    n = st["w"].size
    parts = sr.Particles.from_numpy(st, dim=0)
    grid = sr.grid_struct(0, e0=(0.1, 0.0, 0.2), b0=(0.3, 0.0, 40.0))
    rows, counts, status, at = [], np.zeros(sr.n_chunks_uniform(n), np.int64), 0, 3
    for steps in splits:
        photons = sr.PhotonBuffer(n, pp, dim=3, with_step=True)
        ledger = sr.LedgerBuf(steps, sr.n_chunks_uniform(n), steps_per_call=steps)
        sr.gather_push_emit_steps(parts, grid, cfg.dt, 0xBA7C4, at, steps, prm, table, photons, ledger)
        rows.append(ledger.rows.cpu().numpy())
        counts += photons.seg_count.cpu().numpy()
        status |= ledger.read_status()
        at += steps
    state = torch.stack(parts.x + parts.p).cpu().numpy()
    return state, np.concatenate(rows), counts, status


@pytest.mark.parametrize("n, steps, K, sampler, recoil, pp", [
    (64, 1, 1, 0, 1, 64), (65, 7, 1, 0, 1, 64), (1, 8, 1, 3, 1, 64), (130, 9, 1, 1, 2, 64),
    (127, 17, 2, 0, 1, 64), (200, 5, 3, 3, 2, 64), (63, 6, 4, 1, 1, 64), (70, 11, 5, 0, 0, 64),
    (129, 4, 8, 0, 1, 64), (66, 3, 16, 3, 1, 64), (64, 3, 15, 1, 1, 64),
    (190, 19, 2, 0, 1, 0),      # every photon dropped
])
def test_one_launch_equals_single_step_launches(sr, table, n, steps, K, sampler, recoil, pp):
    print(f"[gpu-case] steps n {n} steps {steps} K {K} sampler {sampler} pp {pp}", flush=True)
    cfg = synth.config("c1")
    st = synth.gen_particles(cfg, n=n, seed=n + steps)
    prm = sr.params_struct(cfg.hbar_n, cfg.alpha, K, sampler=sampler, recoil=recoil,
                           kin_cut=sampler != 0 or K == 5)
    s1, r1, c1, f1 = _run(sr, table, st, [steps], prm, pp)
    s2, r2, c2, f2 = _run(sr, table, st, [1] * steps, prm, pp)
    # with slots to spare nothing depends on where a launch begins; an overflowing
    # segment drops by its fill, so its energies are compared as a whole
    assert np.array_equal(s1, s2) and np.array_equal(c1, c2) and f1 == f2
    assert np.array_equal(r1, r2)
    assert np.all(r1[:, 6] == n) and (c1.sum() > 0 or n * steps * K < 500)


def test_nonfinite_momentum_in_a_batch(sr, table):
    cfg = synth.config("c1")
    st = synth.gen_particles(cfg, n=100, seed=4)
    ok = _run(sr, table, st, [10], sr.params_struct(cfg.hbar_n, cfg.alpha, 2), 64)
    st["px"][70] = np.inf
    print("[gpu-case] steps nonfinite", flush=True)
    got = _run(sr, table, st, [10], sr.params_struct(cfg.hbar_n, cfg.alpha, 2), 64)
    keep = np.arange(100) != 70
    assert np.array_equal(got[0][:, keep], ok[0][:, keep])
    assert got[3] == (ok[3] | 4) and np.all(np.isfinite(got[1])) and got[2][0] == ok[2][0]
