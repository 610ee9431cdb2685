"""The multi-step launch's photon records and its two kernels: every field of every record
against single-step launches, segments that fill up in mid-launch, launches with more chunks
than four waves each are given, and a weight that is not finite."""
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


FIELDS = ("eps", "w", "dx", "dy", "dz", "x", "y", "z", "parent", "k", "step")


def _records(ph, n, pp):
    """The stored records chunk by chunk, as a list of dicts of arrays."""
    cols = dict(zip(FIELDS, (ph.eps, ph.w, *ph.dir, *ph.pos, ph.parent, ph.k, ph.step)))
    cols = {k: t.cpu().numpy() for k, t in cols.items()}
    out = []
    for c, count in enumerate(ph.seg_count.cpu().numpy()):
        m = min(int(count), (min(64 * c + 64, n) - 64 * c) * pp)
        out.append({k: v[64 * c * pp:64 * c * pp + m] for k, v in cols.items()})
    return out


def _launches(sr, table, st, splits, prm, pp):
    cfg = synth.config("c1")
    n, at = st["w"].size, 3
    parts = sr.Particles.from_numpy(st, dim=0)
    grid = sr.grid_struct(0, e0=(0.1, 0.0, 0.2), b0=(0.3, 0.0, 40.0))
    rows, recs = [], []
    for steps in splits:
        ph = sr.PhotonBuffer(n, pp, dim=3, with_step=True)
        ledger = sr.LedgerBuf(steps, sr.n_chunks_uniform(n), steps_per_call=steps)
        sr.gather_push_emit_steps(parts, grid, cfg.dt, 0xBA7C4, at, steps, prm, table, ph, ledger)
        rows.append(ledger.rows.cpu().numpy())
        recs.append(_records(ph, n, pp))
        at += steps
    chunks = [{k: np.concatenate([r[c][k] for r in recs]) for k in FIELDS} for c in range(len(recs[0]))]
    return torch.stack(parts.x + parts.p).cpu().numpy(), np.concatenate(rows), chunks


@pytest.mark.parametrize("n, steps, K, sampler, recoil", [
    (130, 21, 1, 0, 1), (100, 9, 5, 0, 2), (190, 7, 2, 3, 1), (70, 5, 16, 1, 1),
])
def test_records_equal_single_step_launches(sr, table, n, steps, K, sampler, recoil):
    print(f"[gpu-case] step records n {n} steps {steps} K {K} sampler {sampler}", flush=True)
    cfg = synth.config("c1")
    st = synth.gen_particles(cfg, n=n, seed=n + steps)
    prm = sr.params_struct(cfg.hbar_n, cfg.alpha, K, sampler=sampler, recoil=recoil, kin_cut=sampler != 0)
    s1, r1, c1 = _launches(sr, table, st, [steps], prm, 64)
    s2, r2, c2 = _launches(sr, table, st, [1] * steps, prm, 64)
    assert np.array_equal(s1, s2) and np.array_equal(r1, r2)
    assert sum(len(c["eps"]) for c in c1) > 5
    for a, b in zip(c1, c2):
        for k in FIELDS:
            np.testing.assert_array_equal(a[k], b[k], err_msg=k)


@pytest.mark.parametrize("K, sampler", [(2, 0), (8, 3)])
def test_segments_that_fill_up_in_mid_launch(sr, table, K, sampler):
    cfg = synth.config("c1")
    n, steps = 150, 40
    st = synth.gen_particles(cfg, n=n, seed=8)
    prm = sr.params_struct(cfg.hbar_n, cfg.alpha, K, sampler=sampler, kin_cut=sampler != 0)
    print(f"[gpu-case] segments fill up K {K} sampler {sampler}", flush=True)
    s1, r1, c1 = _launches(sr, table, st, [steps], prm, 320)
    s2, r2, c2 = _launches(sr, table, st, [steps], prm, 1)
    assert np.array_equal(s1, s2)
    cut = 0.0
    for c, (a, b) in enumerate(zip(c1, c2)):
        held = len(b["eps"])
        assert held == min(len(a["eps"]), min(64, n - 64 * c))
        for k in FIELDS:
            np.testing.assert_array_equal(a[k][:held], b[k], err_msg=k)
        cut += (a["w"][held:].astype(np.float64) * a["eps"][held:].astype(np.float64)).sum()
    assert cut > 0.0 and len(c2[0]["eps"]) == 64
    # sums of the same 64-bit products in another order
    np.testing.assert_allclose(r2[:, 4].sum(), cut, rtol=1e-12)
    same = [0, 1, 2, 3, 5, 6, 7]
    assert np.array_equal(r1[:, same], r2[:, same])


@pytest.mark.parametrize("chunks, K, sampler", [
    (4097, 1, 0), (4097, 8, 0), (2049, 16, 0), (2049, 2, 1), (1537, 4, 3), (1025, 8, 3),
])
def test_one_wave_a_chunk_equals_four(sr, table, chunks, K, sampler):
    """A launch of too many chunks for four waves each, against the same particles in two
    launches of half of them: the words of a particle come from its id and step alone."""
    print(f"[gpu-case] steps in {chunks} chunks K {K} sampler {sampler}", flush=True)
    cfg = synth.config("c1")
    n, steps, pp = 64 * (chunks - 1) + 19, 5, 16
    st = synth.gen_particles(cfg, n=n, seed=chunks)
    prm = sr.params_struct(cfg.hbar_n, cfg.alpha, K, sampler=sampler, kin_cut=sampler != 0)
    s, r, c = _launches(sr, table, st, [steps], prm, pp)
    cut = 64 * (chunks // 2)
    parts = [_launches(sr, table, {k: v[sl] for k, v in st.items()}, [steps], prm, pp)
             for sl in (slice(0, cut), slice(cut, n))]
    assert np.array_equal(s, np.concatenate([p[0] for p in parts], axis=1))
    halves = parts[0][2] + parts[1][2]
    assert len(halves) == len(c) == chunks and sum(len(a["eps"]) for a in c) > 50
    for k in FIELDS:
        np.testing.assert_array_equal(np.concatenate([a[k] for a in c]),
                                      np.concatenate([b[k] for b in halves]), err_msg=k)
    # 64-bit sums (the weights' of 32-bit ones, exact here) in another order
    np.testing.assert_allclose(r[:, :7], parts[0][1][:, :7] + parts[1][1][:, :7], rtol=1e-11)
    assert np.array_equal(r[:, 7], np.maximum(parts[0][1][:, 7], parts[1][1][:, 7]))


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_nonfinite_weight_shows_in_every_row(sr, table, bad):
    """A weight that is not finite makes the energy sums of every step that, as one step a
    call does, whether or not the particle emits."""
    cfg = synth.config("c1")
    n, steps = 70, 6
    st = synth.gen_particles(cfg, n=n, seed=2)
    st["w"][5] = bad
    prm = sr.params_struct(cfg.hbar_n, cfg.alpha, 1)
    print(f"[gpu-case] steps weight {bad}", flush=True)
    _, rows, _ = _launches(sr, table, st, [steps], prm, 64)
    parts, grid = sr.Particles.from_numpy(st, dim=0), sr.grid_struct(0, e0=(0.1, 0.0, 0.2), b0=(0.3, 0.0, 40.0))
    ph, ledger = sr.PhotonBuffer(n, 64, dim=3), sr.LedgerBuf(1, sr.n_chunks_uniform(n))
    for s in range(steps):
        sr.gather_push_emit(parts, None, grid, cfg.dt, 0xBA7C4, 3 + s, prm, table, ph, ledger, 0)
        one = ledger.row(0)
        assert np.array_equal(np.isnan(one[:2]), np.isnan(rows[s, :2])), (s, one, rows[s])
