"""A tuned handle is not slower than one with the built-in launch, for the column counts that
the half sweep takes, one that it does not, the tile sweep and the direct gather; and its
products stay those of the built-in launch."""
import numpy as np
import pytest

import ftlm_workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _dipolar(n):
    rng = np.random.default_rng(n)
    return W.System(two_s=np.ones(n, np.int32), J=W.ring_couplings(n, 1.0), d=None, e=np.tile([0.0, 0.0, 1.0], (n, 1)),
                    g=np.full(n, 2.0), B=0.5 * W.unit_vectors(rng, 1)[0], pos=W.unit_vectors(rng, n))


def _planar(two_s):
    n = len(two_s)
    rng = np.random.default_rng(n)
    ang = 2 * np.pi * np.arange(n) / n
    return W.System(two_s=np.array(two_s, np.int32), J=W.ring_couplings(n, 0.5), d=np.full(n, -1.0),
                    e=W.unit_vectors(rng, n), g=np.full(n, 2.0), B=np.array([0.0, 0.0, 2.0]),
                    pos=0.8 * np.stack([np.cos(ang), np.sin(ang), np.zeros(n)], 1))


def _ms(ham, v, w, reps=20):
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(reps):
            ham.apply(v, out=w)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / reps)
    return best


@pytest.mark.parametrize("system,K", [("half19", 1), ("half19", 2), ("half19", 4), ("half18", 8), ("half17", 16),
                                      ("half17", 3), ("s2", 1), ("s1", 20)])
def test_tuned_is_not_slower(system, K, tmp_path, monkeypatch):
    import paper_2607_25585_amd as F
    from paper_2607_25585_amd import autotune
    monkeypatch.setenv("FTLM_TUNE_CACHE", str(tmp_path / "tune.json"))
    sysm = {"half": lambda n: _dipolar(n), "s2": lambda n: _planar([4] * 9), "s1": lambda n: _planar([2] * 9)}[
        system[:4] if system.startswith("half") else system](int(system[4:] or 0))
    ham = F.Hamiltonian(sysm)
    for prec, dt in ((F.FTLM_C128, torch.complex128), (F.FTLM_C64, torch.complex64)):
        v = torch.randn((ham.dim, K) if K > 1 else (ham.dim,), dtype=dt, device="cuda")
        w = torch.empty_like(v)
        before, want = _ms(ham, v, w), ham.apply(v)
        choice = autotune.tune(ham, prec, K)
        after, got = _ms(ham, v, w), ham.apply(v)
        print("case tuned", system, K, dt, choice, before, after, flush=True)
        assert float((got - want).abs().max()) < (1e-12 if prec == F.FTLM_C128 else 4e-5) * float(want.abs().max())
        assert after < 1.25 * before
