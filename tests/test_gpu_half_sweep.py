"""The half sweep (variant 5, one column of spins 1/2): from the smallest size, with one
tile per value of the few outer sites, over one and several windows, with every pair or
few of them (groups and outer sites with nothing to do), with and without s+- s^z pieces
and single flips, grids that are and are not a multiple of 8; elementwise against the
oracle, and the Lanczos sums through a short run's tridiagonal."""
import numpy as np
import pytest

import ftlm_workloads as W
from oracle import ftlm as of

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _system(n, couple):
    rng = np.random.default_rng(40 + n)
    J, pos, B = np.triu(rng.uniform(-1, 1, (n, n)), 1), None, rng.uniform(-1, 1, 3)
    far = np.abs(np.subtract.outer(np.arange(n), np.arange(n)))
    if couple == "dipolar":
        pos = W.unit_vectors(rng, n)
    elif couple == "chain":  # nothing but neighbours, no single flips
        J, B = J * (far == 1), np.array([0.0, 0.0, 1.0])
    elif couple == "far":  # no pair inside a layout, most outer sites with few pairs
        J = J * ((far == 7) | (far == 4))
    return W.System(two_s=np.ones(n, np.int32), J=J, d=None, e=np.tile([0.0, 0.0, 1.0], (n, 1)), g=np.full(n, 2.0),
                    B=B, pos=pos, name=couple)


def test_more_outer_pairs_than_lanes():
    """2^23 complex64 rows are one window: 66 pairs of outer sites."""
    import paper_2607_25585_amd as F
    ham = F.Hamiltonian(_system(23, "dipolar"))
    v = torch.randn(ham.dim, dtype=torch.complex64, device="cuda")
    print("case outer pairs n 23", flush=True)
    ham.set_tuning(F.FTLM_C64, 1, 5)
    got = ham.apply(v).clone()
    ham.set_tuning(F.FTLM_C64, 1, 1)
    want = ham.apply(v)
    assert float((got - want).abs().max()) < 4e-5 * float(want.abs().max())


@pytest.mark.parametrize("couple", ["dipolar", "chain", "far"])
@pytest.mark.parametrize("n,K", [(16, 8), (17, 4), (18, 2), (18, 8), (15, 16), (16, 16)])
def test_columns_match_oracle(n, K, couple):
    """2, 4, 8 and 16 columns as the lowest row bits, from the smallest size on."""
    import paper_2607_25585_amd as F
    sysm = _system(n, couple)
    ham, ref = F.Hamiltonian(sysm), of.Ham(sysm)
    rng = np.random.default_rng(n)
    v = rng.standard_normal((ham.dim, K)) + 1j * rng.standard_normal((ham.dim, K))
    want = np.stack([ref.apply(v[:, c]) for c in range(K)], axis=1)
    for cap in (0, 5, 64):
        print("case columns", couple, n, K, "grid", cap, flush=True)
        for prec, dt, tol in ((F.FTLM_C128, torch.complex128, 1e-12), (F.FTLM_C64, torch.complex64, 2e-5)):
            ham.set_tuning(prec, K, 5, cap)
            got = ham.apply(torch.as_tensor(v, device="cuda").to(dt)).cpu().numpy()
            assert np.max(np.abs(got - want)) < tol * np.max(np.abs(want))
    T = np.array([1.0, 10.0])
    ham.set_tuning(F.FTLM_C128, K, 0)
    a = F.run(ham, K, 4, T, seed=3, columns=K, return_tridiagonals=True)
    ham.set_tuning(F.FTLM_C128, K, 1)
    b = F.run(ham, K, 4, T, seed=3, columns=K, return_tridiagonals=True)
    scale = np.max(np.abs(b["alpha"])) + np.max(np.abs(b["beta"]))
    for k in ("alpha", "beta"):
        assert np.max(np.abs(a[k] - b[k])) < 1e-11 * scale
    assert np.max(np.abs(a["M"] - b["M"])) < 1e-9 * np.max(np.abs(b["M"]))


@pytest.mark.parametrize("tile_kb", [0, 128])
@pytest.mark.parametrize("couple", ["dipolar", "exchange", "chain", "far"])
@pytest.mark.parametrize("n", [12, 13, 16, 17])
def test_half_sweep_matches_oracle(n, couple, tile_kb, plan_windows):
    import paper_2607_25585_amd as F
    plan_windows(tile_kb=tile_kb)
    sysm = _system(n, couple)
    ham, ref = F.Hamiltonian(sysm), of.Ham(sysm)
    rng = np.random.default_rng(n)
    v = rng.standard_normal(ham.dim) + 1j * rng.standard_normal(ham.dim)
    want = ref.apply(v)
    for cap in (0, 3, 8):
        print("case", couple, n, "window", tile_kb, "grid", cap, flush=True)
        for prec, dt, tol in ((F.FTLM_C128, torch.complex128, 1e-12), (F.FTLM_C64, torch.complex64, 2e-5)):
            ham.set_tuning(prec, 1, 5, cap)
            got = ham.apply(torch.as_tensor(v, device="cuda").to(dt)).cpu().numpy()
            assert np.max(np.abs(got - want)) < tol * np.max(np.abs(want))
    T = np.array([1.0, 10.0])
    ham.set_tuning(F.FTLM_C128, 1, 5)
    a = F.run(ham, 1, 5, T, seed=3, columns=1, return_tridiagonals=True)
    ham.set_tuning(F.FTLM_C128, 1, 1)
    b = F.run(ham, 1, 5, T, seed=3, columns=1, return_tridiagonals=True)
    scale = np.max(np.abs(b["alpha"])) + np.max(np.abs(b["beta"]))
    for k in ("alpha", "beta"):
        assert np.max(np.abs(a[k] - b[k])) < 1e-11 * scale
    assert np.max(np.abs(a["M"] - b["M"])) < 1e-9 * np.max(np.abs(b["M"]))
