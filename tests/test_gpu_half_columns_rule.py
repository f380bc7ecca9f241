"""The built-in launch of 2, 4, 8 and 16 columns of spins 1/2 with single flips and few pairs
per site: the direct gather below the number of pairs where the half sweep pays, the half
sweep from there (the products are bitwise those of the explicit launch), and without
single flips the half sweep for any number; elementwise against the oracle."""
import numpy as np
import pytest

import ftlm_workloads as W
from oracle import ftlm as of

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _system(n, reach, flips):
    rng = np.random.default_rng(n)
    far = np.abs(np.subtract.outer(np.arange(n), np.arange(n)))
    J = np.triu(rng.uniform(-1, 1, (n, n)) * (np.minimum(far, n - far) <= reach), 1)
    return W.System(two_s=np.ones(n, np.int32), J=J if reach else None, d=None, e=np.tile([0.0, 0.0, 1.0], (n, 1)),
                    g=np.full(n, 2.0), B=np.array([0.3, 0.2, 1.0] if flips else [0.0, 0.0, 1.0]), pos=None)


# (sites, columns, complex64, pairs per site, single flips, the launch's variant)
@pytest.mark.parametrize("n,K,c64,reach,flips,variant", [
    (18, 2, False, 4, True, 1), (18, 2, False, 5, True, 5), (18, 2, False, 1, False, 5), (19, 2, False, 3, True, 1),
    (19, 2, False, 4, True, 5), (19, 2, True, 1, True, 1), (19, 2, True, 2, True, 5), (17, 4, False, 1, True, 1),
    (17, 4, False, 2, True, 5), (18, 4, True, 3, True, 1), (18, 4, True, 4, True, 5), (16, 8, False, 0, True, 1),
    (16, 8, False, 1, True, 5), (16, 8, True, 3, True, 1), (16, 8, True, 4, True, 5), (17, 8, True, 1, True, 5),
    (15, 16, True, 0, True, 1), (15, 16, True, 1, True, 5), (15, 16, False, 0, True, 1)])
def test_columns_launch_by_pairs(n, K, c64, reach, flips, variant):
    import paper_2607_25585_amd as F
    sysm = _system(n, reach, flips)
    ham, ref = F.Hamiltonian(sysm), of.Ham(sysm)
    prec, dt, tol = (F.FTLM_C64, torch.complex64, 2e-5) if c64 else (F.FTLM_C128, torch.complex128, 1e-12)
    rng = np.random.default_rng(1)
    v = rng.standard_normal((ham.dim, K)) + 1j * rng.standard_normal((ham.dim, K))
    x = torch.as_tensor(v, device="cuda").to(dt)
    print("case columns rule", n, K, dt, reach, flips, flush=True)
    got = {}
    for var in (0, 1, 5):
        ham.set_tuning(prec, K, var)
        got[var] = ham.apply(x).cpu().numpy()
    want = np.stack([ref.apply(v[:, c].copy()) for c in range(K)], axis=1)
    for var in got:
        assert np.max(np.abs(got[var] - want)) < tol * np.max(np.abs(want))
    assert np.array_equal(got[0], got[variant])
    if reach:
        assert not np.array_equal(got[0], got[6 - variant])
