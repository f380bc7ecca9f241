"""L2-window passes (variant 4) of several columns of a general-radix system: as many columns
per lane as divide them, up to 8, by default (bitwise the explicit 8's products where 8
divides them), and every explicit number; elementwise against the oracle."""
import numpy as np
import pytest

import ftlm_workloads as W
from oracle import ftlm as of

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("two_s", [[2] * 8, [5, 4, 4, 4, 4]])
@pytest.mark.parametrize("K", [1, 2, 3, 4, 8, 16])
def test_window_columns(two_s, K):
    import paper_2607_25585_amd as F
    rng = np.random.default_rng(K)
    n = len(two_s)
    sysm = W.System(two_s=np.array(two_s, np.int32), J=np.triu(rng.uniform(-1, 1, (n, n)), 1), d=rng.uniform(-2, 2, n),
                    e=W.unit_vectors(rng, n), g=np.full(n, 2.0), B=rng.uniform(-1, 1, 3), pos=W.unit_vectors(rng, n))
    ham, ref = F.Hamiltonian(sysm), of.Ham(sysm)
    v = rng.standard_normal((ham.dim, K)) + 1j * rng.standard_normal((ham.dim, K))
    want = np.stack([ref.apply(v[:, c].copy()) for c in range(K)], axis=1)
    for prec, dt, tol in ((F.FTLM_C128, torch.complex128, 1e-12), (F.FTLM_C64, torch.complex64, 2e-5)):
        x = torch.as_tensor(v, device="cuda").to(dt)
        got = {}
        for kc in (0, 1, 2, 4, 8):
            print("case window columns", two_s, K, dt, kc, flush=True)
            ham.set_tuning(prec, K, 4, 0, kc)
            got[kc] = ham.apply(x).cpu().numpy()
            assert np.max(np.abs(got[kc] - want)) < tol * np.max(np.abs(want))
        assert np.array_equal(got[0], got[8])
    a = []
    for kc in (0, 1):
        ham.set_tuning(F.FTLM_C128, K, 4, 0, kc)
        a.append(F.run(ham, K, 3, np.array([1.0, 10.0]), seed=3, columns=K, return_tridiagonals=True))
    scale = np.max(np.abs(a[0]["alpha"])) + np.max(np.abs(a[0]["beta"]))
    for k in ("alpha", "beta"):
        assert np.max(np.abs(a[0][k] - a[1][k])) < 1e-11 * scale
