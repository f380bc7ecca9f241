"""The LDS tile kernel over L2 windows (variant 5) for the columns that the half sweep does
not take: 3, and 2, 4, 8 of few rows, with 256, 512 and 1024 threads per tile, over one
and over many windows, with and without s+- s^z pieces; elementwise against the oracle,
and the Lanczos sums against the direct gather's."""
import numpy as np
import pytest

import ftlm_workloads as W
from oracle import ftlm as of

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("couple", ["dipolar", "exchange"])
@pytest.mark.parametrize("tile_kb", [0, 128])
@pytest.mark.parametrize("n,K", [(12, 3), (13, 2), (14, 8), (13, 4), (16, 3), (17, 5)])
def test_tile_columns_match_oracle(n, K, tile_kb, couple, plan_windows):
    import paper_2607_25585_amd as F
    plan_windows(tile_kb=tile_kb)
    rng = np.random.default_rng(n)
    sysm = W.System(two_s=np.ones(n, np.int32), J=np.triu(rng.uniform(-1, 1, (n, n)), 1), d=None,
                    e=np.tile([0.0, 0.0, 1.0], (n, 1)), g=np.full(n, 2.0), B=rng.uniform(-1, 1, 3),
                    pos=W.unit_vectors(rng, n) if couple == "dipolar" else None, name=couple)
    ham, ref = F.Hamiltonian(sysm), of.Ham(sysm)
    v = rng.standard_normal((ham.dim, K)) + 1j * rng.standard_normal((ham.dim, K))
    want = np.stack([ref.apply(v[:, c].copy()) for c in range(K)], axis=1)
    T = np.array([1.0, 10.0])
    ham.set_tuning(F.FTLM_C128, K, 1)
    b = F.run(ham, K, 3, T, seed=3, columns=K, return_tridiagonals=True)
    scale = np.max(np.abs(b["alpha"])) + np.max(np.abs(b["beta"]))
    for groups in (0, 1, 2, 4):
        for cap in (0, 5):
            print("case tile columns", couple, n, K, "groups", groups, "grid", cap, "window", tile_kb, flush=True)
            for prec, dt, tol in ((F.FTLM_C128, torch.complex128, 1e-12), (F.FTLM_C64, torch.complex64, 2e-5)):
                ham.set_tuning(prec, K, 5, cap, groups)
                got = ham.apply(torch.as_tensor(v, device="cuda").to(dt)).cpu().numpy()
                assert np.max(np.abs(got - want)) < tol * np.max(np.abs(want))
        a = F.run(ham, K, 3, T, seed=3, columns=K, return_tridiagonals=True)
        for k in ("alpha", "beta"):
            assert np.max(np.abs(a[k] - b[k])) < 1e-11 * scale
