"""The built-in H*v launch on both sides of every size where it changes, against
the oracle (elementwise; complex64 within its storage) and, through a short run's
tridiagonal, with the Lanczos epilogue."""
import numpy as np
import pytest

import ftlm_workloads as W
from oracle import ftlm as of

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _dipolar(n):
    rng = np.random.default_rng(100 + n)
    return W.System(two_s=np.ones(n, np.int32), J=W.ring_couplings(n, 1.0), d=None, e=np.tile([0.0, 0.0, 1.0], (n, 1)),
                    g=np.full(n, 2.0), B=0.5 * W.unit_vectors(rng, 1)[0], pos=W.unit_vectors(rng, n))


@pytest.mark.parametrize("n", [8, 11, 12, 18, 19, 20, 21])
def test_half_default_matches_oracle(n):
    import paper_2607_25585_amd as F
    sysm = _dipolar(n)
    ham, ref = F.Hamiltonian(sysm), of.Ham(sysm)
    rng = np.random.default_rng(n)
    v = rng.standard_normal(ham.dim) + 1j * rng.standard_normal(ham.dim)
    want = ref.apply(v)
    print("case default launch n", n, flush=True)
    for dt, tol in ((torch.complex128, 1e-12), (torch.complex64, 2e-5)):
        got = ham.apply(torch.as_tensor(v, device="cuda").to(dt)).cpu().numpy()
        assert np.max(np.abs(got - want)) < tol * np.max(np.abs(want))
    T = np.array([1.0, 10.0])
    a = F.run(ham, 1, 4, T, seed=3, columns=1, return_tridiagonals=True)
    ham.set_tuning(F.FTLM_C128, 1, 1)
    b = F.run(ham, 1, 4, T, seed=3, columns=1, return_tridiagonals=True)
    scale = np.max(np.abs(b["alpha"])) + np.max(np.abs(b["beta"]))
    assert np.max(np.abs(a["alpha"] - b["alpha"])) < 1e-11 * scale
    assert np.max(np.abs(a["beta"] - b["beta"])) < 1e-11 * scale
