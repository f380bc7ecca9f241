"""The tile sweep where the values below its top tile site fill one wave or less: mixed
radices whose tile ends early because the next site has too many values for it.  Every
element against the oracle, with several outer sites and z-z couplings to them, by the
explicit launch and, from 2^20 rows, by the built-in one."""
import numpy as np
import pytest

import ftlm_workloads as W
from oracle import ftlm as of

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _system(two_s, couple):
    rng = np.random.default_rng(3)
    n = len(two_s)
    J = np.triu(rng.uniform(-1, 1, (n, n)), 1)
    if couple == "chain":
        J *= np.subtract.outer(np.arange(n), np.arange(n)) == -1
    return W.System(two_s=np.array(two_s, np.int32), J=J, d=rng.uniform(-2, 2, n), e=W.unit_vectors(rng, n),
                    g=np.full(n, 2.0), B=rng.uniform(-1, 1, 3), pos=None, name=couple)


# values below the top tile site: 64, 49, 52, 48
@pytest.mark.parametrize("couple", ["all", "chain"])
@pytest.mark.parametrize("two_s,variant", [([7, 7, 5, 15, 15], 6), ([6, 6, 5, 15, 15], 6), ([3, 12, 4, 15, 15], 6),
                                           ([2, 15, 5, 15, 15], 6), ([7, 7, 5, 15, 15, 15], 0)])
def test_narrow_tiles_match_oracle(two_s, variant, couple):
    import paper_2607_25585_amd as F
    sysm = _system(two_s, couple)
    ham, ref = F.Hamiltonian(sysm), of.Ham(sysm)
    rng = np.random.default_rng(5)
    v = rng.standard_normal(ham.dim) + 1j * rng.standard_normal(ham.dim)
    want = ref.apply(v)
    for prec, dt, tol in ((F.FTLM_C128, torch.complex128, 1e-12), (F.FTLM_C64, torch.complex64, 2e-5)):
        print("case", couple, two_s, "dim", ham.dim, dt, flush=True)
        ham.set_tuning(prec, 1, variant)
        got = ham.apply(torch.as_tensor(v, device="cuda").to(dt)).cpu().numpy()
        assert np.max(np.abs(got - want)) < tol * np.max(np.abs(want))
    ham.set_tuning(F.FTLM_C128, 1, variant)
    a = F.run(ham, 1, 4, np.array([1.0, 10.0]), seed=3, columns=1, return_tridiagonals=True)
    ham.set_tuning(F.FTLM_C128, 1, 1)
    b = F.run(ham, 1, 4, np.array([1.0, 10.0]), seed=3, columns=1, return_tridiagonals=True)
    scale = np.max(np.abs(b["alpha"])) + np.max(np.abs(b["beta"]))
    for k in ("alpha", "beta"):
        assert np.max(np.abs(a[k] - b[k])) < 1e-11 * scale
