"""The tile sweep (variant 6, general radix) for every number of rows per thread it is
built for, threads that have no rows, tops that it leaves to the fallback kernel,
tiles dealt to few and to many blocks, staged and direct shifted reads, sparse and
dense couplings, single flips by one and by two; elementwise against the oracle, and
the Lanczos sums through a short run's tridiagonal."""
import numpy as np
import pytest

import ftlm_workloads as W
from oracle import ftlm as of

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (2 s of every site; what couples).  The tile takes the low sites up to 4096 (8192)
# rows and 1024 threads.
SYSTEMS = {
    "top3": [2] * 11, "top4": [3] * 9, "top5": [4] * 8, "top6": [5] * 7,
    "mixed5": [5, 4, 4, 4, 4, 4, 3], "mixed3": [1, 4, 2, 6, 2, 3, 2, 1, 4, 1], "mixed4": [7, 3, 3, 3, 3, 3, 2, 1],
    "fallback2": [3, 3, 3, 1, 1, 1, 1, 1, 1, 1, 3, 3], "fallback7": [6] * 6, "fallback16": [15] * 4,
}


def _system(two_s, couple, seed):
    rng = np.random.default_rng(seed)
    n = len(two_s)
    J = np.triu(rng.uniform(-1, 1, (n, n)), 1)
    pos = None
    if couple == "sparse":
        J *= np.abs(np.subtract.outer(np.arange(n), np.arange(n))) <= 1
    else:  # a planar ring: every ladder term, no s+- s^z pieces
        ang = 2 * np.pi * np.arange(n) / n
        pos = 0.6 * np.stack([np.cos(ang), np.sin(ang), np.zeros(n)], 1)
    single = couple != "sparse"
    return W.System(two_s=np.array(two_s, np.int32), J=J, d=rng.uniform(-2, 2, n) if single else None,
                    e=W.unit_vectors(rng, n), g=np.full(n, 2.0), B=rng.uniform(-1, 1, 3) if single else
                    np.array([0.0, 0.0, 1.0]), pos=pos, name=couple)


@pytest.mark.parametrize("couple", ["sparse", "dense"])
@pytest.mark.parametrize("name", sorted(SYSTEMS))
def test_sweep_matches_oracle(name, couple):
    import paper_2607_25585_amd as F
    sysm = _system(SYSTEMS[name], couple, 11)
    ham, ref = F.Hamiltonian(sysm), of.Ham(sysm)
    rng = np.random.default_rng(5)
    v = rng.standard_normal(ham.dim) + 1j * rng.standard_normal(ham.dim)
    want = ref.apply(v)
    for cap, kc in ((0, 0), (8, 0x20), (3, 0x40), (0, 0x100)):
        print("case", name, couple, "dim", ham.dim, "grid", cap, "kc", hex(kc), flush=True)
        for prec, dt, tol in ((F.FTLM_C128, torch.complex128, 1e-12), (F.FTLM_C64, torch.complex64, 2e-5)):
            ham.set_tuning(prec, 1, 6, cap, kc)
            got = ham.apply(torch.as_tensor(v, device="cuda").to(dt)).cpu().numpy()
            assert np.max(np.abs(got - want)) < tol * np.max(np.abs(want))
    T = np.array([1.0, 10.0])
    ham.set_tuning(F.FTLM_C128, 1, 6)
    a = F.run(ham, 1, 5, T, seed=3, columns=1, return_tridiagonals=True)
    ham.set_tuning(F.FTLM_C128, 1, 1)
    b = F.run(ham, 1, 5, T, seed=3, columns=1, return_tridiagonals=True)
    scale = np.max(np.abs(b["alpha"])) + np.max(np.abs(b["beta"]))
    for k in ("alpha", "beta"):
        assert np.max(np.abs(a[k] - b[k])) < 1e-11 * scale
    assert np.max(np.abs(a["M"] - b["M"])) < 1e-9 * np.max(np.abs(b["M"]))
