"""The general-radix direct gather on both sides of the rule that picks a lane per row or
lanes that share a row: sites of two values (few valid moves) and of more, columns that
one lane takes and others, from the sizes where the choice changes; elementwise against
the oracle, and the Lanczos sums of several columns against those of one."""
import numpy as np
import pytest

import ftlm_workloads as W
from oracle import ftlm as of

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SYSTEMS = {
    "half-98304": [2] + [1] * 15, "half-49152": [1] * 14 + [2], "alternating": [1, 2] * 6 + [1], "s1-177147": [2] * 11,
    "s32-262144": [3] * 9, "s32-65536": [3] * 8, "s3-117649": [6] * 6,
}


def _system(two_s, couple):
    rng = np.random.default_rng(len(two_s))
    n = len(two_s)
    J = np.triu(rng.uniform(-1, 1, (n, n)), 1)
    pos = W.unit_vectors(rng, n) if couple == "dipolar" else None
    if couple == "chain":
        J *= np.subtract.outer(np.arange(n), np.arange(n)) == -1
    return W.System(two_s=np.array(two_s, np.int32), J=J, d=rng.uniform(-2, 2, n), e=W.unit_vectors(rng, n),
                    g=np.full(n, 2.0), B=rng.uniform(-1, 1, 3), pos=pos, name=couple)


@pytest.mark.parametrize("couple", ["dipolar", "chain"])
@pytest.mark.parametrize("name", sorted(SYSTEMS))
def test_direct_gather_matches_oracle(name, couple):
    import paper_2607_25585_amd as F
    sysm = _system(SYSTEMS[name], couple)
    ham, ref = F.Hamiltonian(sysm), of.Ham(sysm)
    rng = np.random.default_rng(5)
    v = rng.standard_normal((ham.dim, 5)) + 1j * rng.standard_normal((ham.dim, 5))
    want = np.stack([ref.apply(v[:, c].copy()) for c in range(5)], axis=1)
    big = np.max(np.abs(want))
    for K in (1, 2, 3, 4, 5, 6, 8, 12, 20):
        cols = [c % 5 for c in range(K)]
        x = np.ascontiguousarray(v[:, cols]) if K > 1 else v[:, 0].copy()
        w = want[:, cols] if K > 1 else want[:, 0]
        for prec, dt, tol in ((F.FTLM_C128, torch.complex128, 1e-12), (F.FTLM_C64, torch.complex64, 2e-5)):
            for kc in (0, 1, 8):
                print("case direct gather", name, couple, "K", K, dt, "kc", kc, flush=True)
                ham.set_tuning(prec, K, 1, 0, kc)
                got = ham.apply(torch.as_tensor(x, device="cuda").to(dt)).cpu().numpy()
                assert np.max(np.abs(got - w)) < tol * big
    T = np.array([1.0, 10.0])
    runs = []
    for K in (1, 3, 4):
        ham.set_tuning(F.FTLM_C128, K, 1)
        runs.append(F.run(ham, 12, 3, T, seed=3, columns=K, return_tridiagonals=True))
    scale = np.max(np.abs(runs[0]["alpha"])) + np.max(np.abs(runs[0]["beta"]))
    for r in runs[1:]:
        for k in ("alpha", "beta"):
            assert np.max(np.abs(r[k] - runs[0][k])) < 1e-11 * scale
        assert np.max(np.abs(r["M"] - runs[0]["M"])) < 1e-9 * np.max(np.abs(runs[0]["M"]))
