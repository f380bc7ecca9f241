"""Products after a change of the field: the plans keep what depends on the pairs alone and
renew what depends on the field, over fields with and without single flips and back."""
import numpy as np
import pytest

import ftlm_workloads as W
from oracle import ftlm as of

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FIELDS = ([0.0, 0.0, 1.0], [0.3, -0.2, 0.7], [0.0, 0.0, -2.0], [1.1, 0.4, 0.0])


def _system(two_s, couple):
    rng = np.random.default_rng(len(two_s))
    n = len(two_s)
    J = np.triu(rng.uniform(-1, 1, (n, n)), 1)
    pos = W.unit_vectors(rng, n) if couple == "dipolar" else None
    d = rng.uniform(-2, 2, n) if max(two_s) > 1 else None
    return W.System(two_s=np.array(two_s, np.int32), J=J, d=d, e=np.tile([0.0, 0.0, 1.0], (n, 1)), g=rng.uniform(1, 3, n),
                    B=np.array(FIELDS[1]), pos=pos, name=couple)


# (the tile sweep takes no s+- s^z pieces)
@pytest.mark.parametrize("two_s,K,variant,couple", [
    (s, K, 5, c) for s, K in (([1] * 13, 1), ([1] * 18, 2), ([1] * 16, 8), ([1] * 15, 16))
    for c in ("dipolar", "exchange")] + [
    ([5, 4, 4, 4, 4, 4, 3], 1, 6, "exchange"), ([2, 3, 1, 4, 2, 2, 3, 3, 2], 1, 6, "exchange"),
    ([1, 2] * 6, 3, 1, "dipolar"), ([2] * 8, 4, 1, "dipolar"), ([2] * 11, 1, 1, "exchange")])
def test_products_follow_the_field(two_s, K, variant, couple):
    import paper_2607_25585_amd as F
    sysm = _system(two_s, couple)
    ham = F.Hamiltonian(sysm)
    rng = np.random.default_rng(1)
    v = rng.standard_normal((ham.dim, K)) + 1j * rng.standard_normal((ham.dim, K))
    cols = range(0, K, 7)
    for B in FIELDS:
        print("case field", len(two_s), K, couple, B, flush=True)
        ham.set_field(B)
        sysm.B = np.array(B)
        ref = of.Ham(sysm)
        want = np.stack([ref.apply(v[:, c].copy()) for c in cols], axis=1)
        for prec, dt, tol in ((F.FTLM_C128, torch.complex128, 1e-12), (F.FTLM_C64, torch.complex64, 2e-5)):
            ham.set_tuning(prec, K, variant)
            x = torch.as_tensor(v if K > 1 else v[:, 0].copy(), device="cuda").to(dt)
            got = ham.apply(x).cpu().numpy().reshape(ham.dim, K)[:, list(cols)]
            assert np.max(np.abs(got - want)) < tol * np.max(np.abs(want))
