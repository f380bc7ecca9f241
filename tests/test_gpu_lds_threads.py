"""Products from several host threads at a time, each on a stream of its own, with kernels
whose LDS exceeds 64 KB by different amounts: bitwise what one thread gets."""
import threading

import numpy as np
import pytest

import ftlm_workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_threads_with_different_lds():
    import paper_2607_25585_amd as F
    cases = []
    for two_s, variant, c64 in (([5, 4, 4, 4, 4, 4, 3], 6, False), ([3] * 9, 6, False), ([2] * 11, 6, False),
                                ([1] * 18, 5, False), ([1] * 13, 5, False), ([4] * 8, 6, True)):
        n = len(two_s)
        rng = np.random.default_rng(n)
        sysm = W.System(two_s=np.array(two_s, np.int32), J=np.triu(rng.uniform(-1, 1, (n, n)), 1), d=None,
                        e=np.tile([0.0, 0.0, 1.0], (n, 1)), g=np.full(n, 2.0), B=rng.uniform(-1, 1, 3), pos=None)
        ham = F.Hamiltonian(sysm)
        ham.set_tuning(F.FTLM_C64 if c64 else F.FTLM_C128, 1, variant)
        v = torch.as_tensor(rng.standard_normal(ham.dim) + 1j * rng.standard_normal(ham.dim), device="cuda")
        cases.append((ham, v.to(torch.complex64) if c64 else v))
    torch.cuda.synchronize()
    got, bad = [None] * len(cases), []

    def work(i):
        try:
            ham, v = cases[i]
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                for _ in range(20):
                    got[i] = ham.apply(v)
            s.synchronize()
        except Exception as e:  # reported by the main thread
            bad.append((i, e))

    print("case threads", len(cases), flush=True)
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(cases))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    for (ham, v), w in zip(cases, got):
        assert torch.equal(ham.apply(v), w)
