"""The tuning cache: a choice timed among earlier launches is not replayed."""
from types import SimpleNamespace

import numpy as np

from paper_2607_25585_amd import autotune


def test_key_names_the_launches(monkeypatch):
    ham = SimpleNamespace(n_sites=4, _J=np.ones((4, 4)), _d=None, _pos=None, _two_s=np.ones(4, np.int32))
    key = autotune.tuning_key(ham, 0, 2)
    assert key.startswith("n4-s") and "-p0-k2" in key and not key.endswith("-p0-k2")
    batched = autotune.batched_key([ham], 0, 8)
    monkeypatch.setattr(autotune, "LAUNCHES", autotune.LAUNCHES + 1)
    assert autotune.tuning_key(ham, 0, 2) != key
    assert autotune.batched_key([ham], 0, 8) == batched  # (its launches are other ones)
