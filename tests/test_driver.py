"""The cache object of block prompt processing (Sec. 2.2): what it holds."""
import torch

from paper_2609_23314_amd import vd
from paper_2609_23314_amd.driver import EvictingCache


def test_cache_keeps_no_scratch(monkeypatch):
    """A cache holds what its constructor made and nothing of a pass: one made (or
    pickled) with these attributes alone evicts, and is left with them."""
    names = {"k", "v", "units", "n", "seen", "budget", "variant", "num_q_heads", "running_sum", "pos", "capacity"}
    made = EvictingCache(1, 1, 1, 64, 8, [4], dtype=torch.float32, device="cpu")
    cache = EvictingCache.__new__(EvictingCache)
    cache.__dict__.update({a: getattr(made, a) for a in names})
    monkeypatch.setattr(vd, "vd_evict_step", lambda *a, **kw: None)
    cache.n = [6]
    cache.evict()
    assert cache.n == [4] and set(vars(cache)) == names == set(vars(made))
