"""The server's account of a plan's device memory."""
from types import SimpleNamespace

import pytest

from paper_2210_01465_amd.serve import GpuBackend


# sparse spaces of many nodes, whose lists the engine would not make, and small ones
@pytest.mark.parametrize("n_raw,n,e,slots,words", [(40_000_000, 3_000_000, 1_800_000, 86, 2),
                                                   (20_000_000, 1_500_000, 400_000, 60, 2),
                                                   (1_000_000, 900_000, 7 << 18, 20, 1),
                                                   (100_000, 60_000, 1_000_000, 66, 2), (129, 100, 600, 22, 1),
                                                   (400_000, 350_000, 26_000_000, 320, 0)])
def test_lists_count_for_at_most_their_limit(n_raw, n, e, slots, words):
    sizes = dict(n_raw=n_raw, n_valid=n, n_edges=e, n_slots=slots, mask_words=words)
    got = GpuBackend.plan_bytes(None, SimpleNamespace(sizes=sizes))
    base = n_raw * 16 + n * (8 * max(words, 1) + 28) + 4 * e
    assert base <= got <= base + (64 << 20)
    # the lists that the engine does make: a stride of whole quads for the longest list, and a group more
    quads = max((slots // 2 + 3) // 4, 4) + 4
    made = (n + 63) // 64 * (quads * 1024 + 4)
    if words and e <= 7 << 18 and made + base <= 64 << 20:
        assert got >= base + made
