"""The two forms of the one-node-per-lane sweep: in-edge lists (small graphs)
and slot records (the others), each against the one-lane CSR sweep, which
adds the same terms in the same order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SLOTS = -1


def fitness(radix, seed, excluded):
    rng = np.random.default_rng([13, seed])
    f = np.exp(0.3 * rng.standard_normal(int(np.prod(radix)))).astype(np.float32)
    f[rng.random(f.size) < excluded] = np.nan
    f[int(rng.integers(f.size))] = 1.0
    return f


# (radices, neighbourhood, excluded share, mask words).  Lists: one node; waves
# of 63, 64 and 65 nodes; complete graphs, whose longest lists take 1 to 8
# groups of 16 steps; a space with no excluded configuration (its zero entry
# follows the last node); one wave per workgroup up to 131 072 nodes, four
# above.  Slots, more than 1.8 M edges: record widths 1 to 5.
LISTS = [((1,), "hamming", 0.0, 1), ((63,), "hamming", 0.0, 3), ((64,), "adjacent", 0.0, 1), ((65,), "hamming", 0.0, 3),
         ((129,), "hamming", 0.0, 5), ((16,), "hamming", 0.0, 2), ((4, 4, 4), "hamming", 0.0, 1),
         ((5, 5, 5, 5, 5), "hamming", 0.9, 2), ((9, 8, 6, 5, 4, 4, 3, 3), "hamming", 0.62, 2),
         ((9, 8, 6, 5, 4, 4, 3, 3), "adjacent", 0.4, 1)]
RECORDS = [((12, 11, 10, 9, 8, 4), "adjacent", 0.0, 1), ((9, 8, 6, 5, 4, 4, 3, 3), "hamming", 0.2, 2),
           ((26, 26, 25, 3), "hamming", 0.0, 3), ((40, 40, 30), "hamming", 0.05, 4), ((50, 50, 30), "hamming", 0.3, 5)]


@pytest.mark.parametrize("radix,nb,excluded,words", LISTS + RECORDS)
def test_equals_csr_sweep(radix, nb, excluded, words):
    import torch
    from paper_2210_01465_amd import api
    f = fitness(radix, len(radix), excluded)
    print(f"[case] {radix} {nb} excluded {excluded}", flush=True)
    with api.Context(0) as ctx:
        plan = api.plan_create(ctx, radix, torch.from_numpy(f).cuda(), nb)
        assert plan.sizes["mask_words"] == words
        assert (plan.n_edges <= 7 << 18) == ((radix, nb, excluded, words) in LISTS)
        runs = {}
        for layout in (SLOTS, 1):
            for kw in ({"separate_step": True}, {}, {"exact": True}):
                pr, _, info = api.execute(plan, 0.85, 0.05, row_mapping=layout, **kw)
                runs[layout, tuple(kw)] = pr.cpu().numpy(), info["iterations"]
        # a step kernel per sweep: every sum has the same order
        a, b = runs[SLOTS, ("separate_step",)], runs[1, ("separate_step",)]
        assert a[1] == b[1] and np.array_equal(a[0], b[0])
        # exact iterates are the same bits; the final scale's FP64 sum has another order
        a, b = runs[SLOTS, ("exact",)], runs[1, ("exact",)]
        assert a[1] == b[1] and np.allclose(a[0], b[0], rtol=plan.n_valid * 2.0 ** -53, atol=0.0)
        # the lagged step's constants differ in FP64 rounding: a rare last bit of an FP32 iterate
        a, b = runs[SLOTS, ()], runs[1, ()]
        assert a[1] == b[1] and float(np.abs(a[0] - b[0]).sum()) <= 2.0 ** -24
        plan.close()
