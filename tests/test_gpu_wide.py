"""Spaces with more than 256 candidate slots: the CSR fill and the binned
sweep by panels of rows, at the edges of panels, lanes and batches."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

BINNED = -2


def fitness(radix, seed, excluded):
    rng = np.random.default_rng([11, seed])
    f = np.exp(0.3 * rng.standard_normal(int(np.prod(radix)))).astype(np.float32)
    f[rng.random(f.size) < excluded] = np.nan
    return f


# one list of r values is a complete graph: every in-degree 0 .. r-1 once, so
# every class of lanes, rows of one to eleven rounds of 64, and (700,), whose
# 64-lane class has several panels; the products have panels of every class
# with a ragged last one
@pytest.mark.parametrize("radix,excluded", [((130,), 0.0), ((129, 2), 0.3), ((257,), 0.0), ((700,), 0.0),
                                            ((64, 70, 5), 0.1), ((17, 140), 0.5), ((3, 2, 131), 0.9)])
def test_wide_space(radix, excluded):
    import torch
    from paper_2210_01465_amd import api
    f = fitness(radix, len(radix), excluded)
    print(f"[case] wide {radix} excluded {excluded}", flush=True)
    with api.Context(0) as ctx:
        plan = api.plan_create(ctx, radix, torch.from_numpy(f).cuda(), "hamming")
        assert plan.sizes["mask_words"] == 0
        ref = oracle.analyze(radix, f, oracle.HAMMING, 0.85, 0.05)
        ex = {k: v.cpu().numpy() for k, v in api.plan_export(plan).items()}
        for k in ("valid_raw", "row_ptr", "col_idx", "out_deg"):
            assert np.array_equal(ex[k], getattr(ref.graph, k)), k
        pr, mins, info = api.execute(plan, 0.85, 0.05)
        assert info["row_mapping"] == BINNED and np.array_equal(mins.cpu().numpy(), ref.graph.minima)
        # stopped at 2e-7, FP32 iterates: the bound every sweep is held to
        assert float(np.abs(pr.cpu().numpy() - ref.pagerank).sum()) <= 1e-5
        # the exact method's iterates are the same bits with panels and with
        # tiles and a step kernel (same order of every FP32 sum, same constant);
        # only the final FP64 scale sums in another order: N terms, 2^-53 each
        runs = [api.execute(plan, 1.0, 0.05, row_mapping=BINNED, exact=True, separate_step=sep)
                for sep in (False, True)]
        a, b = (r[0].cpu().numpy() for r in runs)
        assert runs[0][2]["iterations"] == runs[1][2]["iterations"]
        assert np.allclose(a, b, rtol=plan.n_valid * 2.0 ** -53, atol=0.0)
        plan.close()
