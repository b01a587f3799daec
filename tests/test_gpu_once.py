"""One-shot analyses build only what their sweep reads (in-edge lists, slot
records, or the CSR): the same bits as a kept plan in the same layout."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# lists (one wave, several, every record width up to 5), slot records (more
# than 1.8 M edges), the CSR alone (more than 256 slots)
@pytest.mark.parametrize("radix,excluded", [((1,), 0.0), ((2,), 0.0), ((5, 4, 4, 2), 0.2), ((31, 11, 4, 2, 3), 0.04),
                                            ((60, 20), 0.3), ((65, 65), 0.2), ((9, 8, 6, 5, 4, 4, 3, 2), 0.4),
                                            ((26, 26, 25, 3), 0.0), ((65, 66), 0.3)])
@pytest.mark.parametrize("nb", ["hamming", "adjacent"])
@pytest.mark.parametrize("layout", [0, 4, -2])
def test_one_shot_equals_kept_plan(radix, excluded, nb, layout):
    import torch
    from paper_2210_01465_amd import api
    rng = np.random.default_rng([17, len(radix)])
    f = np.exp(0.3 * rng.standard_normal(int(np.prod(radix)))).astype(np.float32)
    f[rng.random(f.size) < excluded] = np.nan
    f[-1] = 1.0
    fit = torch.from_numpy(f).cuda()
    print(f"[case] once {radix} {nb} layout {layout}", flush=True)
    with api.Context(0) as ctx:
        plan = api.plan_create(ctx, radix, fit, nb)
        ranks, minima, info = api.execute(plan, 0.85, 0.05, row_mapping=layout)
        nodes = api.plan_export(plan)["valid_raw"]
        for no_alloc in (False, True):
            r = api.analyze(radix, fit, nb, 0.85, 0.05, row_mapping=layout, ctx=ctx, no_alloc=no_alloc)
            assert torch.equal(r.pagerank, ranks) and torch.equal(r.minima, minima)
            assert torch.equal(r.valid_raw, nodes) and r.score == info["score"]
            assert r.info["iterations"] == info["iterations"] and r.info["row_mapping"] == info["row_mapping"]
            assert all(r.info[k] == plan.sizes[k] for k in ("n_valid", "n_edges", "n_minima", "n_plateau", "f_opt"))
        plan.close()
