"""The binned sweep by panels with more panels than fit the chip at once: a
workgroup takes several in turn, and the first one does the step as well."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

RADIX = (64, 56, 40, 3)


@pytest.fixture(scope="module")
def plan():
    import torch
    from paper_2210_01465_amd import api
    rng = np.random.default_rng([29, 1])
    f = np.exp(0.3 * rng.standard_normal(int(np.prod(RADIX)))).astype(np.float32)
    f[rng.random(f.size) < 0.2] = np.nan
    with api.Context(0) as ctx:
        plan = api.plan_create(ctx, RADIX, torch.from_numpy(f).cuda(), "hamming")
        assert plan.sizes["mask_words"] == 0
        yield plan
        plan.close()


def test_equals_tiles_and_a_step_kernel(plan):
    from paper_2210_01465_amd import api
    print("[case] panels exact", flush=True)
    runs = [api.execute(plan, 1.0, 0.05, row_mapping=-2, exact=True, separate_step=sep) for sep in (False, True)]
    (a, _, ia), (b, _, ib) = runs
    assert ia["iterations"] == ib["iterations"]
    # the same FP32 iterates; the final FP64 scale sums N terms in another order
    assert np.allclose(a.cpu().numpy(), b.cpu().numpy(), rtol=plan.n_valid * 2.0 ** -53, atol=0.0)
    print("[case] panels power iteration", flush=True)
    (a, _, ia), (b, _, ib) = [api.execute(plan, 0.85, 0.05, row_mapping=-2, separate_step=sep) for sep in (False, True)]
    # each sweep rounds a rank of sum 1 to 2^-24, on either side
    assert float((a - b).abs().sum()) <= 2 * (ia["iterations"] + 1) * 2.0 ** -24
    assert abs(ia["iterations"] - ib["iterations"]) <= 1


@pytest.mark.parametrize("cap", [1, 2, 3, 6, 9, 0])
def test_stops_beside_another_stream(plan, cap):
    """Workgroups of one sweep start late when another stream holds the CUs,
    so some see the stop that the first one sets: same ranks, bit for bit."""
    import torch
    from paper_2210_01465_amd import api
    print(f"[case] panels stop cap {cap}", flush=True)
    quiet, _, info = api.execute(plan, 0.85, 0.05, max_iter=cap, allow_noconv=True)
    assert cap == 0 or info["iterations"] == cap
    other = torch.cuda.Stream()
    m = torch.ones(2048, 2048, dtype=torch.bfloat16, device="cuda")
    torch.cuda.synchronize()
    for _ in range(4):
        with torch.cuda.stream(other):
            for _ in range(100):
                m @ m
        ranks, _, got = api.execute(plan, 0.85, 0.05, max_iter=cap, allow_noconv=True)
        assert got["iterations"] == info["iterations"] and torch.equal(ranks, quiet)
    torch.cuda.synchronize()


# On either side of the lines between panels and tiles: edges, nodes, edges
# per node (16, 32 and 80), and edges per node against nodes
SIDES = [((70, 60, 11), 0.0), ((70, 60, 11), 0.5), ((300, 170), 0.0), ((300, 150), 0.0), ((64, 50, 40, 2), 0.8),
         ((64, 50, 40, 5), 0.85), ((600, 100), 0.0), ((3000,), 0.0)]


@pytest.mark.parametrize("radix,excluded", SIDES)
def test_either_side_equals_the_step_kernel(radix, excluded):
    import torch
    from paper_2210_01465_amd import api
    rng = np.random.default_rng([41, len(radix)])
    f = np.exp(0.3 * rng.standard_normal(int(np.prod(radix)))).astype(np.float32)
    f[rng.random(f.size) < excluded] = np.nan
    with api.Context(0) as ctx:
        plan = api.plan_create(ctx, radix, torch.from_numpy(f).cuda(), "hamming")
        print(f"[case] {radix} excluded {excluded}: {plan.n_valid} nodes, {plan.n_edges} edges", flush=True)
        for exact in (True, False):
            (a, ma, ia), (b, mb, ib) = [api.execute(plan, 0.85, 0.05, exact=exact, separate_step=sep)
                                        for sep in (False, True)]
            assert torch.equal(ma, mb) and abs(ia["iterations"] - ib["iterations"]) <= (0 if exact else 1)
            if exact:
                assert np.allclose(a.cpu().numpy(), b.cpu().numpy(), rtol=plan.n_valid * 2.0 ** -53, atol=0.0)
            else:
                assert float((a - b).abs().sum()) <= 2 * (ia["iterations"] + 1) * 2.0 ** -24
        plan.close()
