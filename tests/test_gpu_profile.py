"""Times of single sweeps (fl_profile) over long runs."""
import failing_malloc
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("separate", [False, True])
@pytest.mark.parametrize("every", [1, 7])
def test_long_runs_take_no_more_events(every, separate):
    """A path of 1 500 nodes settles after as many exact sweeps: each sampled
    one that did work is counted, and the context keeps no more events than for
    a short run."""
    failing_malloc.run(f"every, separate = {every}, {separate}\n" + r"""
import numpy as np, torch
from paper_2210_01465_amd import api
with api.Context(0) as ctx:
    f = torch.from_numpy(np.arange(1, 1501, dtype=np.float32)).cuda()
    plan = api.plan_create(ctx, (1500,), f, "adjacent")
    api.profile(ctx, every)
    before = failing_malloc.events()
    for _ in range(2):
        info = api.execute(plan, 1.0, exact=True, separate_step=separate)[2]
        t = api.plan_timing(plan)
        print(info["iterations"], t, failing_malloc.events() - before)
        assert t["iterations"] >= 1499 and t["sweeps_timed"] == -(-t["iterations"] // every)
        assert 0.0 < t["sweep_ms"] <= t["pagerank_ms"]
    assert failing_malloc.events() - before <= 128
    plan.close()
""")


def test_iterate_time_leaves_out_the_round_trips():
    """With a step kernel per sweep the host reads the state between chunks of
    launches: that time is in pagerank_ms and not in iterate_ms."""
    import torch
    from paper_2210_01465_amd import api, synth
    s = synth.tiny(3)
    with api.Context(0) as ctx:
        plan = api.plan_create(ctx, s.radix, torch.from_numpy(s.fitness_raw).cuda())
        kw = dict(tol=1e-30, max_iter=400, allow_noconv=True)   # never met: chunks of 8 to the cap
        best = {}
        for sep in (True, False):
            for _ in range(3):
                api.execute(plan, 0.85, separate_step=sep, **kw)
                t = api.plan_timing(plan)
                print(sep, t, flush=True)
                best[sep] = min(best.get(sep, 1.0), t["iterate_ms"] / t["pagerank_ms"])
        assert 0.0 < best[True] < 0.95 and 0.0 < best[False] <= 1.0
        plan.close()


def test_a_failed_call_leaves_no_sweeps_behind():
    """A call that fails among its sweeps leaves none that could report a stop
    to the next one (here: an event that cannot be created)."""
    failing_malloc.run(r"""
import numpy as np, torch
from paper_2210_01465_amd import _abi, api
radix = (12, 10, 6, 5, 4, 4, 3, 3, 3, 3)   # sweeps long enough to be under way for a while
f = torch.from_numpy(np.random.default_rng(3).lognormal(0.0, 0.5, int(np.prod(radix))).astype(np.float32)).cuda()
with api.Context(0) as ctx:
    plan = api.plan_create(ctx, radix, f)
    want, _, info = api.execute(plan, 0.85)
    plan.close()
last = 0
for launch in range(info["iterations"] - 1, info["iterations"] + 5):   # one that follows the last sweep closely
    with api.Context(0) as ctx:
        plan = api.plan_create(ctx, radix, f)
        got = torch.empty_like(want)
        api.profile(ctx, 1)
        failing_malloc.fail_event(2 * launch)
        try:
            api.execute(plan, 0.85)
        except api.FLError as e:
            assert e.status == _abi.FL_EHIP
            last = launch
        now = api.execute(plan, 0.85, pagerank=got)[2]
        assert now["iterations"] == info["iterations"] and torch.equal(got, want), (launch, info, now)
        failing_malloc.fail_event(-1)
        plan.close()
print(info["iterations"], "iterations; last refused at launch", last)
assert last >= info["iterations"]
""")
