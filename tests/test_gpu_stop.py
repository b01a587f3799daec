"""Where the lagged sweeps stop: at an iteration cap and at the tolerance, as
with a step kernel per sweep, however far ahead the host has launched."""
import numpy as np
import pytest

from paper_2210_01465_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("exact", [False, True])
@pytest.mark.parametrize("cap", [1, 2, 3, 5, 6, 7, 8, 13, 0])
@pytest.mark.parametrize("layout", [-1, 1, -2])
def test_stops_where_the_step_kernel_does(cap, exact, layout):
    import torch
    from paper_2210_01465_amd import _abi, api
    s = synth.tiny(5)
    print(f"[case] cap {cap} exact {exact} layout {layout}", flush=True)
    with api.Context(0) as ctx:
        plan = api.plan_create(ctx, s.radix, torch.from_numpy(s.fitness_raw).cuda())
        runs = [api.execute(plan, 0.85, 0.05, max_iter=cap, row_mapping=layout, allow_noconv=True, exact=exact,
                            separate_step=sep) for sep in (True, False)]
        (a, _, ia), (b, _, ib) = runs
        assert ia["iterations"] == ib["iterations"] and ia["status"] == ib["status"]
        assert ia["status"] == (_abi.FL_OK if cap == 0 else _abi.FL_ENOCONV) and (cap == 0 or ia["iterations"] == cap)
        # FP32 iterates of FP64 constants that differ in rounding: each of at
        # most 60 sweeps rounds a rank of sum 1 to 2^-24, on either side
        assert float((a - b).abs().sum()) <= 60 * 2.0 ** -23
        assert np.isclose(ia["residual_l1"], ib["residual_l1"], rtol=1e-3, atol=60 * 2.0 ** -23)
        plan.close()
