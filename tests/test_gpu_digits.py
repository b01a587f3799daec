"""Degrees of the node records against a NumPy count: radices at and around
the powers of two, of one value, and as long as an index allows, in every
record width."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _degrees(f, radix, adjacent):
    """(in, out) degrees of the valid points: valid neighbours of higher, of lower fitness."""
    g = f.reshape(radix)
    din, dout = np.zeros(radix, np.int64), np.zeros(radix, np.int64)
    for axis, r in enumerate(radix):
        for d in (range(1, min(2, r)) if adjacent else range(1, r)):
            lo = tuple(slice(None, r - d) if a == axis else slice(None) for a in range(len(radix)))
            hi = tuple(slice(d, None) if a == axis else slice(None) for a in range(len(radix)))
            up, down = g[lo] < g[hi], g[lo] > g[hi]   # false where either is NaN
            din[lo] += up
            dout[hi] += up
            dout[lo] += down
            din[hi] += down
    ok = ~np.isnan(f)
    return din.reshape(-1)[ok], dout.reshape(-1)[ok]


@pytest.mark.parametrize("radix,nb", [((2, 3, 4, 5, 7, 8, 9), "hamming"), ((1, 17, 1, 16, 15, 1), "hamming"),
                                      ((33, 1, 32, 31, 2), "hamming"), ((63, 64, 1), "hamming"),
                                      ((65, 64), "hamming"), ((3, 1, 104729), "adjacent"),
                                      ((262143, 1, 3), "adjacent"), ((2,) * 18, "adjacent")])
def test_degrees(radix, nb):
    import torch
    from paper_2210_01465_amd import api
    rng = np.random.default_rng([23, len(radix)])
    f = rng.integers(1, 1000, int(np.prod(radix))).astype(np.float32)   # with ties
    f[rng.random(f.size) < 0.2] = np.nan
    f[-1] = 1.0
    print(f"[case] digits {radix} {nb}", flush=True)
    with api.Context(0) as ctx:
        plan = api.plan_create(ctx, radix, torch.from_numpy(f).cuda(), nb)
        e = api.plan_export(plan)
        din, dout = _degrees(f, radix, nb == "adjacent")
        assert np.array_equal(np.diff(e["row_ptr"].cpu().numpy()), din)
        assert np.array_equal(e["out_deg"].cpu().numpy(), dout)
        assert plan.sizes["n_edges"] == din.sum() and plan.sizes["n_minima"] == (dout == 0).sum()
        plan.close()
