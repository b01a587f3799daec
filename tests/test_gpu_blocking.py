"""Waits that block: with hipDeviceScheduleBlockingSync or
hipDeviceScheduleYield set for the device the calls wait in the runtime instead
of polling, and give the same results."""
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

SCRIPT = r"""
import ctypes, sys
import numpy as np, torch
want = int(sys.argv[1])
torch.zeros(1, device="cuda")
path = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
hip, flags = ctypes.CDLL(path), ctypes.c_uint(99)
if want:
    assert hip.hipSetDeviceFlags(want) == 0
assert hip.hipGetDeviceFlags(ctypes.byref(flags)) == 0
assert want == 0 or flags.value & want
from paper_2210_01465_amd import api
radix = (32, 32, 32, 32)
f = torch.from_numpy(np.random.default_rng(7).lognormal(0.0, 0.5, int(np.prod(radix))).astype(np.float32)).cuda()
small = f[:1000].clone()
with api.Context(0) as ctx:
    plan = api.plan_create(ctx, radix, f)
    out = []
    for kw in (dict(damping=0.85), dict(damping=0.85, max_iter=5, allow_noconv=True), dict(damping=1.0, exact=True)):
        pr, mins, info = api.execute(plan, **kw)
        out += [float(pr.sum()), float(pr.square().sum()), int(mins.sum()), info["iterations"]]
    r = api.analyze((10, 10, 10), small, ctx=ctx)
    out += [r.score, r.info["iterations"]]
    plan.close()
print(out)
"""


def test_waits_that_block_give_the_same_results():
    got = []
    for flags in (0, 4, 2):
        print("[case] device flags", flags, flush=True)
        p = subprocess.run([sys.executable, "-u", "-c", SCRIPT, str(flags)], capture_output=True, text=True, timeout=30)
        assert p.returncode == 0, p.stderr
        got.append(p.stdout)
    assert got[0] and got[1] == got[0] and got[2] == got[0], got
