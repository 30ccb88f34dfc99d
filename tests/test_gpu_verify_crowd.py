"""FP64 verify with many circles in one place, around the number of candidates
from which they are all taken in FP64, against the oracle; a circle of the
crowd that is not finite, and coordinates far outside."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("crowd", [20, 31, 32, 33, 34, 35, 36, 37, 64, 130, 299])
@pytest.mark.parametrize("centre", [0.0, 3e18, -3e38])
def test_crowd(crowd, centre):
    import paper_2303_02650_amd as P

    rng = synth.rng_for(crowd)
    R = 22.0
    x = synth.disk_uniform(300, R, rng)
    who = rng.choice(300, size=crowd, replace=False)
    x[who] = rng.uniform(-0.9, 0.9, size=(crowd, 2)) + [centre, 5.0]
    inst = synth.pack([x, x[who], x], [R, R, R])
    flat = inst.xy.reshape(-1).copy()
    flat[2 * (inst.offset[2] + who[crowd // 2])] = np.nan
    d = P.DeviceInstances.from_host(inst.offset, inst.R)
    e, mp, mc, f = [t.cpu().numpy() for t in P.verify(d, torch.from_numpy(flat).cuda())]
    for b in range(2):
        v = oracle.verify(inst.instance(b), R)
        # FP64 sums of non-negative terms in another order
        assert abs(e[b] - v["E"]) <= 1e-12 * v["E"]
        assert bool(f[b]) == v["feasible"]
        # four FP64 steps of the distance
        assert abs(mp[b] - v["max_pair_overlap"]) <= 4 * np.finfo(np.float64).eps * 2.0
    assert np.isnan(e[2]) and np.isnan(mp[2]) and np.isnan(mc[2]) and f[2] == 0
